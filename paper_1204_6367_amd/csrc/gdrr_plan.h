// LDS of a transport launch: the sizes of what a workgroup keeps there.  Host
// and device agree on them; plain C++, no HIP.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <initializer_list>

namespace gdrr {

// Bytes of cube records per cube in LDS: the all-local instantiations and the
// screened one keep one word (the density bound, whose low 5 bits are zero,
// with a table row there), the others the record as built.
constexpr size_t lds_record_bytes(int local_kind) { return local_kind >= 3 ? 4 : 8; }

// Per wavefront, after the tables and cube records: slots of started photons,
// from a 16-byte boundary.  A slot is a 16-byte word (direction and aim pixel),
// an 8-byte one (distance from the source to the box, energy; the position follows from
// them) and, where a volume may track with a single majorant, the
// distance left to the box (4 bytes): 24 or 28 bytes, so that 32 slots
// (64 where the LDS holds them) take less than the 16 bytes a lane that drawing photons
// ahead took.  With the position in the slot, 36 bytes, launches of local and
// single-majorant volumes lost a workgroup per compute unit (1e7 photons each of
// 128x128x96 and 96x96x64 voxels 7.9 -> 8.6 ms, now 7.8 ms).
constexpr int kMinSlots = 32;                              // (powers of two)
constexpr size_t slots_offset_bytes(size_t tables_and_records_bytes) { return (tables_and_records_bytes + 15) & ~(size_t)15; }
constexpr uint32_t slot_bytes(int local_kind) { return local_kind == 3 || local_kind == 4 ? 24u : 28u; }

// LDS allocation granule of a gfx950 workgroup (160 KiB / 128), as measured by
// calib/lds_granule: three 512-thread workgroups share a compute unit up to 42
// granules (53760 bytes) each, where hipOccupancyMaxActiveBlocksPerMultiprocessor
// still reports three up to 54528.
constexpr size_t kLdsGranule = 1280;

// How a workgroup's LDS is shared out: slots of started photons per wavefront, rows of material
// sets, and the workgroups per compute unit that this leaves (0: it does not fit).
struct LdsPlan {
    int slots, rows, per_cu;
    size_t bytes;
};

// fixed: bytes of the tables and records without set rows; a row takes row_bytes, up to `sets` of
// them are of use; most: the workgroups per compute unit that registers and wavefronts allow;
// wanted: the caller's workgroups per compute unit, or 0.
//
// Rows come before slots, slots before workgroups: a cube whose set has no row costs a loop
// over its materials and a read of its global record at every visit (a screened flight: the
// whole test), which phantoms of 4 materials show while fewer than half of the 11 sets have
// one.  So the plan is the most workgroups, down to half of what would fit, that leave room
// for half of the sets with 64 slots or kMinSlots; where none does, the most workgroups, and rows
// only as they fit.  Screened launches wait on their tests: there the trade stops at 24
// wavefronts per compute unit, and goes on to half of the workgroups for the two commonest sets alone.
// Measured, all-local (2e7 photons, 256x256x160 voxels in cubes of 40 mm, 512 lanes, waits 16): 4 workgroups with
// 64 slots and 2 rows 3.74 ms, 32 and 6 2.90, 3 workgroups with 64 and 8 2.89; three phantoms
// (1.5e7): 3 with 64 and 1 3.61, 3 with 32 and 5 3.29, 2 with 64 and 11 2.96; 256 lanes, waits 32:
// 7 with 32 and none 5.34, 4 with 64 and 6 4.46.  Screened (6e6): 512 lanes 4 with 32 and 2 1.54, 3
// with 32 and 7 1.38; 256 lanes, waits 32, three phantoms (9e6): 3 with 32 and 7 4.39, 4 with 32 and 2 4.26.
inline LdsPlan plan_lds(size_t fixed, size_t row_bytes, int sets, bool screened, int waves, uint32_t slot,
                        size_t lds_max, int most, int wanted) {
    const auto bytes = [&](int rows, int slots) { return slots_offset_bytes(fixed + rows * row_bytes) + (size_t)waves * slots * slot; };
    const auto fit = [&](size_t b) {
        if (b > lds_max) return 0;
        const int n = (int)(lds_max / ((b + kLdsGranule - 1) / kLdsGranule * kLdsGranule));
        return n < most ? n : most;
    };
    int hi = fit(bytes(0, kMinSlots));
    if (hi == 0) return {kMinSlots, 0, 0, bytes(0, kMinSlots)};
    if (wanted > 0 && wanted < hi) hi = wanted;
    const int half = wanted > 0 ? hi : (hi + 1) / 2;
    int nb = hi, slots = 0;
    const auto trade = [&](int rows, int lo) {
        for (int n = hi; n >= lo && slots == 0 && rows > 0; --n)
            for (const int s : {64, kMinSlots})
                if (slots == 0 && fit(bytes(rows, s)) >= n) {
                    nb = n;
                    slots = s;
                }
    };
    if (screened) {
        const int busy = (24 + waves - 1) / waves;
        trade((sets + 1) / 2, hi < busy ? hi : half > busy ? half : busy);
        trade(sets < 2 ? sets : 2, half);
    } else {
        trade((sets + 1) / 2, half);
    }
    if (slots == 0) slots = fit(bytes(0, 64)) >= nb ? 64 : kMinSlots;
    int rows = 0;
    while (rows < sets && fit(bytes(rows + 1, slots)) >= nb) ++rows;
    return {slots, rows, fit(bytes(rows, slots)), bytes(rows, slots)};
}

}  // namespace gdrr
