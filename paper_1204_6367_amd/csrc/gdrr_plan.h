// LDS of a transport launch: the sizes of what a workgroup keeps there.  Host
// and device agree on them; plain C++, no HIP.
#pragma once

#include <stddef.h>
#include <stdint.h>

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

}  // namespace gdrr
