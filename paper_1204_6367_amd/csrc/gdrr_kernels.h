// Kernels of the gfx950 Monte Carlo projection step (Step 2 of gDRR,
// Sec. 2.4 of arXiv:1204.6367) and their launch parameters.
//
// One wavefront lane carries one photon history at a time.  Lanes live for
// the whole launch (a persistent grid): a lane whose history ends takes the
// next photon index of its wavefront's chunk, and wavefronts take chunks of
// (job, photon range) from atomic dispensers, so all the angles and
// phantoms of a batch run in the same launch.  Each loop iteration has three
// phases -- refill (start new histories), flight (one Woodcock step of every
// flying lane) and collision (interaction sampling) -- and the two rare ones
// run only when enough lanes wait for them (`defer` for refills, `cdefer` for
// collisions), so that the wavefront's SIMD lanes mostly execute the same
// free-flight code.
#pragma once

#include "gdrr_device.h"
#include "gdrr_plan.h"

namespace gdrr {

enum : int { kDead = 0, kFly = 1, kColl = 2 };
enum : int { kModeForward = 0, kModeTrace = 1, kModeBackward = 2 };

constexpr int kMaxVol = 8;
constexpr int kMaxSrc = 8;

constexpr int kDispensers = 8;       // one per XCD (workgroup i runs on XCD i mod 8)
constexpr int kDispStride = 32;      // elements between them: a cache line each

struct KParams {
    DVolume vol[kMaxVol];
    DSource src[kMaxSrc];
    const DJob* jobs;
    const unsigned long long* chunk_prefix;   // [n_jobs + 1]: first chunk of each job
    unsigned long long* counter;              // n_disp chunk dispensers, kDispStride apart
    unsigned long long* tally;                // fixed-point tallies
    const float* mu_mass;                     // [n_mat][n_e][3]
    const float* response;                    // [n_e] or null
    const float* majorants;                   // [n_vols][n_e - 1], 1/cm
    unsigned long long total_chunks;
    unsigned int n_disp;                      // workgroup b uses dispenser b mod n_disp
    int n_jobs, n_vols, n_mat, n_e;
    int n_maj;                                // volumes whose single-majorant table is staged in LDS (0 or n_vols)
    int tot_rows;                             // rows per energy of the LDS attenuation table (>= n_mat)
    int mask_rows;                            // rows after the materials' kept for material sets of cubes
    float e0, inv_de, e_max, e_cut, x0, mhx0;   // mhx0 = -x0 / 2
    uint32_t k0, k1;
    uint32_t flags;
    int chunk, defer, cdefer;
    // diagnostics (trace mode)
    int8_t* t_cls;
    int32_t* t_pixel;
    float* t_e;
    int32_t* t_steps;
    int32_t* t_nc;
    int32_t* t_nr;
    // adjoint (backward mode)
    const double* adj;
    double* grad;
    // local majorants staged in LDS after the tables: per volume the offset (records) or -1
    int macro_lds[kMaxVol];
    int macro_lds_n;          // records staged in total
    int n_slots;              // started photons a wavefront keeps in LDS
};

// LDS holds what every free flight reads: the total attenuation per
// (grid point, row) and the majorants; interaction-type splits are read from
// the global table at the (rarer) real collisions.  Rows 0 .. n_mat-1 are the
// materials; with local majorants the rows after them hold, for the material
// sets of several materials that cubes have, the chord between the largest
// mu_tot of the set at the interval's two grid energies (the set's bound).
__host__ __device__ inline size_t table_floats2(int tot_rows, int n_e, int n_maj) {
    return (size_t)tot_rows * n_e + (size_t)n_maj * (n_e - 1);
}

// The row field of an all-local LDS record: 31 = no row (the bound then comes
// from the cube's material mask in its global record).
constexpr uint32_t kNoRow = 31u;

// All-local LDS grids are padded: one more word per row and one more row per
// slab, which close a row and a slab on both sides, and a slab before and after.
// The padding holds kOutside, a NaN density bound (no record has one) with
// row 0: a walk that steps out of the grid ends on it without a test of its
// own.  Words per slab:
constexpr uint32_t kOutside = 0x7FC00000u;
__host__ __device__ inline int outside_stride(int mnx, int mny) { return (mnx + 1) * (mny + 1); }

struct Tables {
    const float2* tot;    // [j][row] (tot_j, tot_j+1 - tot_j): the rows of one interval side by side
    const float2* maj;    // [v][j] (mbar, mean free path per unit of -ln u, mm)
};

// Energy-interval cache of a photon: interval index, fraction, majorant, mfp.
struct ECache {
    int j;
    float f, mbar, mfp;
};

// vol_off < 0: the volume tracks with local majorants and has no staged table.
__device__ __forceinline__ ECache energy_cache(const KParams& P, const Tables& T, int vol_off, float E) {
    const float g = (E - P.e0) * P.inv_de;
    int j = (int)floorf(g);
    j = j < 0 ? 0 : (j > P.n_e - 2 ? P.n_e - 2 : j);
    const float2 m = vol_off >= 0 ? T.maj[vol_off + j] : make_float2(0.0f, 0.0f);
    return ECache{j, g - (float)j, m.x, m.y};
}

// Density at x (tri-linear on the voxel-centre lattice, clamped to the edge
// voxels; or the containing voxel's) and the containing voxel's material, from
// the cell records (one 32-byte record; the voxel array only for the material
// of a cell whose corners differ).
// The containing voxel is corner (f >= 1/2) of the cell along each axis.
__device__ __forceinline__ float cell_density(const DVolume& V, bool interp, float px, float py, float pz,
                                              int& mat) {
    const float hx = (px - V.lox) * V.idx - 0.5f, hy = (py - V.loy) * V.idy - 0.5f, hz = (pz - V.loz) * V.idz - 0.5f;
    const float fx0 = floorf(hx), fy0 = floorf(hy), fz0 = floorf(hz);
    const int ix = min(max((int)fx0, -1), V.nx - 1);
    const int iy = min(max((int)fy0, -1), V.ny - 1);
    const int iz = min(max((int)fz0, -1), V.nz - 1);
    const float fx = fminf(fmaxf(hx - fx0, 0.0f), 1.0f);
    const float fy = fminf(fmaxf(hy - fy0, 0.0f), 1.0f);
    const float fz = fminf(fmaxf(hz - fz0, 0.0f), 1.0f);
    const CellRec* r = V.cells + ((iz + 1) * V.cxy + (iy + 1) * V.cx + (ix + 1));
    const float4 lo4 = *reinterpret_cast<const float4*>(&r->d[0]);
    const float4 hi4 = *reinterpret_cast<const float4*>(&r->d[4]);
    const int bits = (fx >= 0.5f ? 1 : 0) | (fy >= 0.5f ? 2 : 0) | (fz >= 0.5f ? 4 : 0);
    const uint32_t s0 = __float_as_uint(lo4.x);
    if (!(s0 >> 31)) {
        mat = (int)((__float_as_uint(lo4.y) >> 31) | ((__float_as_uint(lo4.z) >> 30) & 2u) |
                    ((__float_as_uint(lo4.w) >> 29) & 4u) | ((__float_as_uint(hi4.x) >> 28) & 8u));
    } else {
        const int vx = min(max(ix + (bits & 1), 0), V.nx - 1);
        const int vy = min(max(iy + ((bits >> 1) & 1), 0), V.ny - 1);
        const int vz = min(max(iz + (bits >> 2), 0), V.nz - 1);
        mat = V.material[vz * V.nxy + vy * V.nx + vx];
    }
    const float c0 = fabsf(lo4.x), c1 = fabsf(lo4.y), c2 = fabsf(lo4.z), c3 = fabsf(lo4.w);
    const float c4 = fabsf(hi4.x), c5 = hi4.y, c6 = hi4.z, c7 = hi4.w;
    if (!interp) {
        const int b2 = bits & 3;
        return bits & 4 ? (b2 == 0 ? c4 : (b2 == 1 ? c5 : (b2 == 2 ? c6 : c7)))
                        : (b2 == 0 ? c0 : (b2 == 1 ? c1 : (b2 == 2 ? c2 : c3)));
    }
    const float a00 = c0 + fx * (c1 - c0), a01 = c2 + fx * (c3 - c2);
    const float a10 = c4 + fx * (c5 - c4), a11 = c6 + fx * (c7 - c6);
    const float b0 = a00 + fy * (a01 - a00), b1 = a10 + fy * (a11 - a10);
    return b0 + fz * (b1 - b0);
}

// (read from global memory: one lookup per scored photon; j <= n_e - 2)
__device__ __forceinline__ float response_at(const KParams& P, const Tables& T, const ECache& ec, float E) {
    if (!P.response) return E;
    const float r0 = P.response[ec.j], r1 = P.response[ec.j + 1];
    return r0 + ec.f * (r1 - r0);
}

// Per-lane photon state.
struct Photon {
    float px, py, pz, dx, dy, dz, E, trem;
    uint32_t pid, step, jid;   // photon index, free flights so far, Philox job word
    int job;                   // index into the job table
    int pix0;                  // sampled aim pixel (the pixel of a primary)
    uint32_t nsc;              // Compton count | Rayleigh count << 16
    int st;
    bool passb;                // adjoint: second (visiting) pass
    ECache ec;
    uint32_t pair;             // flight pairs opened so far (Philox step of the flight block)
    bool half;                 // screened flights: the pair's second flight is still to come, on
    uint32_t rz, rw;           // these words
    float sel;                 // pending collision: ladder / rho, compared with mu_R and mu_R + mu_C
    int pm;                    // pending collision: material
    double w;                  // adjoint weight of the history
};

// Source photon (Sec. 2.1/2.4): aim pixel and energy channel by inverse CDF
// (the energy from the row of the pixel's column for a joint source), aim
// point uniform inside the pixel, straight line from S to the phantom.  It
// depends on the photon index alone, so that a wavefront can start the next
// photons of its chunk all at once.  in: the photon enters the phantom;
// otherwise it reaches its aim pixel unscattered.
struct Start {
    float tin, dx, dy, dz, E, trem;
    int pix;
    bool in;
};

__device__ __forceinline__ Start start_state(const KParams& P, const DJob& J, const DVolume& V, uint32_t pid) {
    const DSource& S = P.src[J.src];
    const Block b0 = philox(pid, J.job_id, 0u, 0u, P.k0, P.k1);
    const Block b1 = philox(pid, J.job_id, 0u, 1u, P.k0, P.k1);
    const int kf = sample_cdf(S.flu_cdf, S.flu_guide, S.npix, S.flu_k, u53(b0.z, b0.w));
    const int iv = kf / J.nu, iu = kf - iv * J.nu;
    const int row = S.spec_rows > 1 ? iu : 0;
    const int ke = sample_cdf(S.spec_cdf + (size_t)row * S.n_spec, S.spec_guide + (size_t)row * S.spec_k, S.n_spec,
                              S.spec_k, u53(b0.x, b0.y));
    const float uc = ((float)iu + u24(b1.x) - 0.5f * (float)J.nu) * J.du;
    const float vc = ((float)iv + u24(b1.y) - 0.5f * (float)J.nv) * J.dv;
    Start s;
    float dx = J.Px + uc * J.ux - J.Sx;
    float dy = J.Py + uc * J.uy - J.Sy;
    float dz = J.Pz + uc * J.uz + vc - J.Sz;
    const float inv = __builtin_amdgcn_rsqf(dx * dx + dy * dy + dz * dz);
    dx *= inv; dy *= inv; dz *= inv;
    s.dx = dx; s.dy = dy; s.dz = dz;
    s.E = fminf(fmaxf(S.spec_e[ke], P.e0), P.e_max);
    s.pix = kf;
    float tout;
    s.in = box_entry(V, J.Sx, J.Sy, J.Sz, dx, dy, dz, s.tin, tout);
    s.trem = tout - s.tin;
    return s;
}

// A lane takes a started photon of job J (one that misses the phantom is nowhere in it).
__device__ __forceinline__ void take_start(const KParams& P, const Tables& T, const DJob& J, int vol_off, Photon& ph,
                                           const Start& s) {
    ph.px = __builtin_fmaf(s.tin, s.dx, J.Sx);
    ph.py = __builtin_fmaf(s.tin, s.dy, J.Sy);
    ph.pz = __builtin_fmaf(s.tin, s.dz, J.Sz);
    ph.dx = s.dx; ph.dy = s.dy; ph.dz = s.dz;
    ph.E = s.E;
    ph.trem = s.trem;
    ph.ec = energy_cache(P, T, vol_off, s.E);
    ph.step = 0;
    ph.pair = 0;
    ph.half = false;
    ph.nsc = 0;
    ph.pix0 = s.pix;
}

__device__ __forceinline__ bool start_photon(const KParams& P, const Tables& T, const DVolume& V, int vol_off,
                                             Photon& ph) {
    const DJob& J = P.jobs[ph.job];
    const Start s = start_state(P, J, V, ph.pid);
    take_start(P, T, J, vol_off, ph, s);
    return s.in;
}

// Detector hit of a photon leaving the phantom: the primary pixel for an
// unscattered photon, else the intersection of its line with the detector
// plane (half-open pixels).  Returns the class (primary / scatter / missed).
__device__ __forceinline__ int detector_pixel(const DJob& J, const Photon& ph, int& pixel) {
    if (ph.nsc == 0) { pixel = ph.pix0; return kPrimary; }
    const float dn = ph.dx * J.nx + ph.dy * J.ny + ph.dz * J.nz;
    pixel = -1;
    if (!(dn > 0.0f)) return kMissed;
    const float t = ((J.Px - ph.px) * J.nx + (J.Py - ph.py) * J.ny + (J.Pz - ph.pz) * J.nz) * fast_rcp(dn);
    if (!(t >= 0.0f)) return kMissed;
    const float hx = ph.px + t * ph.dx - J.Px, hy = ph.py + t * ph.dy - J.Py, hz = ph.pz + t * ph.dz - J.Pz;
    const float fu = (hx * J.ux + hy * J.uy + hz * J.uz) * J.idu + 0.5f * (float)J.nu;
    const float fv = hz * J.idv + 0.5f * (float)J.nv;
    const float ku = floorf(fu), kv = floorf(fv);
    if (ku >= 0.0f && ku < (float)J.nu && kv >= 0.0f && kv < (float)J.nv) {
        pixel = (int)kv * J.nu + (int)ku;
        return kScatter;
    }
    return kMissed;
}

__device__ __forceinline__ bool counts_as_scatter(uint32_t flags, uint32_t nsc) {
    const uint32_t nc = nsc & 0xFFFFu, nr = nsc >> 16;
    if (flags & 16u) return nc == 1 && nr == 0;
    if (flags & 8u) return nc + nr == 1;
    return true;
}

__device__ __forceinline__ void tally_add(const KParams& P, const DJob& J, int cls, int pixel, float r) {
    const int npix = J.nu * J.nv;
    unsigned long long* t = P.tally + J.tally_off + (cls == kPrimary ? 0 : 2 * npix) + pixel;
    const double rd = (double)r;
    atomicAdd(t, (unsigned long long)__double2ll_rn(rd * kQ1));
    if (P.flags & 2u) atomicAdd(t + npix, (unsigned long long)__double2ll_rn(rd * rd * kQ2));
}

template <int MODE>
__device__ __forceinline__ void trace_out(const KParams& P, const Photon& ph, int cls, int pixel) {
    if (MODE != kModeTrace) return;
    const uint32_t i = ph.pid - P.jobs[ph.job].first;
    if (P.t_cls) P.t_cls[i] = (int8_t)cls;
    if (P.t_pixel) P.t_pixel[i] = pixel;
    if (P.t_e) P.t_e[i] = ph.E;
    if (P.t_steps) P.t_steps[i] = (int32_t)ph.step;
    if (P.t_nc) P.t_nc[i] = (int32_t)(ph.nsc & 0xFFFFu);
    if (P.t_nr) P.t_nr[i] = (int32_t)(ph.nsc >> 16);
}

// The end of a history: score it (forward), record it (trace) or turn it
// into the adjoint's visiting pass (backward).
template <int MODE>
__device__ __forceinline__ void finish(const KParams& P, const Tables& T, const DVolume& V, int vol_off,
                                      Photon& ph, int cls, int pixel) {
    const DJob& J = P.jobs[ph.job];
    const bool counted = cls == kPrimary || (cls == kScatter && counts_as_scatter(P.flags, ph.nsc));
    if (MODE == kModeTrace) trace_out<MODE>(P, ph, cls, pixel);
    if (MODE == kModeForward) {
        if (counted) tally_add(P, J, cls, pixel, fminf(fmaxf(response_at(P, T, ph.ec, ph.E), 0.0f), kMaxResponse));
        ph.st = kDead;
        return;
    }
    if (MODE == kModeBackward && !ph.passb && counted) {
        const double n = (double)J.n_lo + 4294967296.0 * (double)J.n_hi;
        const int npix = J.nu * J.nv;
        const double a = P.adj[J.adj_off + (cls == kPrimary ? 0 : npix) + pixel];
        const float r = fminf(fmaxf(response_at(P, T, ph.ec, ph.E), 0.0f), kMaxResponse);
        const double w = a * (double)r / n;
        if (w != 0.0) {
            ph.w = w;
            ph.passb = true;
            ph.st = start_photon(P, T, V, vol_off, ph) ? kFly : kDead;
            return;
        }
    }
    ph.st = kDead;
}

// Score-function terms of one tentative collision (adjoint, second pass):
// base w_v / rho (real) or -mu_tot w_v / (mbar - rho mu_tot) (null) times the
// history's weight, added to every stencil voxel v.  The stencil -- the eight
// lattice corners of the interpolation (clamped to the edge voxels, so a
// clamped corner repeats a voxel) and their weights, or the containing voxel --
// comes from the position alone: rho is the density the collision test has
// just computed, so no voxel is read again.
__device__ __forceinline__ void visit(const KParams& P, const DVolume& V, bool interp, const Photon& ph,
                                      bool real, float rho, float tot, float mbar) {
    const float base = real ? 1.0f / rho : -tot / (mbar - rho * tot);
    const float gx = (ph.px - V.lox) * V.idx, gy = (ph.py - V.loy) * V.idy, gz = (ph.pz - V.loz) * V.idz;
    if (!interp) {
        const int cx = min(max((int)floorf(gx), 0), V.nx - 1);
        const int cy = min(max((int)floorf(gy), 0), V.ny - 1);
        const int cz = min(max((int)floorf(gz), 0), V.nz - 1);
        if (base != 0.0f) unsafeAtomicAdd(P.grad + (cz * V.nxy + cy * V.nx + cx), ph.w * (double)base);
        return;
    }
    const float hx = gx - 0.5f, hy = gy - 0.5f, hz = gz - 0.5f;
    const float fx0 = floorf(hx), fy0 = floorf(hy), fz0 = floorf(hz);
    const float fx = hx - fx0, fy = hy - fy0, fz = hz - fz0;
    const int ix = (int)fx0, iy = (int)fy0, iz = (int)fz0;
    const int x0 = min(max(ix, 0), V.nx - 1), x1 = min(max(ix + 1, 0), V.nx - 1);
    const int y0 = min(max(iy, 0), V.ny - 1) * V.nx, y1 = min(max(iy + 1, 0), V.ny - 1) * V.nx;
    const int z0 = min(max(iz, 0), V.nz - 1) * V.nxy, z1 = min(max(iz + 1, 0), V.nz - 1) * V.nxy;
    const float gx0 = 1.0f - fx, gy0 = 1.0f - fy, gz0 = 1.0f - fz;
    const int vox[8] = {z0 + y0 + x0, z0 + y0 + x1, z0 + y1 + x0, z0 + y1 + x1,
                        z1 + y0 + x0, z1 + y0 + x1, z1 + y1 + x0, z1 + y1 + x1};
    const float wt[8] = {gx0 * gy0 * gz0, fx * gy0 * gz0, gx0 * fy * gz0, fx * fy * gz0,
                         gx0 * gy0 * fz, fx * gy0 * fz, gx0 * fy * fz, fx * fy * fz};
    const double wb = ph.w * (double)base;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (wt[k] != 0.0f) unsafeAtomicAdd(P.grad + vox[k], wb * (double)wt[k]);
}

// One Woodcock free flight with uniforms (ra, rb): flight length -ln(u)/mbar,
// then the collision ladder.  Returns true after a null collision (the photon
// flies on); escape, a real collision or the step limit return false.
template <int MODE>
__device__ __forceinline__ bool flight(const KParams& P, const Tables& T, const DVolume& V, int vo, bool interp,
                                       Photon& ph, uint32_t ra, uint32_t rb) {
    if (ph.step >= kMaxSteps) {                          // step limit: the history is lost
        if (MODE == kModeTrace) trace_out<MODE>(P, ph, kLost, -1);
        ph.st = kDead;
        return false;
    }
    ph.step += 1;
    const float s = -fast_log(u24(ra)) * ph.ec.mfp;
    if (!(s < ph.trem)) {
        int pixel;
        const int cls = detector_pixel(P.jobs[ph.job], ph, pixel);
        finish<MODE>(P, T, V, vo, ph, cls, pixel);
        return false;
    }
    ph.px += s * ph.dx;
    ph.py += s * ph.dy;
    ph.pz += s * ph.dz;
    ph.trem -= s;
    int m;
    const float rho = cell_density(V, interp, ph.px, ph.py, ph.pz, m);
    m = m < P.n_mat ? m : P.n_mat - 1;
    const float2 tt = T.tot[ph.ec.j * P.tot_rows + m];
    const float tot = tt.x + ph.ec.f * tt.y;
    // one uniform on [0, mbar): real below mu = rho tot, then the type ladder
    const float ladder = u24(rb) * ph.ec.mbar;
    const bool real = ladder < rho * tot;
    if (MODE == kModeBackward && ph.passb) visit(P, V, interp, ph, real, rho, tot, ph.ec.mbar);
    if (real) {
        ph.st = kColl;
        ph.sel = ladder * fast_rcp(rho);
        ph.pm = m;
        return false;
    }
    return true;
}

// Flights of a wavefront's lanes under the single majorant, screened (every lane
// is active, those in state kFly fly).  The majorant is the densest voxel's: in a
// body about 25 tentative collisions a history are tested, and 3 in 4 of them are
// null with a ladder value above anything their surroundings can reach.  A bound
// of rho mu_tot over the cube around the point (from one LDS word: largest density,
// with a margin over all rounding, and the table row of the cube's materials)
// settles those without the 32-byte gather, the interpolation and the material
// lookup; the others, and the escapes, leave the loop and are tested together.  The
// decisions, and so the histories, are those of flight().  The loop goes on while
// kKeepFlying lanes still fly, or no lane has anything else to do.  1e7 photons of 256x256x160 voxels:
// 4.73 -> 2.2 ms (kKeepFlying 8: 2.4, 32: 2.4).
constexpr int kKeepFlying = 16;
constexpr double kScreenScale = 1.0 + 1.0 / 65536.0;      // of a screening cube's density

template <int MODE>
__device__ __forceinline__ void flights_screened(const KParams& P, const Tables& T, const DVolume& V, int vo,
                                                 bool interp, Photon& ph, const uint32_t* lds_rec) {
    const float2* const tot = T.tot + ph.ec.j * P.tot_rows;
    enum : int { kOn = 0, kTest = 1, kOut = 2 };         // null by its bound; to be tested; box or step limit
    const auto one = [&](uint32_t ra, uint32_t rb) -> int {
        const float s = -fast_log(u24(ra)) * ph.ec.mfp;
        if (!(s < ph.trem) || ph.step >= kMaxSteps) return kOut;
        ph.step += 1;
        ph.px += s * ph.dx;
        ph.py += s * ph.dy;
        ph.pz += s * ph.dz;
        ph.trem -= s;
        ph.sel = u24(rb) * ph.ec.mbar;                   // the ladder value
        const float bx = __builtin_amdgcn_fmed3f(floorf((ph.px - V.lox) * V.imx), 0.0f, V.mlx);
        const float by = __builtin_amdgcn_fmed3f(floorf((ph.py - V.loy) * V.imy), 0.0f, V.mly);
        const float bz = __builtin_amdgcn_fmed3f(floorf((ph.pz - V.loz) * V.imz), 0.0f, V.mlz);
        // (at most kScreenCubes cubes: exact in float32)
        const uint32_t rec = lds_rec[(int)__builtin_fmaf(__builtin_fmaf(bz, V.mly + 1.0f, by), V.mlx + 1.0f, bx)];
        const float2 tt = tot[rec & 31u];
        return ph.sel >= __uint_as_float(rec & ~31u) * (tt.x + ph.ec.f * tt.y) ? kOn : kTest;
    };
    bool fly = ph.st == kFly;
    int end = kOn;
    do {
        if (fly) {
            bool second = ph.half;
            if (!second) {
                ph.pair += 1u;
                const Block b = philox(ph.pid, ph.jid, ph.pair, 0u, P.k0, P.k1);
                ph.rz = b.z;
                ph.rw = b.w;
                end = one(b.x, b.y);
                ph.half = true;
                second = end == kOn;
            }
            if (second) {
                end = one(ph.rz, ph.rw);
                ph.half = false;
            }
            fly = end == kOn;
        }
    } while (__popcll(__ballot(fly)) >= (__ballot(end != kOn) ? kKeepFlying : 1));
    const bool tested = end == kTest;
    if (end == kOut) {
        if (ph.step >= kMaxSteps) {                      // step limit: the history is lost
            if (MODE == kModeTrace) trace_out<MODE>(P, ph, kLost, -1);
            ph.st = kDead;
        } else {
            ph.step += 1;
            int pixel;
            const int cls = detector_pixel(P.jobs[ph.job], ph, pixel);
            finish<MODE>(P, T, V, vo, ph, cls, pixel);
        }
    }
    if (tested) {
        int m;
        const float rho = cell_density(V, interp, ph.px, ph.py, ph.pz, m);
        m = m < P.n_mat ? m : P.n_mat - 1;
        const float2 tt = tot[m];
        const float tot_m = tt.x + ph.ec.f * tt.y;
        if (ph.sel < rho * tot_m) {
            ph.st = kColl;
            ph.sel = ph.sel * fast_rcp(rho);
            ph.pm = m;
            ph.half = false;                             // a real collision ends the pair
        }
    }
}

// Material factor of a cube's bound from its material mask, tot pointing at the
// row of the photon's energy interval j: the chord between the largest mu_tot
// of the cube's materials at E_j and at E_j+1 (the next interval's rows; j <=
// n_e - 2), the same float operations as a row of the set's (stage_records_rows),
// so that a cube's bound does not depend on where it is read from.
__device__ __forceinline__ float set_bound(const float2* tot, int rows, uint32_t mask, float f) {
    float t0 = 0.0f, t1 = 0.0f;
    for (; mask; mask &= mask - 1u) {
        const int m = __builtin_ctz(mask);
        const float a = tot[m].x, b = tot[rows + m].x;
        t0 = a > t0 ? a : t0;
        t1 = b > t1 ? b : t1;
    }
    return t0 + f * (t1 - t0);
}

// One free flight under local majorants (uniforms ra, rb): an optical depth
// tau = -ln(u) is spent cube by cube along the line, each cube at its own
// bound mbar_B = (1 + margin) rho_max(B) max_{m in B} mu_tot(m, E); where tau
// runs out the collision ladder runs against that cube's bound; leaving the
// last cube is an escape.  Returns true after a null collision.  REC: where
// the cube records are read: 0 = global memory; 1 = their LDS copy lds_rec
// (a separate instantiation, so that the load is an LDS read, not a generic
// one).  All-local launches walk by walk_flight instead.
template <int MODE, int REC>
__device__ __forceinline__ bool flight_local(const KParams& P, const Tables& T, const DVolume& V, int vo,
                                             bool interp, Photon& ph, uint32_t ra, uint32_t rb,
                                             const void* lds_rec) {
    if (ph.step >= kMaxSteps) {
        if (MODE == kModeTrace) trace_out<MODE>(P, ph, kLost, -1);
        ph.st = kDead;
        return false;
    }
    ph.step += 1;
    float tau = -fast_log(u24(ra));
    int bx = min(max((int)floorf((ph.px - V.lox) * V.imx), 0), V.mnx - 1);
    int by = min(max((int)floorf((ph.py - V.loy) * V.imy), 0), V.mny - 1);
    int bz = min(max((int)floorf((ph.pz - V.loz) * V.imz), 0), V.mnz - 1);
    // Distances along the line (from the flight's start) to the next cube face
    // on each axis, advanced by one cube edge per crossing (Amanatides-Woo).
    const float rx = ph.dx != 0.0f ? fast_rcp(ph.dx) : 0.0f;
    const float ry = ph.dy != 0.0f ? fast_rcp(ph.dy) : 0.0f;
    const float rz = ph.dz != 0.0f ? fast_rcp(ph.dz) : 0.0f;
    const int sx = ph.dx > 0.0f ? 1 : (ph.dx < 0.0f ? -1 : 0);
    const int sy = ph.dy > 0.0f ? 1 : (ph.dy < 0.0f ? -1 : 0);
    const int sz = ph.dz > 0.0f ? 1 : (ph.dz < 0.0f ? -1 : 0);
    // where the line leaves the box through a face on the positive side of an axis (the last
    // cube there may reach past the face); leaving through a negative side is the cube index
    // leaving the grid
    const float tex = fminf(sx > 0 ? (V.hix - ph.px) * rx : INFINITY,
                            fminf(sy > 0 ? (V.hiy - ph.py) * ry : INFINITY, sz > 0 ? (V.hiz - ph.pz) * rz : INFINITY));
    float tmx = sx > 0 ? (V.lox + (float)(bx + 1) * V.mex - ph.px) * rx
              : (sx < 0 ? (V.lox + (float)bx * V.mex - ph.px) * rx : INFINITY);
    float tmy = sy > 0 ? (V.loy + (float)(by + 1) * V.mey - ph.py) * ry
              : (sy < 0 ? (V.loy + (float)by * V.mey - ph.py) * ry : INFINITY);
    float tmz = sz > 0 ? (V.loz + (float)(bz + 1) * V.mez - ph.pz) * rz
              : (sz < 0 ? (V.loz + (float)bz * V.mez - ph.pz) * rz : INFINITY);
    const float dtx = V.mex * fabsf(rx), dty = V.mey * fabsf(ry), dtz = V.mez * fabsf(rz);
    const float2* tot = T.tot + ph.ec.j * P.tot_rows;
    // the cube index moves by one of these per crossing
    const int cix = sx, ciy = sy * V.mnx, ciz = sz * V.mnx * V.mny;
    int ci = (bz * V.mny + by) * V.mnx + bx;
    float mb = 0.0f, t = 0.0f;
    bool hit = false;
    // (selects instead of fminf/fmaxf below: no NaN can occur, and these need
    // no canonicalisation of their operands)
    for (;;) {
        const uint2 rec = REC == 1 ? reinterpret_cast<const uint2*>(lds_rec)[ci] : V.macro[ci];
        const float tmax = set_bound(tot, P.tot_rows, rec.y, ph.ec.f);
        mb = __uint_as_float(rec.x) * tmax;
        const float tnext = fminf(tmx, fminf(tmy, tmz));
        const float tn = tnext < tex ? tnext : tex;                    // the cube's exit, within the box
        const float span = tn - t;
        const float need = 0.1f * mb * (span > 0.0f ? span : 0.0f);   // mbar in 1/cm, lengths in mm
        if (tau < need) {                                                // (need = 0 when mb = 0: tau > 0)
            t += tau * fast_rcp(0.1f * mb);
            hit = true;
            break;
        }
        tau -= need;
        t = tn > t ? tn : t;
        if (!(tn < tex)) break;                                        // left the box
        // the axis of the nearest face (ties to x, then y)
        const bool ax = tmx == tnext, ay = !ax && tmy == tnext, az = !ax && !ay;
        ci += ax ? cix : (ay ? ciy : ciz);
        tmx = ax ? tmx + dtx : tmx;
        tmy = ay ? tmy + dty : tmy;
        tmz = az ? tmz + dtz : tmz;
        bx += ax ? sx : 0;
        by += ay ? sy : 0;
        bz += az ? sz : 0;
        if ((unsigned)bx >= (unsigned)V.mnx || (unsigned)by >= (unsigned)V.mny || (unsigned)bz >= (unsigned)V.mnz)
            break;
    }
    ph.px += t * ph.dx;
    ph.py += t * ph.dy;
    ph.pz += t * ph.dz;
    if (!hit) {
        int pixel;
        const int cls = detector_pixel(P.jobs[ph.job], ph, pixel);
        finish<MODE>(P, T, V, vo, ph, cls, pixel);
        return false;
    }
    int m;
    const float rho = cell_density(V, interp, ph.px, ph.py, ph.pz, m);
    m = m < P.n_mat ? m : P.n_mat - 1;
    const float2 tt = T.tot[ph.ec.j * P.tot_rows + m];
    const float tot_m = tt.x + ph.ec.f * tt.y;
    const float ladder = u24(rb) * mb;
    const bool real = ladder < rho * tot_m;
    if (MODE == kModeBackward && ph.passb) visit(P, V, interp, ph, real, rho, tot_m, mb);
    if (real) {
        ph.st = kColl;
        ph.sel = ladder * fast_rcp(rho);
        ph.pm = m;
        return false;
    }
    return true;
}

// A walk through the cubes of an all-local volume: distances along the line
// from its start to the next cube face on each axis and to the box, advanced by
// one cube edge per crossing (Amanatides-Woo); the LDS address of the cube's word
// in the padded grid and its step per axis, in bytes.  The set-up has no branch: cube
// coordinates are exact in float32 (clamped by one med3), an axis the line does
// not move along gets infinite distances.
struct Walk {
    float tmx, tmy, tmz, tex, dtx, dty, dtz;
    uint32_t ci, cix, ciy, ciz;
};

// LDS addresses in bytes, as the LDS instructions take them.
using LdsWord = __attribute__((address_space(3))) const uint32_t;
__device__ __forceinline__ uint32_t lds_address(const uint32_t* p) { return (uint32_t)(size_t)(LdsWord*)p; }
__device__ __forceinline__ LdsWord* lds_word(uint32_t address) { return (LdsWord*)(size_t)address; }

// Minimum and maximum of numbers that are no NaN (fminf and fmaxf first quiet
// signalling ones, an instruction per operand).
__device__ __forceinline__ float min_nn(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float max_nn(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ __forceinline__ Walk walk_setup(const DVolume& V, const Photon& ph, const uint32_t* lds_rec) {
    const float bx = __builtin_amdgcn_fmed3f(floorf((ph.px - V.lox) * V.imx), 0.0f, V.mlx);
    const float by = __builtin_amdgcn_fmed3f(floorf((ph.py - V.loy) * V.imy), 0.0f, V.mly);
    const float bz = __builtin_amdgcn_fmed3f(floorf((ph.pz - V.loz) * V.imz), 0.0f, V.mlz);
    const bool ux = ph.dx > 0.0f, uy = ph.dy > 0.0f, uz = ph.dz > 0.0f;
    const float rx = fast_rcp(ph.dx), ry = fast_rcp(ph.dy), rz = fast_rcp(ph.dz);
    Walk w;
    // where the line leaves the box through a face on the positive side of an axis (the last
    // cube there may reach past the face); leaving through a negative side is leaving the grid
    w.tex = fminf(ux ? (V.hix - ph.px) * rx : INFINITY,
                  fminf(uy ? (V.hiy - ph.py) * ry : INFINITY, uz ? (V.hiz - ph.pz) * rz : INFINITY));
    w.tmx = (V.lox + (bx + (ux ? 1.0f : 0.0f)) * V.mex - ph.px) * rx;
    w.tmy = (V.loy + (by + (uy ? 1.0f : 0.0f)) * V.mey - ph.py) * ry;
    w.tmz = (V.loz + (bz + (uz ? 1.0f : 0.0f)) * V.mez - ph.pz) * rz;
    w.tmx = ph.dx != 0.0f ? w.tmx : INFINITY;
    w.tmy = ph.dy != 0.0f ? w.tmy : INFINITY;
    w.tmz = ph.dz != 0.0f ? w.tmz : INFINITY;
    w.dtx = V.mex * fabsf(rx);
    w.dty = V.mey * fabsf(ry);
    w.dtz = V.mez * fabsf(rz);
    w.ci = lds_address(lds_rec) + 4u * (uint32_t)((int)bx + (int)by * V.msy + (int)bz * V.msz);
    w.cix = ux ? 4 : -4;
    w.ciy = 4 * (uy ? V.msy : -V.msy);
    w.ciz = 4 * (uz ? V.msz : -V.msz);
    return w;
}

// One free flight along a walk: the optical depth tau is spent cube by cube,
// each at its own bound mb.  True where tau runs out, false where the line
// leaves the box or the grid; t: the distance to there from the walk's origin.
// Cube records are the LDS words (density bound and table row; NO_ROWS: some
// cube of the workgroup has no row and takes its material mask from the global
// record).  A wavefront walks until its slowest lane is done (about 6 visits a
// flight for 2 on average), so the visit is kept short: one exit of the loop,
// the collision point computed after it, the end of the grid found as a bound
// (kOutside: a NaN is not >=).  A visit went
// from 36 to 27 vector and from 15 to 5 scalar instructions: 1e8 photons through
// 256x256x160 voxels 14.4 -> 13.05 ms, three phantoms (7.6e7) 11.4 -> 10.3 ms.
template <bool NO_ROWS>
__device__ __forceinline__ bool walk_flight(const KParams& P, const DVolume& V, const float2* tot, float f,
                                            const uint32_t* lds_rec, Walk& w, float tau, float& t, float& mb) {
    // (values, not members: a select between members becomes an indexed load from scratch memory)
    const uint32_t cix = w.cix, ciy = w.ciy, ciz = w.ciz;
    float tmx = w.tmx, tmy = w.tmy, tmz = w.tmz;
    const float tex = w.tex;
    uint32_t ci = w.ci, rec;
    float at = 0.0f, tn, tnext, m, need;
    const auto visit_cube = [&]() {
        rec = *lds_word(ci);
        const uint32_t row = rec & 31u;
        float tmax;
        if (NO_ROWS && row == kNoRow) {
            // (quotients of whole numbers below 2^15 from their float reciprocals: the halves added are
            // 2^-16 of the dividend from a whole quotient at least, the roundings 2^-22; with integer
            // divisions 8e6 photons of 256x256x160 voxels of 9 materials took 2.41 ms, 2.16 now)
            const int c = (int)((ci - lds_address(lds_rec)) >> 2);
            const int z = (int)(((float)c + 0.5f) * fast_rcp((float)V.msz)), r = c - z * V.msz;
            const int y = (int)(((float)r + 0.5f) * fast_rcp((float)V.msy)), x = r - y * V.msy;
            tmax = set_bound(tot, P.tot_rows, V.macro[(z * V.mny + y) * V.mnx + x].y, f);
        } else {
            const float2 tt = tot[row];
            tmax = tt.x + f * tt.y;
        }
        m = __uint_as_float(rec & ~31u) * tmax;
        tnext = fminf(tmx, fminf(tmy, tmz));
        tn = max_nn(min_nn(tnext, tex), at);                           // the cube's exit, within the box
        need = 0.1f * m * (tn - at);                                  // mbar in 1/cm, lengths in mm
        return tau >= need && tnext < tex;                            // (need = 0 when m = 0)
    };
    // (the first visit ahead of the loop: its body then ends on the one exit, without copies)
    if (visit_cube()) do {
        tau -= need;
        at = tn;
        // on through the nearest face (ties to x, then y)
        const bool ex = tmx == tnext, ey = tmy == tnext;
        ci += ex ? cix : (ey ? ciy : ciz);
        tmz = (ex || ey) ? tmz : tmz + w.dtz;
        tmy = (ex || !ey) ? tmy : tmy + w.dty;
        tmx = ex ? tmx + w.dtx : tmx;
    } while (visit_cube());
    w.tmx = tmx;
    w.tmy = tmy;
    w.tmz = tmz;
    w.ci = ci;
    mb = m;
    const bool go = tau >= need, out = go || rec == kOutside;
    t = go ? tn : (out ? at : at + tau * fast_rcp(0.1f * m));
    return !out;
}

// Both free flights of a pair (words x, y for the first, z, w for the second)
// in the all-local instantiations.  With interpolated density the forward sets
// the walk up once: after a null collision the second flight goes on along the
// same line from the same cube, whose face distances stay valid (re-based to
// the null collision).  The adjoint sets a walk up for each flight: the walk's
// state across the collision test and its gradient visit would spill its
// registers.  So does the nearest-voxel lookup, whose flights are those of
// flight_local to the last bit.
template <int MODE, bool INTERP>
__device__ __forceinline__ void flight_pair_all_local(const KParams& P, const Tables& T, const DVolume& V, int vo,
                                                      Photon& ph, const Block& b, const uint32_t* lds_rec,
                                                      bool no_rows) {
    constexpr bool kOneWalk = INTERP && MODE != kModeBackward;
    Walk w;
    if constexpr (kOneWalk) w = walk_setup(V, ph, lds_rec);
    const float2* tot = T.tot + ph.ec.j * P.tot_rows;
#pragma nounroll
    for (int f = 0; f < 2; ++f) {
        if (ph.step >= kMaxSteps) {
            if (MODE == kModeTrace) trace_out<MODE>(P, ph, kLost, -1);
            ph.st = kDead;
            return;
        }
        ph.step += 1;
        if constexpr (!kOneWalk) w = walk_setup(V, ph, lds_rec);
        const float tau = -fast_log(u24(f == 0 ? b.x : b.z));
        float t, mb;
        const bool hit = no_rows ? walk_flight<true>(P, V, tot, ph.ec.f, lds_rec, w, tau, t, mb)
                                 : walk_flight<false>(P, V, tot, ph.ec.f, lds_rec, w, tau, t, mb);
        ph.px += t * ph.dx;
        ph.py += t * ph.dy;
        ph.pz += t * ph.dz;
        if (!hit) {
            int pixel;
            const int cls = detector_pixel(P.jobs[ph.job], ph, pixel);
            finish<MODE>(P, T, V, vo, ph, cls, pixel);
            return;
        }
        int m;
        const float rho = cell_density(V, INTERP, ph.px, ph.py, ph.pz, m);
        m = m < P.n_mat ? m : P.n_mat - 1;
        const float2 tt = tot[m];
        const float tot_m = tt.x + ph.ec.f * tt.y;
        const float ladder = u24(f == 0 ? b.y : b.w) * mb;
        const bool real = ladder < rho * tot_m;
        if (MODE == kModeBackward && ph.passb) visit(P, V, INTERP, ph, real, rho, tot_m, mb);
        if (real) {
            ph.st = kColl;
            ph.sel = ladder * fast_rcp(rho);
            ph.pm = m;
            return;
        }
        // a null collision: the second flight starts here, the distances re-based to it
        if constexpr (kOneWalk) {
            w.tmx -= t;
            w.tmy -= t;
            w.tmz -= t;
            w.tex -= t;
        }
    }
}

// Real collisions of a wavefront's lanes (Sec. 2.4; every lane is active, those
// in state kColl have one): the ladder value picks Rayleigh, Compton or
// photoelectric absorption; scattering samples the angle, updates energy and
// direction and the distance to the phantom's boundary.
template <int MODE, bool ALL_LOCAL>
__device__ __forceinline__ void collide(const KParams& P, const Tables& T, const DVolume& V, int vo, const FormFactor& F,
                                        Photon& ph) {
    bool scatter = false, is_rayleigh = false;
    if (ph.st == kColl) {
        const int m = ph.pm;
        const float* a = P.mu_mass + ((size_t)m * P.n_e + ph.ec.j) * 3;   // j <= n_e - 2
        const float R = a[0] + ph.ec.f * (a[3] - a[0]);
        const float C = a[1] + ph.ec.f * (a[4] - a[1]);
        const float sel = ph.sel;
        scatter = sel < R + C;
        is_rayleigh = sel < R;
        if (!scatter) {
            if (MODE == kModeTrace) trace_out<MODE>(P, ph, kAbsorbed, -1);
            ph.st = kDead;
        }
    }
    float ct, az;
    scatter_angles(scatter, is_rayleigh, ph.pid, ph.jid, ph.step, P.k0, P.k1, F, ph.E, ct, az);
    if (!scatter) return;
    if (is_rayleigh) {
        ph.nsc += 1u << 16;
    } else {
        ph.nsc += 1u;
        ph.ec = energy_cache(P, T, vo, ph.E);
    }
    rotate(ph.dx, ph.dy, ph.dz, ct, az);
    if (ph.E < P.e_cut) {
        if (MODE == kModeTrace) trace_out<MODE>(P, ph, kCut, -1);
        ph.st = kDead;
        return;
    }
    if (!ALL_LOCAL && !V.macro) ph.trem = box_exit(V, ph.px, ph.py, ph.pz, ph.dx, ph.dy, ph.dz);   // local majorants walk cubes instead
    ph.st = kFly;
}

// Copies the per-launch tables into LDS (all threads of the workgroup).
// mu_tot of material m at grid point j (float32, summed as everywhere)
__device__ __forceinline__ float tot_at(const KParams& P, int m, int j) {
    const float* a = P.mu_mass + ((size_t)m * P.n_e + j) * 3;
    return a[0] + a[1] + a[2];
}

__device__ __forceinline__ Tables stage_tables(const KParams& P, float2* lds) {
    float2* s_tot = lds;
    float2* s_maj = s_tot + P.tot_rows * P.n_e;
    for (int i = threadIdx.x; i < P.n_mat * P.n_e; i += blockDim.x) {
        const int j = i / P.n_mat, m = i - j * P.n_mat;
        const float t0 = tot_at(P, m, j), t1 = tot_at(P, m, j + 1 < P.n_e ? j + 1 : j);
        s_tot[j * P.tot_rows + m] = make_float2(t0, t1 - t0);
    }
    for (int i = threadIdx.x; i < P.n_maj * (P.n_e - 1); i += blockDim.x) {
        const float mb = P.majorants[i];
        s_maj[i] = make_float2(mb, mb > 0.0f ? 1.0f / (0.1f * mb) : INFINITY);
    }
    return Tables{s_tot, s_maj};
}

// Rank of bit b among the set bits of the 256-bit set bm.
__device__ __forceinline__ int set_rank(const uint32_t* bm, uint32_t b) {
    int r = __popc(bm[b >> 5] & ((1u << (b & 31u)) - 1u));
    for (uint32_t w = 0; w < (b >> 5); ++w) r += __popc(bm[w]);
    return r;
}

// All-local and screened launches: one LDS word per cube, its density bound with the row of
// the LDS table that holds its material factor: the material's own for a cube
// of one material; for several, a row of their set, if the set is among the
// first mask_rows distinct sets (by mask value) of the staged volumes (n_mat
// <= 8, masks < 256); kNoRow otherwise.  Returns whether some cube has no row.
// SCREEN: the screening cubes of single-majorant volumes, unpadded; the rows of sets
// are raised by 2^-20 of the larger node value, over the rounding of any
// material's own interpolation between the nodes.  Where sets outnumber the rows (and with more
// than 8 materials, whose sets are not told apart) the last row is that of all materials,
// for every set without its own: with an infinite bound, which tests all points of such cubes,
// 6e6 photons of 256x256x160 voxels of 9 materials took 3.80 ms, unscreened 3.03, now 1.68.  Without any
// row the bound is infinite.
// bm: 8 + 32 + 1 words of LDS scratch, free again on return (which synchronises).
template <bool SCREEN>
__device__ __forceinline__ bool stage_records_rows(const KParams& P, float2* s_tot, uint32_t* rec_lds,
                                                   uint32_t* bm) {
    if (threadIdx.x < 8) bm[threadIdx.x] = 0u;
    if (threadIdx.x == 8) bm[40] = 0u;
    __syncthreads();
    bool all_row = false;                                      // the last row is that of all materials
    if (P.mask_rows > 0) {
        for (int v = 0; v < P.n_vols; ++v) {
            const uint2* const recs = SCREEN ? P.vol[v].screen : P.vol[v].macro;
            if (P.macro_lds[v] < 0 || !recs) continue;
            const int n = P.vol[v].mnx * P.vol[v].mny * P.vol[v].mnz;
            for (int i = threadIdx.x; i < n; i += blockDim.x) {
                const uint32_t mask = recs[i].y;
                if (mask & (mask - 1u)) atomicOr(&bm[(mask >> 5) & 7u], 1u << (mask & 31u));
            }
        }
        __syncthreads();
        for (int t = threadIdx.x; t < 256; t += blockDim.x)
            if ((bm[t >> 5] >> (t & 31)) & 1u) {
                const int r = set_rank(bm, (uint32_t)t);
                if (r < P.mask_rows) bm[8 + r] = (uint32_t)t;
            }
        __syncthreads();
        int n_sets = 0;
        for (int w = 0; w < 8; ++w) n_sets += __popc(bm[w]);
        all_row = SCREEN && (P.n_mat > 8 || n_sets > P.mask_rows);
        for (int i = threadIdx.x; i < P.mask_rows * P.n_e; i += blockDim.x) {
            const int j = i / P.mask_rows, k = i - j * P.mask_rows;
            const int j1 = j + 1 < P.n_e ? j + 1 : j;
            float t0 = 0.0f, t1 = 0.0f;
            const bool all = all_row && k == P.mask_rows - 1;
            if (all || k < n_sets)
                for (uint32_t mask = all ? (1u << P.n_mat) - 1u : bm[8 + k]; mask; mask &= mask - 1u) {
                    const int m = __builtin_ctz(mask);
                    const float a = tot_at(P, m, j), b = tot_at(P, m, j1);
                    t0 = a > t0 ? a : t0;
                    t1 = b > t1 ? b : t1;
                }
            if (SCREEN) {
                const float up = 0x1p-20f * (t0 > t1 ? t0 : t1);
                t0 += up;
                t1 += up;
            }
            s_tot[j * P.tot_rows + P.n_mat + k] = make_float2(t0, t1 - t0);
        }
    }
    for (int v = 0; v < P.n_vols; ++v) {
        const DVolume& V = P.vol[v];
        const uint2* const recs = SCREEN ? V.screen : V.macro;
        if (P.macro_lds[v] < 0 || !recs) continue;
        const int n = SCREEN ? V.mnx * V.mny * V.mnz : V.msz * (V.mnz + 2);
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            uint32_t* word = rec_lds + P.macro_lds[v] + i;
            int c = i;
            if (!SCREEN) {
                const int z = i / V.msz - 1, y = (i - (z + 1) * V.msz) / V.msy, x = i - (z + 1) * V.msz - y * V.msy;
                word -= V.msz;
                if (z < 0 || z >= V.mnz || y >= V.mny || x >= V.mnx) {
                    *word = kOutside;
                    continue;
                }
                c = (z * V.mny + y) * V.mnx + x;
            }
            const uint2 rec = recs[c];
            uint32_t row = kNoRow;
            if (!(rec.y & (rec.y - 1u))) {
                const uint32_t m = rec.y ? (uint32_t)__builtin_ctz(rec.y) : kNoRow;
                row = m < kNoRow ? m : kNoRow;
            } else if (P.mask_rows > 0) {
                const int r = all_row && P.n_mat > 8 ? P.mask_rows : set_rank(bm, rec.y & 255u);
                row = r < P.mask_rows - (int)all_row ? (uint32_t)(P.n_mat + r)
                    : all_row ? (uint32_t)(P.n_mat + P.mask_rows - 1) : kNoRow;
            }
            *word = SCREEN && row == kNoRow ? 0x7F800000u : (rec.x & ~31u) | row;
            if (row == kNoRow) bm[40] = 1u;
        }
    }
    __syncthreads();
    const bool no_rows = __builtin_amdgcn_readfirstlane((int)bm[40]) != 0;
    __syncthreads();
    return no_rows;
}

// LOCAL: 0 = every volume has one majorant per energy interval; 1 = some
// volume tracks with local majorants, cube records read from global memory;
// 2 = the same with every such volume's records staged in LDS; 3 = every
// traced volume tracks with local majorants, records in LDS, and density is
// interpolated (no single-majorant flight in the code at all); 4 = the same
// with the nearest voxel's density; 5 = every traced volume tracks with a single
// majorant, screened by cube bounds in LDS.  Separate instantiations, so that each
// loop keeps its register budget.
template <int MODE, int LOCAL>
__device__ __forceinline__ void mc_body(const KParams& P) {
    constexpr bool kAllLocal = LOCAL == 3 || LOCAL == 4, kTrem = !kAllLocal;
    extern __shared__ float2 lds[];
    const Tables T = stage_tables(P, lds);
    // local majorants small enough to stage: every volume's cube records after the tables
    float2* const lds_rec = lds + table_floats2(P.tot_rows, P.n_e, P.n_maj);
    // the slots of started photons (offset in bytes from the LDS base of the first wavefront's)
    const uint32_t slots_off = (uint32_t)slots_offset_bytes(
        table_floats2(P.tot_rows, P.n_e, P.n_maj) * 8 + (size_t)P.macro_lds_n * lds_record_bytes(LOCAL));
    // this wavefront's slots (wavefront-uniform): directions and pixels, entries and energies, distances
    const uint32_t n_slots = (uint32_t)P.n_slots;
    const uint32_t wave_off =
        __builtin_amdgcn_readfirstlane((int)(slots_off + (threadIdx.x >> 6) * n_slots * slot_bytes(LOCAL)));
    float4* const slot_d = reinterpret_cast<float4*>(reinterpret_cast<char*>(lds) + wave_off);
    float2* const slot_e = reinterpret_cast<float2*>(slot_d + n_slots);
    float* const slot_t = reinterpret_cast<float*>(slot_e + n_slots);
    bool no_rows = false;
    if (LOCAL >= 3) {
        // (the slots serve as scratch until the transport starts)
        no_rows = stage_records_rows<LOCAL == 5>(P, lds, reinterpret_cast<uint32_t*>(lds_rec),
                                                 reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(lds) + slots_off));
    } else if (LOCAL == 2) {
        uint2* r = reinterpret_cast<uint2*>(lds_rec);
        for (int v = 0; v < P.n_vols; ++v) {
            if (P.macro_lds[v] < 0 || !P.vol[v].macro) continue;
            const int n = P.vol[v].mnx * P.vol[v].mny * P.vol[v].mnz;
            for (int i = threadIdx.x; i < n; i += blockDim.x) r[P.macro_lds[v] + i] = P.vol[v].macro[i];
        }
    }
    __syncthreads();
    const bool interp = LOCAL == 3 || (LOCAL != 4 && (P.flags & 1u) != 0);
    const int lane = __lane_id();
    const FormFactor F{P.x0, P.mhx0,
                       __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(-2.0f * fast_rcp(P.x0))))};

    Photon ph;
    ph.st = kDead;
    ph.passb = false;
    ph.w = 0.0;
    ph.job = 0;
    ph.pid = 0;
    ph.jid = 0;
    ph.nsc = 0;
    ph.E = 0.0f;
    ph.step = 0u;
    ph.sel = 0.0f;
    ph.pair = 0u;
    ph.half = false;
    ph.rz = ph.rw = 0u;
    ph.pm = 0;

    // wavefront-uniform dispenser state; the slots hold photons [w_next, d_end) of the chunk,
    // photon i in slot i mod n_slots
    int w_vol = -1, w_job = 0, w_hold = 0, w_done = 0, w_first = 1;
    uint32_t w_next = 0, w_end = 0, d_end = 0;

    for (;;) {
        const uint64_t dead = __ballot(ph.st == kDead);
        const int n_dead = __popcll(dead);
        const int n_coll = __popcll(__ballot(ph.st == kColl));
        const int n_fly = 64 - n_dead - n_coll;

        // ---- refill ----
        if (w_hold && n_dead == 64) {       // drained: switch to the held chunk's phantom
            w_vol = __builtin_amdgcn_readfirstlane(P.jobs[w_job].vol);
            w_hold = 0;
        }
        if (!w_done && !w_hold && n_dead > 0 && (n_dead >= P.defer || n_fly == 0)) {
            if (w_next >= w_end) {
                // A wavefront's first chunk follows from its own number (numbered across the
                // workgroups, so that few chunks spread over the chip), the rest come from its
                // dispenser.  An atomic on one address that all XCDs use takes about 10 ns of its
                // own; one of every wavefront of the grid at the start, and one at the end, made
                // 70 us of any launch.  Each dispenser is used by the workgroups of one XCD and
                // hands out every n_disp-th chunk (1 photon: 108 -> 39 us, 4e6 adjoint photons in chunks of 64: 1.21 -> 0.87 ms).
                const unsigned int disp = blockIdx.x % P.n_disp;
                const unsigned long long here = (gridDim.x - disp + P.n_disp - 1) / P.n_disp;    // its workgroups
                unsigned long long c = (threadIdx.x >> 6) * here + blockIdx.x / P.n_disp;
                if (!w_first) {
                    c = here * (blockDim.x >> 6);
                    if (lane == 0 && c * P.n_disp + disp < P.total_chunks)
                        c += atomicAdd(P.counter + disp * kDispStride, 1ull);
                }
                w_first = 0;
                c = c * P.n_disp + disp;
                // lane 0's value in scalar registers (every lane is active here): the branches on
                // it, and so the wavefront's volume and job, stay wavefront-uniform to the compiler,
                // which then reads the volume's fields with scalar loads
                c = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(c >> 32)) << 32) |
                    (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)c);
                if (c >= P.total_chunks) {
                    w_done = 1;
                } else {
                    int lo = 0, hi = P.n_jobs - 1;          // last job whose first chunk <= c
                    while (lo < hi) {
                        const int mid = (lo + hi + 1) >> 1;
                        if (P.chunk_prefix[mid] <= c) lo = mid; else hi = mid - 1;
                    }
                    w_job = __builtin_amdgcn_readfirstlane(lo);
                    const DJob& J = P.jobs[w_job];
                    const unsigned long long nph = (unsigned long long)J.n_lo | ((unsigned long long)J.n_hi << 32);
                    const unsigned long long first = (c - P.chunk_prefix[w_job]) * (unsigned long long)P.chunk;
                    const unsigned long long last = first + (unsigned long long)P.chunk < nph ? first + P.chunk : nph;
                    // photon indices J.first + [first, last); J.first + nph < 2^32
                    w_next = (uint32_t)__builtin_amdgcn_readfirstlane((int)(J.first + (uint32_t)first));
                    w_end = (uint32_t)__builtin_amdgcn_readfirstlane((int)(J.first + (uint32_t)last));
                    d_end = w_next;                            // none of this chunk started yet
                    const int v = __builtin_amdgcn_readfirstlane(J.vol);
                    if (v != w_vol) {
                        if (n_dead == 64) w_vol = v; else w_hold = 1;
                    }
                }
            }
            if (!w_done && !w_hold) {
                // Not enough started photons left for the waiting lanes: the free slots are filled
                // with the chunk's next photons, one a lane, from the source draw to the entry into
                // the phantom.  Started here, on (almost) full wavefronts, a refill of the few lanes
                // that wait is two LDS reads; photons that miss the phantom are scored here, once,
                // and marked (E < 0).  (Started by the waiting lanes themselves, with only the draw
                // done ahead: 13.0 against 12.5 ms for 7.6e7 photons of three phantoms.)
                if ((uint32_t)n_dead > d_end - w_next && d_end < w_end) {
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // other lanes have read the slots filled now
                    const uint32_t room = n_slots - (d_end - w_next);
                    const uint32_t nd = w_end - d_end < room ? w_end - d_end : room;
                    if ((uint32_t)lane < nd) {
                        const DJob& J = P.jobs[w_job];
                        const DVolume& V = P.vol[w_vol];
                        const uint32_t pid = d_end + (uint32_t)lane;
                        Start s = start_state(P, J, V, pid);
                        if (!s.in) {
                            if (MODE != kModeBackward) {       // (no collision: nothing for the adjoint)
                                Photon q;
                                q.pid = pid;
                                q.job = w_job;
                                take_start(P, T, J, V.lds_majorant, q, s);
                                finish<MODE>(P, T, V, V.lds_majorant, q, kPrimary, q.pix0);
                            }
                            s.E = -1.0f;
                        }
                        const uint32_t k = pid & (n_slots - 1u);
                        slot_e[k] = make_float2(s.tin, s.E);
                        slot_d[k] = make_float4(s.dx, s.dy, s.dz, __int_as_float(s.pix));
                        if (kTrem) slot_t[k] = s.trem;
                    }
                    d_end += nd;
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // the slots are read by other lanes
                }
                const uint32_t avail = d_end - w_next;
                const uint32_t rank = (uint32_t)lanes_below(dead);
                if (ph.st == kDead && rank < avail) {
                    ph.pid = w_next + rank;
                    ph.job = w_job;
                    ph.jid = P.jobs[w_job].job_id;
                    ph.passb = false;
                    const uint32_t k = ph.pid & (n_slots - 1u);
                    const float2 a = slot_e[k];
                    const float4 b = slot_d[k];
                    if (a.y >= 0.0f) {
                        const Start s{a.x, b.x, b.y, b.z, a.y, kTrem ? slot_t[k] : 0.0f, __float_as_int(b.w), true};
                        take_start(P, T, P.jobs[w_job], P.vol[w_vol].lds_majorant, ph, s);
                        ph.st = kFly;
                    }
                }
                w_next += (uint32_t)n_dead < avail ? (uint32_t)n_dead : avail;
            }
        }
        if (w_done && n_dead == 64) break;
        if (w_vol < 0) continue;
        const DVolume& V = P.vol[w_vol];
        const int vo = V.lds_majorant;

        // ---- flight: one Woodcock step (Sec. 2.4) ----
        // Free flights in pairs (Sec. 2.4): one Philox block per pair, two words per
        // flight; a null collision continues the pair, a real one ends it.
        if constexpr (LOCAL == 5) {
            flights_screened<MODE>(P, T, V, vo, interp, ph,
                                   reinterpret_cast<const uint32_t*>(lds_rec) + P.macro_lds[w_vol]);
        } else if (ph.st == kFly) {
            ph.pair += 1u;
            const Block b = philox(ph.pid, ph.jid, ph.pair, 0u, P.k0, P.k1);
            if constexpr (kAllLocal) {
                const uint32_t* lr = reinterpret_cast<const uint32_t*>(lds_rec) + P.macro_lds[w_vol];
                flight_pair_all_local<MODE, LOCAL == 3>(P, T, V, vo, ph, b, lr, no_rows);
            } else if (LOCAL == 2 && V.macro) {
                const uint2* lr = reinterpret_cast<const uint2*>(lds_rec) + P.macro_lds[w_vol];
                if (flight_local<MODE, 1>(P, T, V, vo, interp, ph, b.x, b.y, lr))
                    flight_local<MODE, 1>(P, T, V, vo, interp, ph, b.z, b.w, lr);
            } else {
                if (LOCAL == 1 && V.macro) {
                    if (flight_local<MODE, 0>(P, T, V, vo, interp, ph, b.x, b.y, nullptr))
                        flight_local<MODE, 0>(P, T, V, vo, interp, ph, b.z, b.w, nullptr);
                } else if (flight<MODE>(P, T, V, vo, interp, ph, b.x, b.y)) {
                    flight<MODE>(P, T, V, vo, interp, ph, b.z, b.w);
                }
            }
        }

        // ---- collision: interaction type and sampling ----
        const int n_coll2 = __popcll(__ballot(ph.st == kColl));
        const int n_fly2 = __popcll(__ballot(ph.st == kFly));
        if (n_coll2 > 0 && (n_coll2 >= P.cdefer || n_fly2 == 0 || w_done || w_hold)) {
            collide<MODE, kAllLocal>(P, T, V, vo, F, ph);
        }
    }
}

// The forward and trace transport: at most 80 VGPRs (6 wavefronts per SIMD);
// the all-local and the screened forward at most 64 (61, 64 and 57: 8 wavefronts per SIMD),
// which the 1024-thread workgroups, two per compute unit, then use.  No VGPR of theirs is
// spilled to memory; 90, 124 and 42 scalars are, to lanes of VGPRs (a VALU instruction to get one back).
template <int MODE, int LOCAL>
__global__ __launch_bounds__(1024)
__attribute__((amdgpu_waves_per_eu(MODE == kModeForward && LOCAL >= 3 ? 8 : 6))) void mc_kernel(KParams P) {
    mc_body<MODE, LOCAL>(P);
}

// The adjoint: at most 96 VGPRs (5 wavefronts per SIMD), where it would
// otherwise take 97 and drop to 4; the all-local instantiation takes 72 of them and
// runs 6 wavefronts per SIMD in workgroups of 512 and 768.  Wider ones, which a caller may ask for, would fit a
// compute unit once; for them (EU = 8) it is held to 64, two workgroups, with a spill of 40 bytes a lane in
// every flight: 2e7 histories of 128x128x96 voxels, 1024 lanes, waits 8 and 12, 3.45 -> 2.94 ms (512 lanes or
// 768 without spills 2.7; spilled and drawing photons ahead 3.74).
template <int LOCAL, int EU = 5>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(EU))) void mc_adjoint_kernel(
    KParams P) {
    mc_body<kModeBackward, LOCAL>(P);
}

// ---------------------------------------------------------------------------
// One pass over a volume: its cell records (the per-flight data layout), the
// input checks, and for the majorant the per-material maximum density (over the
// 3x3x3 neighbourhood with interpolation).
// ---------------------------------------------------------------------------
struct VoxelParams {
    const float* density;
    const uint8_t* material;
    int nx, ny, nz, n_mat;
    int planes;                  // cells in z per lane
    int seg_log;                 // 2^seg_log lanes (fewer than 256 if the volume has fewer columns) side by side, the
                                 // workgroup's others further up in z
    CellRec* cells;
    unsigned int* error;         // input-error bits (invalid densities or materials)
    unsigned int* rho_max;       // [256] float bits, zeroed
    unsigned int* present;       // [256], zeroed
};

// Four voxels of a plane, the corners of a cell column: densities as the
// transport uses them (invalid ones 0, without the sign of -0) and materials
// (beyond the table: the last one, here as everywhere), a byte each.
struct Corners {
    uint32_t d0, d1, d2, d3, m;
};

// CELLS: write the records.  MAX: 1, 2: the maxima, without and with
// interpolation.  With it the maximum over a voxel's neighbourhood is that over
// the cells that it is a corner of, so a cell gives its largest density to the
// materials of its corners.
// A lane goes through `planes` cells of its column in z, the upper corners of
// one being the lower ones of the next; 64 columns run along x (and on to the next
// row), so a wavefront reads rows and writes 2 KiB of consecutive records, and no
// index is divided but once; a volume of few columns (a tall one) has a workgroup's lanes above
// each other as well (the majorant of 1x1x200000 voxels 108 -> 18 us).  Bound by the records' 32 bytes a cell, written past the caches
// (692 against 800 us): 512 x 512 x 256 560 us, 4.5 TB/s with the volume's reads, was 1100
// with a division and eight pairs of loads a cell, and as much as 640 more for the maxima in
// a pass of their own.
template <bool CELLS, int MAX>
__global__ __launch_bounds__(256) void voxels_kernel(VoxelParams C) {
    __shared__ unsigned int s_max[MAX ? 256 : 1];              // bits + 1, 0: absent
    if (MAX) {
        s_max[threadIdx.x] = 0u;
        __syncthreads();
    }
    const uint32_t cx = (uint32_t)C.nx + 1u;
    const long long columns = (long long)cx * (C.ny + 1);
    const int segs = 256 >> C.seg_log, seg = (int)(threadIdx.x >> C.seg_log);
    const long long col = blockIdx.x * 256ll + (threadIdx.x & ((1u << C.seg_log) - 1u));
    const int k0 = ((int)blockIdx.y * segs + seg) * C.planes - 1, k1 = min(k0 + C.planes, C.nz);
    if (col < columns && k0 < C.nz) {
        const int i = (int)((uint32_t)col % cx) - 1, j = (int)((uint32_t)col / cx) - 1;
        const int xa = max(i, 0), xb = min(i + 1, C.nx - 1), ya = max(j, 0), yb = min(j + 1, C.ny - 1);
        const uint32_t o0 = (uint32_t)ya * C.nx + xa, o1 = (uint32_t)ya * C.nx + xb;
        const uint32_t o2 = (uint32_t)yb * C.nx + xa, o3 = (uint32_t)yb * C.nx + xb;
        const long long nxy = (long long)C.nx * C.ny;
        const uint32_t m_last = (uint32_t)(C.n_mat - 1);
        unsigned int err = 0u;
        uint32_t cur_m = ~0u, cur_d = 0u;                      // what this lane gave to s_max last
        const auto give = [&](uint32_t m, uint32_t d) {
            if (m == cur_m && d <= cur_d) return;
            cur_m = m;
            cur_d = d;
            if (*(volatile unsigned int*)&s_max[m] < d + 1u) atomicMax(&s_max[m], d + 1u);
        };
        const auto corners = [&](int z) {
            const float* den = C.density + (long long)z * nxy;
            const uint8_t* mat = C.material + (long long)z * nxy;
            const float r0 = den[o0], r1 = den[o1], r2 = den[o2], r3 = den[o3];
            const uint32_t q0 = mat[o0], q1 = mat[o1], q2 = mat[o2], q3 = mat[o3];
            if (!(density_ok(r0) && density_ok(r1) && density_ok(r2) && density_ok(r3))) err |= kErrDensity;
            if (max(max(q0, q1), max(q2, q3)) > m_last) err |= kErrMaterial;
            Corners c;
            c.d0 = __float_as_uint(clean_density(r0)) & 0x7FFFFFFFu;
            c.d1 = __float_as_uint(clean_density(r1)) & 0x7FFFFFFFu;
            c.d2 = __float_as_uint(clean_density(r2)) & 0x7FFFFFFFu;
            c.d3 = __float_as_uint(clean_density(r3)) & 0x7FFFFFFFu;
            c.m = min(q0, m_last) | min(q1, m_last) << 8 | min(q2, m_last) << 16 | min(q3, m_last) << 24;
            if (MAX == 1) {
                give(c.m & 255u, c.d0);
                give((c.m >> 8) & 255u, c.d1);
                give((c.m >> 16) & 255u, c.d2);
                give(c.m >> 24, c.d3);
            }
            return c;
        };
        // (a voxel's maximum by itself: the one upper corner of each cell is every voxel, four
        // loads in flight; all corners of every cell took 253 us for 512 x 512 x 256, these 118)
        if (!CELLS && MAX == 1)
            for (int k = k0; k < k1; k += 4) {
                float r[4];
                uint32_t q[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const long long v = (long long)min(min(k + u, k1 - 1) + 1, C.nz - 1) * nxy + o3;
                    r[u] = C.density[v];
                    q[u] = C.material[v];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (!density_ok(r[u])) err |= kErrDensity;
                    if (q[u] > m_last) err |= kErrMaterial;
                    give(min(q[u], m_last), __float_as_uint(clean_density(r[u])) & 0x7FFFFFFFu);
                }
            }
        const bool pairs = CELLS || MAX == 2;
        Corners lo{};
        if (pairs) lo = corners(max(k0, 0));
        for (int k = k0; pairs && k < k1; ++k) {
            const Corners hi = corners(min(k + 1, C.nz - 1));
            const uint32_t m0 = lo.m & 255u;
            const bool same = lo.m == hi.m && lo.m == m0 * 0x01010101u;
            if (MAX == 2) {
                const uint32_t d = max(max(max(lo.d0, lo.d1), max(lo.d2, lo.d3)), max(max(hi.d0, hi.d1), max(hi.d2, hi.d3)));
                give(m0, d);
                if (!same) {
                    for (int c = 8; c < 32; c += 8) give((lo.m >> c) & 255u, d);
                    for (int c = 0; c < 32; c += 8) give((hi.m >> c) & 255u, d);
                }
            }
            if (CELLS) {
                // the top bits: 0 and the material in the next four, or 1 where the corners' differ
                const uint32_t b = same ? m0 : 0u;
                typedef uint32_t Half __attribute__((ext_vector_type(4)));
                const Half h0 = {lo.d0 | (same ? 0u : 0x80000000u), lo.d1 | b << 31, lo.d2 | (b >> 1) << 31, lo.d3 | (b >> 2) << 31};
                const Half h1 = {hi.d0 | (b >> 3) << 31, hi.d1, hi.d2, hi.d3};
                Half* out = reinterpret_cast<Half*>(C.cells + (size_t)(k + 1) * columns + col);
                __builtin_nontemporal_store(h0, out);
                __builtin_nontemporal_store(h1, out + 1);
            }
            lo = hi;
        }
        if (err) atomicOr(C.error, err);
    }
    if (MAX) {
        __syncthreads();
        // (other workgroups give the same few materials: read before the atomic)
        if (s_max[threadIdx.x]) {
            const unsigned int d = s_max[threadIdx.x] - 1u;
            if (__hip_atomic_load(&C.rho_max[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < d)
                atomicMax(&C.rho_max[threadIdx.x], d);
            if (!__hip_atomic_load(&C.present[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicOr(&C.present[threadIdx.x], 1u);
        }
    }
}

struct MajFinParams {
    const unsigned int* rho_max;
    const unsigned int* present;
    const float* mu_mass;
    int n_mat, n_e;
    double scale;              // 1 + margin
    float* out;                // [n_e - 1]
    unsigned int* error;
};

__global__ __launch_bounds__(256) void majorant_kernel(MajFinParams F) {
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < F.n_e - 1; j += gridDim.x * blockDim.x) {
        double best = 0.0;
        for (int m = 0; m < F.n_mat; ++m) {
            if (!F.present[m]) continue;
            const float* a = F.mu_mass + ((size_t)m * F.n_e + j) * 3;
            const double t0 = (double)a[0] + (double)a[1] + (double)a[2];
            const double t1 = (double)a[3] + (double)a[4] + (double)a[5];
            const double t = (double)__uint_as_float(F.rho_max[m]) * (t0 > t1 ? t0 : t1);
            best = t > best ? t : best;
        }
        F.out[j] = __double2float_ru(best * F.scale);
    }
}

// ---------------------------------------------------------------------------
// Local majorants: per cube of mcube^3 voxels, the largest density (at least
// rho_min) and the materials over the cube grown by one voxel (the
// interpolation corners of every point in the cube, with a voxel to spare at
// its faces).
// ---------------------------------------------------------------------------
struct MacroParams {
    const float* density;
    const uint8_t* material;
    int nx, ny, nz, mcube, mnx, mny, mnz, n_mat;
    double scale;              // 1 + margin
    float rho_min;             // least density a cube's bound assumes
    uint2* out;
};

// One workgroup per cube (grid-stride over the cubes): the lanes stride over
// the voxels of the cube grown by one voxel, x fastest (coalesced; `lanes`, a
// power of two, take a row), then the largest density and the union of the
// materials are reduced over the workgroup.  Max and or are exact in any order, so
// the records are those of a plain loop over the voxels.
// Bound by the latency of the loads: four rows in flight per lane, and no division per
// voxel.  512 x 512 x 256 in cubes of 40: 118 us, was 235.
__global__ __launch_bounds__(1024) void macro_kernel(MacroParams M) {
    __shared__ float s_r[16];
    __shared__ uint32_t s_m[16];
    const long long n = (long long)M.mnx * M.mny * M.mnz;
    const int lanes_log = min(32 - __clz(M.mcube + 1), 6), row0 = threadIdx.x >> lanes_log;
    const int lane = threadIdx.x & ((1 << lanes_log) - 1), step = (int)blockDim.x >> lanes_log;
    for (long long c = blockIdx.x; c < n; c += gridDim.x) {
        const int bx = (int)(c % M.mnx), by = (int)((c / M.mnx) % M.mny), bz = (int)(c / ((long long)M.mnx * M.mny));
        const int x0 = max(bx * M.mcube - 1, 0), x1 = min((bx + 1) * M.mcube, M.nx - 1);
        const int y0 = max(by * M.mcube - 1, 0), y1 = min((by + 1) * M.mcube, M.ny - 1);
        const int z0 = max(bz * M.mcube - 1, 0), z1 = min((bz + 1) * M.mcube, M.nz - 1);
        const int nyc = y1 - y0 + 1;
        const int dy = step % nyc, dz = step / nyc;            // from a lane's row to its next
        float r = M.rho_min;
        uint32_t mask = 0u;
        for (int xs = x0; xs <= x1; xs += 1 << lanes_log) {
            const int x = min(xs + lane, x1);
            int y = y0 + row0 % nyc, z = z0 + row0 / nyc;
            while (z <= z1) {                                  // (a last voxel or row may be read twice)
                float q[4];
                int m[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const long long v = ((long long)min(z, z1) * M.ny + y) * M.nx + x;
                    q[u] = M.density[v];
                    m[u] = M.material[v];
                    y += dy;
                    z += dz;
                    if (y > y1) {
                        y -= nyc;
                        ++z;
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    r = fmaxf(r, clean_density(q[u]));
                    mask |= 1u << min(m[u], M.n_mat - 1);
                }
            }
        }
        for (int o = 32; o > 0; o >>= 1) {
            r = fmaxf(r, __shfl_xor(r, o));
            mask |= __shfl_xor(mask, o);
        }
        if ((threadIdx.x & 63) == 0) {
            s_r[threadIdx.x >> 6] = r;
            s_m[threadIdx.x >> 6] = mask;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
                r = fmaxf(r, s_r[w]);
                mask |= s_m[w];
            }
            // the density factor rounded up to 19 significant bits: the low 5 bits stay free
            const uint32_t rb = __float_as_uint(__double2float_ru((double)r * M.scale));
            M.out[c] = make_uint2((rb + 31u) & ~31u, mask);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Source preparation: normalised CDFs (running float64 sum in index order,
// divided by the total) and guide tables.  The sums are those of 1024 contiguous
// segments, each summed in index order, whose totals are scanned: those of the
// definition in a different association (float64 rounding only).
// ---------------------------------------------------------------------------
constexpr int kSegs = 1024;        // segments, and threads of a workgroup
constexpr int kSegBlock = 64;      // segments per workgroup of a long table (one wavefront sums them)
constexpr int kSegTile = 64;       // elements of each that go through LDS at a time

struct CdfTable {
    const float* w;           // [rows][n]
    int n, rows;
    double* cdf;              // [rows][n]
    uint32_t* guide;          // [rows][k]
    int k;
};

// Tables of more elements than this are shared by 16 workgroups, in three launches
// (sums, running sums, guide: 4.7 + 6.6 + 5.7 us for 256 x 192 against 90 + 6 with one, whose
// lanes read a segment each, uncoalesced); shorter ones
// take one workgroup per row and one launch.  (A long table's guide holds the
// segments' totals at first: kSegs doubles need 2 kSegs entries.)
constexpr int kLongTable = 2 * kSegs;

struct SrcPrepParams {
    CdfTable t[2];            // the spectrum's rows, the fluence
    int row_blocks;           // workgroups for the rows
    unsigned int* error;
};

__device__ __forceinline__ uint32_t guide_entry(const double* cdf, int n, int g, int k) {
    const double t = (double)g / (double)k;
    int lo = 0, hi = n - 1;                       // smallest i with cdf[i] > t
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (cdf[mid] > t) hi = mid; else lo = mid + 1;
    }
    return (uint32_t)lo;
}

// Inclusive Hillis-Steele scan of the segments' totals.
__device__ __forceinline__ void scan_totals(double* part) {
    const int t = threadIdx.x;
    for (int off = 1; off < kSegs; off <<= 1) {
        const double v = t >= off ? part[t - off] : 0.0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
}

// One row in one workgroup, its guide included.
__device__ void short_table(const CdfTable& T, int row, unsigned int* error, double* part) {
    const int t = threadIdx.x;
    const float* w = T.w + (size_t)row * T.n;
    double* cdf = T.cdf + (size_t)row * T.n;
    const int per = (T.n + kSegs - 1) / kSegs;
    const int a = min(T.n, t * per), b = min(T.n, a + per);
    double s = 0.0;
    bool bad = false;
    for (int i = a; i < b; ++i) {
        const double x = (double)w[i];
        bad = bad || !(x >= 0.0) || isinf(x);
        s += x;
    }
    part[t] = s;
    __syncthreads();
    scan_totals(part);
    const double total = part[kSegs - 1];
    double run = t > 0 ? part[t - 1] : 0.0;
    for (int i = a; i < b; ++i) {
        run += (double)w[i];
        cdf[i] = run / total;
    }
    if (bad || (t == 0 && !(total > 0.0))) atomicOr(error, kErrWeights);
    __syncthreads();
    for (int g = t; g < T.k; g += kSegs) T.guide[(size_t)row * T.k + g] = guide_entry(cdf, T.n, g, T.k);
}

// A tile of kSegBlock segments from element `at` on, rows padded to an odd length (a lane
// per segment reads down a column of banks).
typedef float SegTile[kSegBlock][kSegTile + 1];

__device__ __forceinline__ void load_segments(const CdfTable& T, int first, int per, int at, SegTile& tile) {
    for (int e = threadIdx.x; e < kSegBlock * kSegTile; e += kSegs) {
        const int q = e / kSegTile, x = e % kSegTile;
        const long long i = (long long)(first + q) * per + at + x;
        tile[q][x] = at + x < per && i < T.n ? T.w[i] : 0.0f;
    }
}

// The first launch: short tables whole, the segments' totals of long ones.
__global__ __launch_bounds__(kSegs) void cdf_kernel(SrcPrepParams S) {
    __shared__ double part[kSegs];
    __shared__ SegTile tile;
    if ((int)blockIdx.x < S.row_blocks) {
        for (int row = blockIdx.x; row < S.t[0].rows; row += S.row_blocks) {
            short_table(S.t[0], row, S.error, part);
            __syncthreads();
        }
        return;
    }
    const CdfTable& T = S.t[1];
    const int block = blockIdx.x - S.row_blocks;
    if (T.n <= kLongTable) return short_table(T, block, S.error, part);
    const int per = (T.n + kSegs - 1) / kSegs, first = block * kSegBlock;
    double s = 0.0;
    bool bad = false;
    for (int at = 0; at < per; at += kSegTile) {
        load_segments(T, first, per, at, tile);
        __syncthreads();
        if (threadIdx.x < kSegBlock) {
            const int m = (int)min((long long)min(kSegTile, per - at),
                                   max(T.n - ((long long)(first + threadIdx.x) * per + at), 0ll));
            for (int x = 0; x < m; ++x) {
                const double v = (double)tile[threadIdx.x][x];
                bad = bad || !(v >= 0.0) || isinf(v);
                s += v;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < kSegBlock) reinterpret_cast<double*>(T.guide)[first + threadIdx.x] = s;
    if (bad) atomicOr(S.error, kErrWeights);
}

// The second launch of a long table: each workgroup scans the totals and writes its segments.
struct LongCdfParams {
    CdfTable t;
    unsigned int* error;
};

__global__ __launch_bounds__(kSegs) void long_cdf_kernel(LongCdfParams L) {
    const CdfTable& T = L.t;
    __shared__ double part[kSegs];
    __shared__ SegTile tile;
    __shared__ double runs[kSegBlock][kSegTile + 1];
    const int t = threadIdx.x;
    part[t] = reinterpret_cast<const double*>(T.guide)[t];
    __syncthreads();
    scan_totals(part);
    const double total = part[kSegs - 1];
    if (blockIdx.x == 0 && t == 0 && !(total > 0.0)) atomicOr(L.error, kErrWeights);
    const int per = (T.n + kSegs - 1) / kSegs, first = blockIdx.x * kSegBlock;
    double run = t < kSegBlock && first + t > 0 ? part[first + t - 1] : 0.0;
    for (int at = 0; at < per; at += kSegTile) {
        load_segments(T, first, per, at, tile);
        __syncthreads();
        if (t < kSegBlock)
            for (int x = 0; x < kSegTile; ++x) {
                run += (double)tile[t][x];                     // (beyond the segment: zeros)
                runs[t][x] = run;
            }
        __syncthreads();
        for (int e = t; e < kSegBlock * kSegTile; e += kSegs) {
            const int q = e / kSegTile, x = e % kSegTile;
            const long long i = (long long)(first + q) * per + at + x;
            if (at + x < per && i < T.n) T.cdf[i] = runs[q][x] / total;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void guide_kernel(CdfTable T) {
    for (int g = blockIdx.x * 256 + threadIdx.x; g < T.k; g += gridDim.x * 256)
        T.guide[g] = guide_entry(T.cdf, T.n, g, T.k);
}

// ---------------------------------------------------------------------------
// Clear and finalize.
// ---------------------------------------------------------------------------
struct FillParams {
    unsigned long long* p;
    long long n;
};

__global__ __launch_bounds__(256) void fill_zero_kernel(FillParams F) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < F.n; i += (long long)gridDim.x * blockDim.x)
        F.p[i] = 0ull;
}

// What a call needs before its first kernel reads anything: ranges cleared, and
// its small tables written from the kernel's own arguments.  One launch took the place of 4 to
// 6 (about 4.5 us each, however little they clear) and of 3 to 5 copies from pageable memory:
// one projection of 1e5 histories 238 -> 221 us; a batch with larger tables makes one copy.
constexpr int kSetupFills = 6, kSetupWords = 704;          // (the arguments stay below 4 KiB)

struct SetupParams {
    FillParams f[kSetupFills];
    int fills, words;
    uint32_t* tables;
    uint32_t image[kSetupWords];
};

__global__ __launch_bounds__(256) void setup_kernel(SetupParams S) {
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < S.words; i += 256) S.tables[i] = S.image[i];
    for (int r = 0; r < S.fills; ++r) {
        const FillParams F = S.f[r];
        for (long long i = blockIdx.x * 256ll + threadIdx.x; i < F.n; i += gridDim.x * 256ll) F.p[i] = 0ull;
    }
}

struct FinParams {
    const DJob* jobs;
    int n_jobs;
    const unsigned long long* tally;
    double* out;
    const long long* out_off;   // [n_jobs] double element offsets in `out`
    uint32_t flags;             // GDRR_TALLY_SUMSQ 2, GDRR_ACCUMULATE 4, GDRR_RESUME 32
};

__global__ __launch_bounds__(256) void finalize_kernel(FinParams F) {
    const int k = blockIdx.y;
    const DJob& J = F.jobs[k];
    const int npix = J.nu * J.nv;
    // per source photon of the run: a resumed run's sums cover [0, first + n)
    const double n = (double)J.n_lo + 4294967296.0 * (double)J.n_hi + ((F.flags & 32u) ? (double)J.first : 0.0);
    const double inv = n > 0.0 ? 1.0 / n : 0.0;
    const bool sumsq = (F.flags & 2u) != 0, acc = (F.flags & 4u) != 0;
    double* out = F.out + F.out_off[k];
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < 4 * npix; i += gridDim.x * blockDim.x) {
        const int plane = i / npix;
        if ((plane & 1) && !sumsq) continue;
        const double q = (plane & 1) ? kQ2 : kQ1;
        const double v = (double)F.tally[J.tally_off + i] / q * inv;
        out[i] = acc ? out[i] + v : v;
    }
}

}  // namespace gdrr
