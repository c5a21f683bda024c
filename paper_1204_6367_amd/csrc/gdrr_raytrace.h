// Primary signal by ray tracing (Sec. 2.3, Eq. 1): one lane per detector
// pixel, every energy channel of the spectrum.
//
//   P(u) = sum_k phi_k w(u) r(E_k) exp(-sum_j dl_j mu(x_j, E_k))
//
// The ray from the source to the pixel centre is cut into intervals
// [j dl, (j+1) dl) of its length from the source; the part of an interval
// inside the phantom box is one term, evaluated at that part's midpoint.
// mu(x, E) is the trilinear interpolation of the voxel attenuation
// coefficients rho_v mu_tot(m_v, E) (the corners of the lattice cell around
// x, clamped at the edges), or the containing voxel's value with the
// interpolation off.
//
// mu is linear in the per-voxel products, so the energy channels share one
// march: the lane accumulates, per material m, the line integral of the
// density carried by m's corners (L_m), and the channel sums come out as
// sum_m mu_tot(m, E_k) L_m after it.  Almost every lattice cell has a single
// material; those steps add the interpolated density into one register
// accumulator that is written to the lane's LDS slot of its material only when
// the material changes.  Mixed cells add each corner's share to its
// material's slot.
#pragma once

#include <type_traits>

#include "gdrr_device.h"

namespace gdrr {

constexpr int kRtBlock = 256;     // 16 x 16 pixels; each wavefront 4 detector columns of 16 rows
constexpr int kXcds = 8;          // workgroup i runs on XCD i mod 8

struct RtSource {
    const float* fluence;         // [nv][nu] weights w(u) (unnormalised)
    const float* coef;            // [rows][n_spec] phi_k r(E_k) / sum phi (row iu: detector column iu)
    const float* tab;             // [n_spec][n_mat] 0.1 mu_tot(m, E_k): mm of density-length -> optical depth
    const double* inv_wsum;       // 1 / sum_u w(u)
    int n_spec, rows;
};

// The lattice of voxel centres as the ray tracer reads it: per cell column
// (i, j), i in [-1, nx-1], j in [-1, ny-1], one 16-byte record per plane of
// voxel centres, z fastest: the densities of the column's four corners in
// plane z (clamped into the volume), corner c = bx + 2 by; cell k's corners are
// planes k and k+1, 32 bytes in a row (planes run from -1 to nz).  The sign
// bits (densities are >= 0; corner 0's the highest) of plane k carry the common
// material of cell k's eight corners, or kPlaneLook where they differ or it is that
// number: the materials are then the codes of planes k and k+1, 4 bits a corner in an
// array of their own.
//
// Rays are nearly horizontal and a wavefront holds 4 detector columns of 16
// rows, so its lanes read runs of z in 4 or so cell columns: about 20 cache
// lines a step, each used by several lanes at once.  With records of whole
// cells, x fastest, 8 x 8 lanes of a wavefront whose rays run along x read 64
// lines a step, and the lines kept for the next steps overflowed L1 and L2.
// 60 images of 512x512x256 voxels: 12.4 -> 6.6 ms (whole-cell records with z
// fastest: 6.85, and twice the bytes to build).
constexpr int kPlaneLook = 15;
using CodePair = __attribute__((aligned(2))) uint32_t;         // two neighbouring codes
using Plane = __attribute__((ext_vector_type(4))) float;    // (a value in registers: float4's members went to scratch)

__host__ __device__ inline size_t plane_count(int nx, int ny, int nz) {
    return (size_t)(nx + 1) * (size_t)(ny + 1) * (size_t)(nz + 2);
}

struct RtParams {
    DVolume vol[GDRR_MAX_VOLUMES];
    const Plane* planes[GDRR_MAX_VOLUMES];
    const uint16_t* codes[GDRR_MAX_VOLUMES];
    RtSource src[GDRR_MAX_SOURCES];
    float dl[GDRR_MAX_VOLUMES];   // interval length per volume, mm
    const DJob* jobs;
    // Work units (runs of consecutive tiles within one tile row of one job),
    // listed XCD by XCD:
    // XCD x owns units [xcd_start[x], xcd_start[x+1]); unit_pref is the
    // running tile count within its XCD's list.
    const int* unit_job;
    const unsigned int* unit_first;    // first tile of the unit within its job
    const unsigned int* unit_pref;
    unsigned int xcd_start[kXcds + 1];
    unsigned int xcd_tiles[kXcds];
    const long long* out_off;     // [n_jobs] element offset of each job's image in out
    double* out;
    int n_mat, interp, accumulate;
};

// Slab clip of t in [t0, t1] to lo <= s + t d <= hi.
__device__ __forceinline__ void rt_slab(float s, float d, float lo, float hi, float& t0, float& t1) {
    if (d != 0.0f) {
        const float ta = (lo - s) / d, tb = (hi - s) / d;
        t0 = fmaxf(t0, fminf(ta, tb));
        t1 = fminf(t1, fmaxf(ta, tb));
    } else if (s < lo || s > hi) {
        t1 = -1.0f;
    }
}

// The sign bits of a plane record as a number, the first corner's the highest.
__device__ __forceinline__ int plane_code(Plane d) {
    uint32_t c = __float_as_uint(d.x) >> 31;
    c = __builtin_amdgcn_alignbit(c, __float_as_uint(d.y), 31u);       // (c << 1) | sign
    c = __builtin_amdgcn_alignbit(c, __float_as_uint(d.z), 31u);
    return (int)__builtin_amdgcn_alignbit(c, __float_as_uint(d.w), 31u);
}

// a b for a, b < 2^24 (the low 32 bits; one instruction with an addition, where the
// full product takes four times as long).
__device__ __forceinline__ uint32_t mul_u24(uint32_t a, uint32_t b) { return (a & 0xFFFFFFu) * (b & 0xFFFFFFu); }

// A lane's value from lane K of its group of G (DPP: quads by quad_perm, rows of
// 16 by row_newbcast).
template <int G, int K>
__device__ __forceinline__ int group_lane(int v) {
    if constexpr (G == 1) return v;
    return __builtin_amdgcn_mov_dpp(v, G == 4 ? K * 0x55 : 0x150 + K, 0xf, 0xf, true);
}
template <int G, int K>
__device__ __forceinline__ float group_lane(float v) {
    return __int_as_float(group_lane<G, K>(__float_as_int(v)));
}

// f(integral constant k) for k = 0 .. G - 1.
template <int G, int K = 0, class F>
__device__ __forceinline__ void for_group(const F& f) {
    if constexpr (K < G) {
        f(std::integral_constant<int, K>{});
        for_group<G, K + 1>(f);
    }
}

// The lanes of a ray share its LDS slots: what one wrote before this, another
// reads after it (an order for the compiler; one wavefront's LDS accesses are
// carried out in theirs).
template <int G>
__device__ __forceinline__ void rt_share() {
    if constexpr (G > 1) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// G lanes per ray: lane l of a ray's group reads and interpolates intervals
// j + l, and the group adds them in their order (every lane the same sums, the
// ray's LDS slots written by one), so that the image does not depend on G.
// Many rays take one lane each.  Few rays leave the chip idle, a lone wavefront
// spending 0.6 us on each of a ray's 560 steps: one 256x192 image of 256x256x160 voxels
// 330 -> 138 us at G = 4; one of 64x48 pixels 380 -> 92 us at G = 16.
// A mixed cell's materials come from the corner codes: along with the corners for G > 1,
// where a wait costs more than the bytes, when such a cell is met for G = 1 (with every
// interval 8.7 against 6.5 ms for 60 images of 512x512x256 voxels).  Read from the voxel
// array, x fastest, they cost a wavefront of 16 rows as many lines as it has lanes: 64
// images of 256x192 of 256x256x160 voxels 2820 -> 2440 us, 16 of the same phantom with noise
// in 5 % of the materials 2330 -> 1255 (planes of whole cells, 8 x 8 pixels: 2074), in all
// of them 6810 -> 1234.  M16 (G = 1): 16 materials, one of them kPlaneLook.  SMALL: no index of the plane records or their
// rows' stride reaches 2^24, so a cell's number takes two 24-bit products (full ones cost
// four instructions each) and floats hold every bound; with the material in the lower
// plane's record alone, 8 of 75 instructions an interval: 64 images of 256x192 of 256x256x160
// voxels 2980 -> 2807 us, 60 of 512x512x256 (bound by the records' 4.8 TB/s) 6480 -> 6400.
template <int G, bool M16, bool SMALL>
__global__ __launch_bounds__(kRtBlock) void raytrace_kernel(RtParams P) {
    constexpr int kRays = kRtBlock / G;        // rays of the workgroup: 16 / G columns of 16 rows
    extern __shared__ float rt_lds[];          // [n_mat][kRays]: the rays' L_m
    // Workgroups are dealt to the XCDs in turn; each XCD walks its own list of
    // units in order.  The host orders the units by phantom, then tile row,
    // then job, and deals them round the XCDs, so at any time the whole chip
    // traces one band of detector rows -- one slab of the phantom -- over all
    // that phantom's projections.
    const unsigned int xcd = blockIdx.x % kXcds, in_xcd = blockIdx.x / kXcds;
    const unsigned int slot = in_xcd / G, part = in_xcd % G;
    if (slot >= P.xcd_tiles[xcd]) return;       // whole workgroup; no barrier in this kernel
    int lo = (int)P.xcd_start[xcd], hi = (int)P.xcd_start[xcd + 1] - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (P.unit_pref[mid] <= slot) lo = mid; else hi = mid - 1;
    }
    const DJob& J = P.jobs[P.unit_job[lo]];
    const unsigned int local = P.unit_first[lo] + (slot - P.unit_pref[lo]);
    const int tiles_u = (J.nu + 15) >> 4;
    const int ray = threadIdx.x / G, l = threadIdx.x % G;
    // Wavefronts of 16 rows by 4 columns (one lane per ray) suit planes with z fastest.  The
    // nearest voxel comes from the volume itself, x fastest: there a wavefront takes 8 x 8
    // pixels, whose rays run side by side in y and z (4 images of 512 x 384 of 256x256x160 voxels: 4 x 16
    // 1589 us, 8 x 8 1035 us; with a few lanes per ray their intervals run along x anyway).
    const bool square = G == 1 && !P.interp;
    const int w = ray >> 6, q = ray & 63;
    const int iu = (int)(local % tiles_u) * 16 + (square ? (w & 1) * 8 + (q & 7) : (int)part * (16 / G) + (ray >> 4));
    const int iv = (int)(local / tiles_u) * 16 + (square ? (w >> 1) * 8 + (q >> 3) : ray & 15);
    if (iu >= J.nu || iv >= J.nv) return;       // (whole groups)

    float* Lm = rt_lds + ray;
    if (l == 0)
        for (int m = 0; m < P.n_mat; ++m) Lm[m * kRays] = 0.0f;
    rt_share<G>();

    const DVolume& V = P.vol[J.vol];
    const float uc = ((float)iu + 0.5f - 0.5f * (float)J.nu) * J.du;
    const float vc = ((float)iv + 0.5f - 0.5f * (float)J.nv) * J.dv;
    float dx = J.Px + uc * J.ux - J.Sx;
    float dy = J.Py + uc * J.uy - J.Sy;
    float dz = J.Pz + vc - J.Sz;                       // v axis = +z
    const float len = sqrtf(dx * dx + dy * dy + dz * dz);
    dx /= len; dy /= len; dz /= len;
    float t0 = 0.0f, t1 = len;
    rt_slab(J.Sx, dx, V.lox, V.hix, t0, t1);
    rt_slab(J.Sy, dy, V.loy, V.hiy, t0, t1);
    rt_slab(J.Sz, dz, V.loz, V.hiz, t0, t1);

    if (t0 < t1) {
        const float dl = P.dl[J.vol];
        // the volume's fields in registers for the march
        const Plane* __restrict__ planes = P.planes[J.vol];
        const uint16_t* __restrict__ codes = P.codes[J.vol];
        const float* __restrict__ dens = V.density;
        const uint8_t* __restrict__ mats = V.material;
        const int nx = V.nx, ny = V.ny, nz = V.nz, nxy = V.nxy, cx = V.cx, cz = V.nz + 2;
        const uint32_t row = (uint32_t)cx * (uint32_t)cz;
        const float nx1 = (float)(nx - 1), ny1 = (float)(ny - 1), nz1 = (float)(nz - 1);
        // the ray in lattice coordinates (voxel units, cell corners at integers):
        // g(t) = g0 + t gd per axis, one FMA per axis and interval
        const float g0x = (J.Sx - V.lox) * V.idx - 0.5f, g0y = (J.Sy - V.loy) * V.idy - 0.5f,
                    g0z = (J.Sz - V.loz) * V.idz - 0.5f;
        const float gdx = dx * V.idx, gdy = dy * V.idy, gdz = dz * V.idz;
        const int n_mat = P.n_mat;
        float acc = 0.0f;
        int cur = -1;
        // Interval j: its length inside the box h (<= 0 outside the ray's part
        // in the box), the lattice cell (ix, iy, iz) of its midpoint (clamped)
        // and the fractions there.  from: j dl.
        auto interval = [&](float from, float to, float& h, float& fx, float& fy, float& fz, int& ix, int& iy, int& iz) {
            const float a = fmaxf(from, t0), e = fminf(to, t1);
            h = e - a;
            const float t = 0.5f * (a + e);
            const float gx = g0x + t * gdx, gy = g0y + t * gdy, gz = g0z + t * gdz;
            const float fx0 = floorf(gx), fy0 = floorf(gy), fz0 = floorf(gz);
            // (volumes beyond 2^24 voxels along an axis: the clamp still keeps the index inside)
            ix = (int)__builtin_amdgcn_fmed3f(fx0, -1.0f, nx1);
            iy = (int)__builtin_amdgcn_fmed3f(fy0, -1.0f, ny1);
            iz = (int)__builtin_amdgcn_fmed3f(fz0, -1.0f, nz1);
            if (!SMALL) {
                ix = min(ix, nx - 1);
                iy = min(iy, ny - 1);
                iz = min(iz, nz - 1);
            }
            fx = fminf(fmaxf(gx - fx0, 0.0f), 1.0f);
            fy = fminf(fmaxf(gy - fy0, 0.0f), 1.0f);
            fz = fminf(fmaxf(gz - fz0, 0.0f), 1.0f);
        };
        // one interval's density-length, in its ray's order: the register sum of the current
        // material, to its slot when the material changes
        const auto add_single = [&](int m, float h, float rho) {
            if (m != cur) {
                if (cur >= 0 && l == 0) Lm[cur * kRays] += acc;
                cur = m;
                acc = 0.0f;
            }
            acc += h * rho;
        };
        // one interval of slack on both sides (rounding of t / dl); empty ones have h <= 0
        const int jb = (int)floorf(t0 / dl) - 1, je = (int)ceilf(t1 / dl) + 1;
        if (!P.interp) {
            for (int j0 = jb; j0 < je; j0 += G) {
                const int j = j0 + l;
                float h, fx, fy, fz;
                int ix, iy, iz;
                interval((float)j * dl, (float)(j + 1) * dl, h, fx, fy, fz, ix, iy, iz);
                // containing voxel: the cell corner nearest to the point
                const int vx = min(max(ix + (fx >= 0.5f ? 1 : 0), 0), nx - 1);
                const int vy = min(max(iy + (fy >= 0.5f ? 1 : 0), 0), ny - 1);
                const int vz = min(max(iz + (fz >= 0.5f ? 1 : 0), 0), nz - 1);
                const long long v = (long long)vz * nxy + (long long)vy * nx + vx;
                const int m = h > 0.0f ? min((int)mats[v], n_mat - 1) : -1;
                const float rho = clean_density(dens[v]);
                for_group<G>([&](auto k) {
                    const int mk = group_lane<G, k.value>(m);
                    const float hk = group_lane<G, k.value>(h), rk = group_lane<G, k.value>(rho);
                    if (mk >= 0) add_single(mk, hk, rk);
                });
            }
        } else {
            // an interval with the corners around its midpoint
            struct Step {
                float h, fx, fy, fz;
                int ix, iy, iz;
                uint32_t cell;
                Plane d0, d1;
                uint32_t cm;                                   // materials of the eight corners, 4 bits each (G > 1)
            };
            const auto place = [&](float from, float to, Step& q) {
                interval(from, to, q.h, q.fx, q.fy, q.fz, q.ix, q.iy, q.iz);
                // (unsigned: up to 3/2 of 2^31 records)
                if (SMALL)
                    q.cell = mul_u24((uint32_t)(q.iy + 1), row) + mul_u24((uint32_t)(q.ix + 1), (uint32_t)cz) + (uint32_t)(q.iz + 1);
                else
                    q.cell = (uint32_t)((q.iy + 1) * cx + (q.ix + 1)) * (uint32_t)cz + (uint32_t)(q.iz + 1);
            };
            const auto read = [&](Step& q) {
                q.d0 = planes[q.cell];
                q.d1 = planes[(size_t)q.cell + 1];
                if (G > 1) q.cm = *reinterpret_cast<const CodePair*>(codes + q.cell);
            };
            const auto add = [&](const Step& q) {
                // the densities without their flag bits
                const float c0 = fabsf(q.d0.x), c1 = fabsf(q.d0.y), c2 = fabsf(q.d0.z), c3 = fabsf(q.d0.w);
                const float c4 = fabsf(q.d1.x), c5 = fabsf(q.d1.y), c6 = fabsf(q.d1.z), c7 = fabsf(q.d1.w);
                const float fx = q.fx, fy = q.fy, fz = q.fz;
                // the cell's material; -1 for several, -2 outside the box
                int m = plane_code(q.d0);
                m = m != kPlaneLook ? m : -1;
                m = q.h > 0.0f ? m : -2;
                uint32_t cm = q.cm;
                if (m == -1) {
                    if (G == 1) cm = *reinterpret_cast<const CodePair*>(codes + q.cell);
                    // (material kPlaneLook itself; without it nothing waits for the codes here)
                    if ((G > 1 || M16) && cm == 0x11111111u * (cm & 15u)) m = (int)(cm & 15u);
                }
                const float a00 = c0 + fx * (c1 - c0), a01 = c2 + fx * (c3 - c2);
                const float a10 = c4 + fx * (c5 - c4), a11 = c6 + fx * (c7 - c6);
                const float b0 = a00 + fy * (a01 - a00), b1 = a10 + fy * (a11 - a10);
                const float rho = b0 + fz * (b1 - b0);
                for_group<G>([&](auto k) {
                    const int mk = group_lane<G, k.value>(m);
                    const float hk = group_lane<G, k.value>(q.h), rk = group_lane<G, k.value>(rho);
                    if (mk >= 0) {
                        add_single(mk, hk, rk);
                    } else if (mk == -1) {
                        rt_share<G>();
                        if (l == k.value) {
                            const float gx0 = 1.0f - fx, gy0 = 1.0f - fy, gz0 = 1.0f - fz;
                            const float wz0 = q.h * gz0, wz1 = q.h * fz;
                            const float cd[8] = {c0, c1, c2, c3, c4, c5, c6, c7};
                            if constexpr (G <= 4) {
#pragma unroll
                                for (int c = 0; c < 8; ++c) {
                                    const float wc = (c & 1 ? fx : gx0) * (c & 2 ? fy : gy0) * (c & 4 ? wz1 : wz0);
                                    Lm[((cm >> (4 * c)) & 15u) * kRays] += wc * cd[c];
                                }
                            } else {
                                // Material by material, each one's corners in their order (the latency of two
                                // LDS updates instead of eight: one 16 x 16 image 81 us against 87).  left: a bit
                                // (the highest) in the nibble of every corner still to add.
                                uint32_t left = 0x88888888u;
                                do {
                                    const uint32_t mat = (cm >> (__builtin_ctz(left) - 3)) & 15u;
                                    const uint32_t other = cm ^ (0x11111111u * mat);       // nibble 0: this material
                                    float sum = Lm[mat * kRays];
#pragma unroll
                                    for (int c = 0; c < 8; ++c) {
                                        const float wc = (c & 1 ? fx : gx0) * (c & 2 ? fy : gy0) * (c & 4 ? wz1 : wz0);
                                        sum = __builtin_fmaf(wc, other & (15u << (4 * c)) ? 0.0f : cd[c], sum);
                                    }
                                    Lm[mat * kRays] = sum;
                                    left &= ((other & 0x77777777u) + 0x77777777u) | other;
                                } while (left);
                            }
                        }
                        rt_share<G>();
                    }
                });
            };
            // Software-pipelined: the next interval's corners are read while this one is summed,
            // unless it lies in the same cell (intervals are half a voxel long: two in five do;
            // their lanes send no request).  Reading further ahead gains nothing.
            float edge = (float)(jb + l + 1) * dl;             // the current interval's end
            Step q;
            place((float)(jb + l) * dl, edge, q);
            read(q);
            for (int j0 = jb; j0 < je; j0 += G) {
                Step n;
                const float from = G == 1 ? edge : (float)(j0 + l + G) * dl;
                edge = (float)(j0 + l + G + 1) * dl;
                place(from, edge, n);
                n.d0 = q.d0;
                n.d1 = q.d1;
                if (G > 1) n.cm = q.cm;
                if (n.cell != q.cell) read(n);
                add(q);
                q = n;
            }
        }
        if (cur >= 0 && l == 0) Lm[cur * kRays] += acc;
    }
    rt_share<G>();

    float Lr[GDRR_MAX_MATERIALS];
#pragma unroll
    for (int m = 0; m < GDRR_MAX_MATERIALS; ++m) Lr[m] = m < P.n_mat ? Lm[m * kRays] : 0.0f;
    const RtSource& S = P.src[J.src];
    const float* coef = S.coef + (S.rows > 1 ? iu * S.n_spec : 0);
    float sum = 0.0f;
    for (int k0 = 0; k0 < S.n_spec; k0 += G) {
        const int k = G == 1 ? k0 : min(k0 + l, S.n_spec - 1);
        const float* row = S.tab + k * P.n_mat;
        float tau = 0.0f;
#pragma unroll
        for (int m = 0; m < GDRR_MAX_MATERIALS; ++m)
            if (m < P.n_mat) tau += row[m] * Lr[m];
        const float c = coef[k], e = expf(-tau);
        for_group<G>([&](auto q) {
            const float cq = group_lane<G, q.value>(c), eq = group_lane<G, q.value>(e);
            if (G == 1 || k0 + q.value < S.n_spec) sum += cq * eq;
        });
    }
    if (l != 0) return;
    const int pix = iv * J.nu + iu;
    const double val = (double)S.fluence[pix] * S.inv_wsum[0] * (double)sum;
    double* o = P.out + P.out_off[J.index] + pix;
    *o = P.accumulate ? *o + val : val;
}

// Plane records of a volume, by tiles of kPlX cell columns in x by up to kPlZ
// planes of one cell row: the tile's two voxel rows go through LDS (read with x
// along the lanes, written with z along the lanes, both contiguous; the odd row
// length keeps the LDS banks apart).
constexpr int kPlX = 32, kPlZ = 64;

struct PlaneParams {
    const float* density;
    const uint8_t* material;
    int nx, ny, nz, n_mat;
    int tiles_x, tiles_z, tz;  // planes per tile (<= kPlZ)
    unsigned int tiles;        // tiles_x tiles_z (ny + 1), taken in turns by the workgroups
    Plane* planes;
    uint16_t* codes;           // the four corners' materials, 4 bits each
    unsigned int* error;       // input-error bits (invalid densities or materials)
};

__global__ __launch_bounds__(256) void planes_kernel(PlaneParams C) {
    __shared__ float s_d[2][kPlZ + 1][kPlX + 1];
    __shared__ uint8_t s_m[2][kPlZ + 1][kPlX + 4];
    unsigned int err = 0u;
    for (unsigned int tile = blockIdx.x; tile < C.tiles; tile += gridDim.x) {
        const unsigned int tx = tile % (unsigned)C.tiles_x, rest = tile / (unsigned)C.tiles_x;
        const int tz = (int)(rest % (unsigned)C.tiles_z), j = (int)(rest / (unsigned)C.tiles_z) - 1;
        const int i0 = (int)tx * kPlX - 1;                         // the tile's first cell column
        const int cols = min(kPlX, C.nx - i0);                     // columns i0 .. i0 + cols - 1 <= nx - 1
        const int p0 = tz * C.tz, np = min(C.tz, C.nz + 2 - p0);   // planes p0 .. p0 + np - 1
        for (int e = threadIdx.x; e < 2 * (np + 1) * (cols + 1); e += 256) {        // (and the plane above the tile)
            const int q = e / (cols + 1), x = e - q * (cols + 1);
            const int r = q / (np + 1), z = q - r * (np + 1);
            const int vx = min(max(i0 + x, 0), C.nx - 1), vy = min(max(j + r, 0), C.ny - 1);
            const int vz = min(max(p0 + z - 1, 0), C.nz - 1);
            const size_t v = ((size_t)vz * C.ny + vy) * C.nx + vx;
            const float rho = C.density[v];
            const int mr = C.material[v];
            if (!density_ok(rho)) err |= kErrDensity;
            if (mr >= C.n_mat) err |= kErrMaterial;
            s_d[r][z][x] = fabsf(clean_density(rho));              // (-0 loses its sign too)
            s_m[r][z][x] = (uint8_t)min(mr, C.n_mat - 1);
        }
        __syncthreads();
        for (int e = threadIdx.x; e < cols * kPlZ; e += 256) {
            const int x = e / kPlZ, z = e % kPlZ;
            if (z >= np) continue;
            const int m0 = s_m[0][z][x], m1 = s_m[0][z][x + 1], m2 = s_m[1][z][x], m3 = s_m[1][z][x + 1];
            const int n0 = s_m[0][z + 1][x], n1 = s_m[0][z + 1][x + 1], n2 = s_m[1][z + 1][x], n3 = s_m[1][z + 1][x + 1];
            const bool same = m0 == m1 && m0 == m2 && m0 == m3 && m0 == n0 && m0 == n1 && m0 == n2 && m0 == n3;
            const uint32_t code = same ? (uint32_t)m0 : (uint32_t)kPlaneLook;
            Plane d;
            d.x = __uint_as_float(__float_as_uint(s_d[0][z][x]) | (code & 8u) << 28);
            d.y = __uint_as_float(__float_as_uint(s_d[0][z][x + 1]) | (code & 4u) << 29);
            d.z = __uint_as_float(__float_as_uint(s_d[1][z][x]) | (code & 2u) << 30);
            d.w = __uint_as_float(__float_as_uint(s_d[1][z][x + 1]) | (code & 1u) << 31);
            const size_t at = ((size_t)(j + 1) * (C.nx + 1) + (i0 + x + 1)) * (C.nz + 2) + (p0 + z);
            __builtin_nontemporal_store(d, &C.planes[at]);   // (512 x 512 x 256: 427 us, 482 through the caches)
            C.codes[at] = (uint16_t)(m0 | m1 << 4 | m2 << 8 | m3 << 12);
        }
        __syncthreads();                                           // (before the next tile's voxels)
    }
    if (err) atomicOr(C.error, err);
}

// Input check of a volume the ray tracer reads without plane records (no
// interpolation): the status bits of invalid densities and materials.
struct VolCheckParams {
    const float* density;
    const uint8_t* material;
    long long n;
    int n_mat;
    unsigned int* error;
};

__global__ __launch_bounds__(256) void volume_check_kernel(VolCheckParams C) {
    unsigned int err = 0u;
    for (long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x; v < C.n; v += (long long)gridDim.x * blockDim.x) {
        if (!density_ok(C.density[v])) err |= kErrDensity;
        if (C.material[v] >= C.n_mat) err |= kErrMaterial;
    }
    if (err) atomicOr(C.error, err);
}

// Per source: the channel weights phi_k r(E_k) / sum phi (workgroup r: rows r, r + grid
// - 1, ... of a joint source), the table 0.1 mu_tot(m, E_k) (linear in E between grid
// points; workgroup 0) and 1 / sum w (the last workgroup, one CU's loads: 16 in
// flight per lane: 256 x 192 weights 6.6 us, was 56 with 256 lanes and one load each).
struct RtPrepParams {
    const float* spec_e;
    const float* spec_p;          // [rows][n_spec]
    const float* fluence;
    int n_spec, npix, rows;
    const float* mu_mass;         // [n_mat][n_e][3]
    const float* response;        // [n_e] or null
    int n_mat, n_e;
    double e0, de;
    float* coef;
    float* tab;
    double* inv_wsum;
    unsigned int* error;          // input-error bits (invalid spectrum or fluence weights)
};

constexpr int kRtPrepBlock = 1024;

__global__ __launch_bounds__(kRtPrepBlock) void raytrace_prep_kernel(RtPrepParams R) {
    __shared__ double red[kRtPrepBlock];
    const bool fluence = blockIdx.x + 1 == gridDim.x;
    for (int row = fluence ? R.rows - 1 : (int)blockIdx.x; row < R.rows; row += (int)gridDim.x - 1) {
        const float* phi = fluence ? R.fluence : R.spec_p + (size_t)row * R.n_spec;
        const int n = fluence ? R.npix : R.n_spec;
        double sum = 0.0;
        bool bad = false;
        int k = threadIdx.x;
        for (; k + 15 * kRtPrepBlock < n; k += 16 * kRtPrepBlock) {    // 16 loads in flight
            float v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = phi[k + u * kRtPrepBlock];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const double x = (double)v[u];
                bad = bad || !(x >= 0.0) || isinf(x);
                sum += x;
            }
        }
        for (; k < n; k += kRtPrepBlock) {
            const double x = (double)phi[k];
            bad = bad || !(x >= 0.0) || isinf(x);
            sum += x;
        }
        red[threadIdx.x] = sum;
        __syncthreads();
        for (int s = kRtPrepBlock / 2; s > 0; s >>= 1) {
            if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
            __syncthreads();
        }
        const double psum = red[0];
        if (bad || (threadIdx.x == 0 && !(psum > 0.0))) atomicOr(R.error, kErrWeights);
        if (fluence) {
            if (threadIdx.x == 0) R.inv_wsum[0] = psum > 0.0 ? 1.0 / psum : 0.0;
            return;
        }
        float* coef = R.coef + (size_t)row * R.n_spec;
        for (int k = threadIdx.x; k < R.n_spec; k += kRtPrepBlock) {
            const double E = (double)R.spec_e[k];
            const double g = (E - R.e0) / R.de;
            int j = (int)floor(g);
            j = j < 0 ? 0 : (j > R.n_e - 2 ? R.n_e - 2 : j);
            const double f = g - (double)j;
            double r = E;
            if (R.response) r = (double)R.response[j] + f * ((double)R.response[j + 1] - (double)R.response[j]);
            coef[k] = psum > 0.0 ? (float)((double)phi[k] / psum * r) : 0.0f;
            if (row != 0) continue;
            for (int m = 0; m < R.n_mat; ++m) {
                const float* a = R.mu_mass + ((size_t)m * R.n_e + j) * 3;
                const double ta = (double)a[0] + (double)a[1] + (double)a[2];
                const double tb = (double)a[3] + (double)a[4] + (double)a[5];
                R.tab[k * R.n_mat + m] = (float)(0.1 * (ta + f * (tb - ta)));
            }
        }
        __syncthreads();
    }
}

}  // namespace gdrr
