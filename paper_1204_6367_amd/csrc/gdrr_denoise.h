// Scatter denoising (Sec. 2.5, Eq. 5) and noise assembly (Sec. 2.6).
//
// Eq. 5 is a Jacobi-type sweep: every pixel's new value needs its four
// neighbours' previous values.  A pass loads a region of the image into
// registers and runs several sweeps on it without touching memory: a wrong
// value at the region's edge (its missing neighbours are taken as itself) moves
// inward one pixel per sweep, so all pixels `halo` away from it stay exact for
// `halo` sweeps.  Regions are shifted to lie inside the image, and at the
// image's own edges the missing neighbour is the pixel itself, as in the
// definition, so pixels there need no halo, and an image that fits one region
// takes all its sweeps in one pass.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace gdrr {

constexpr int kDnMaxWaves = 16;

struct DnParams {
    const double* shat;       // image k at shat + k * shat_stride, [nv][nu]
    long long shat_stride;
    const float* h_in;        // Shat as float32 [n][nv][nu] from an earlier pass, or null: from shat
    float* h_out;             // for the next passes, or null
    const float* s_in;        // previous pass [n][nv][nu], or null: start from max(shat, floor)
    float* s_out;             // next pass (float), or null
    double* out;              // final pass [n][nv][nu] (double), or null
    int n_img, nv, nu, tiles_u, tiles_v, halo;
    int iters;                // sweeps in this pass (<= halo, unless the image is one tile)
    float omega, inv_beta, s_floor;
};

// Values from the lanes on either side (DPP whole-wavefront shifts: lane i reads
// v of lane i - 1, resp. i + 1); lane 0, resp. 63, gets its own `own`, the missing
// neighbour at the region's edge.
__device__ __forceinline__ float dn_from_left(float own, float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(own), __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float dn_from_right(float own, float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(own), __float_as_int(v), 0x130, 0xf, 0xf, false));
}

// 1 - Shat/S with the hardware reciprocal (about 1 ulp); 1 where Shat = 0.  SEL:
// by a comparison; otherwise 0 times the reciprocal is 0 by itself, which holds
// while no iterate is below the least normal number (the reciprocal would be
// infinite).
template <bool SEL>
__device__ __forceinline__ float dn_data(float h, float s) {
    const float d = 1.0f - h * __builtin_amdgcn_rcpf(s);
    return SEL && h == 0.0f ? 1.0f : d;
}

// One pass over tiles of an image: the region is 64 C columns by R rows per
// wavefront, lane l holding columns l C .. l C + C - 1 of its wavefront's rows in
// registers.  Vertical neighbours are registers (the bands' edge rows go through
// LDS, in two buffers used by turns: the writes of sweep i + 2 come after the
// barrier of sweep i + 1, which every read of sweep i precedes, so one barrier a
// sweep suffices); horizontal ones come from the neighbouring lanes by DPP.
// EDGE: the image is narrower or shorter than the region.  The right edge is
// then a select, and the row below the last one is kept equal to it.
// The first RL of a wavefront's rows of Shat are kept in LDS, where the registers do not hold
// them all (whole images).
// Two sweeps per turn of the loop, one downwards and one upwards: a row's new values go
// to the registers that held its neighbour's old ones, and the second sweep brings them
// back without moves (not for whole images, where that spilled).
// Whole images of 64 and 256 columns are read and written from one pointer by uniform offsets: an
// address for each row spilled 64 and 14 VGPRs around the loop (1000 images of 64x384, 30 sweeps, 429 -> 375 us).
// With 128 columns that is kept, 24 VGPRs outside the loop: the loop that comes with one pointer
// waits more (1000 images of 128x384, 256 sweeps, 4.18 ms, 4.45 without the spills; 8 sweeps 270 and 272 us).
// Bound by VALU issue, about 10 instructions a pixel and sweep of which the reciprocal
// counts four times, and for few regions by the barrier's round trip (0.25 us a sweep).
// 256 sweeps: one 512 x 384 image 167 us, 460 with regions of 64 x 80 pixels on 4 wavefronts
// and halos of 8; one 256 x 192 image 155, 1160 in one workgroup; 360 of them 2140, one
// workgroup each (2 x 256 x 4.2 us), 2390 with the comparison of dn_data; 64 sweeps of 60
// images of 512 x 384: 512, was 815; 100 sweeps of 2000 images of 64 x 48: 310, was 1220.
template <int C, int R, int RL, bool EDGE, bool SEL>
__global__ __launch_bounds__(64 * kDnMaxWaves) void denoise_tile_kernel(DnParams D) {
    __shared__ float edge[2][2][kDnMaxWaves][64 * C];
    __shared__ float4 h_lds[RL ? RL : 1][RL ? kDnMaxWaves : 1][RL ? 16 * C : 1];   // [row][wavefront][lane's C values]
    constexpr bool WHOLE = RL > 0, ONE = WHOLE && C != 2;  // the image is one region exactly; and from one pointer
    const int waves = blockDim.x >> 6, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int cols = 64 * C, rows = R * waves;
    const int per_img = D.tiles_u * D.tiles_v;
    const int img = blockIdx.x / per_img, t = blockIdx.x % per_img;
    const int tv = t / D.tiles_u, tu = t % D.tiles_u;
    const int du = cols - 2 * D.halo, dv = rows - 2 * D.halo;              // from tile to tile
    const int x0 = WHOLE ? 0 : max(min(tu * du, D.nu - cols), 0), y0 = WHOLE ? 0 : max(min(tv * dv, D.nv - rows), 0);
    // the tile's own pixels
    const int ux0 = tu == 0 ? 0 : tu * du + D.halo, ux1 = tu + 1 == D.tiles_u ? D.nu : (tu + 1) * du + D.halo;
    const int vy0 = tv == 0 ? 0 : tv * dv + D.halo, vy1 = tv + 1 == D.tiles_v ? D.nv : (tv + 1) * dv + D.halo;
    const size_t npix = (size_t)D.nv * D.nu;
    const int r0 = y0 + wave * R, c0 = x0 + lane * C;
    const double* H = D.shat + (size_t)img * D.shat_stride;
    const float* Hf = D.h_in ? D.h_in + (size_t)img * npix : nullptr;
    const float* Sin = D.s_in ? D.s_in + (size_t)img * npix : nullptr;
    const double* const Hw = H + (size_t)r0 * D.nu + c0;
    float s[R][C], h[R - RL][C];
    float* const hl = reinterpret_cast<float*>(&h_lds[0][RL ? wave : 0][0]) + lane * C;   // row k at hl[k kDnMaxWaves 64 C]
#pragma unroll
    for (int k = 0; k < R; ++k)
#pragma unroll
        for (int c = 0; c < C; ++c) {
            // (EDGE: rows and columns beyond the image repeat its last ones)
            const int y = EDGE ? min(r0 + k, D.nv - 1) : r0 + k, x = EDGE ? min(c0 + c, D.nu - 1) : c0 + c;
            const size_t p = (size_t)y * D.nu + x;
            const float hv = ONE ? (float)Hw[(size_t)k * D.nu + c] : !WHOLE && Hf ? Hf[p] : (float)H[p];
            if (k < RL) hl[k * kDnMaxWaves * 64 * C + c] = hv;
            else h[k - RL][c] = hv;
            s[k][c] = !WHOLE && Sin ? Sin[p] : fmaxf(hv, D.s_floor);
            if (!WHOLE && D.h_out && y >= vy0 && y < vy1 && x >= ux0 && x < ux1) D.h_out[(size_t)img * npix + p] = hv;
        }
    const float w1 = 1.0f - D.omega, qw = 0.25f * D.omega;
    // one sweep, from the first row down (DOWN) or from the last row up; e: its edge buffer
    auto sweep = [&](auto down_, int e) {
        constexpr bool DOWN = decltype(down_)::value;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            edge[e][0][wave][lane * C + c] = s[0][c];
            edge[e][1][wave][lane * C + c] = s[R - 1][c];
        }
        __syncthreads();
        float above[C], below[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            above[c] = wave > 0 ? edge[e][1][wave - 1][lane * C + c] : s[0][c];
            below[c] = wave < waves - 1 ? edge[e][0][wave + 1][lane * C + c] : s[R - 1][c];
        }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int k = DOWN ? q : R - 1 - q;
            // the row's old values and its neighbours outside this lane's columns
            float row[C], hrow[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                row[c] = s[k][c];
                hrow[c] = k < RL ? hl[k * kDnMaxWaves * 64 * C + c] : h[k < RL ? 0 : k - RL][c];
            }
            const float left = dn_from_left(row[0], row[C - 1]);
            const float right = dn_from_right(row[C - 1], row[0]);
            const bool last = EDGE && r0 + k == D.nv - 1;                  // (wavefront-uniform)
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float sk = row[c];
                const float up = DOWN || k == 0 ? above[c] : s[k - 1][c];
                const float next = !DOWN || k + 1 == R ? below[c] : s[k + 1][c];
                const float dn = last ? sk : next;
                const float lf = c > 0 ? row[c - 1] : left;
                float rt = c + 1 < C ? row[c + 1] : right;
                if (EDGE) rt = c0 + c == D.nu - 1 ? sk : rt;
                const float v = w1 * sk + qw * ((up + dn + lf + rt) - dn_data<SEL>(hrow[c], sk) * D.inv_beta);
                s[k][c] = fmaxf(v, D.s_floor);
                (DOWN ? above : below)[c] = sk;           // old value, a neighbour of the next row
            }
        }
    };
    if (WHOLE) {
        for (int it = 0; it < D.iters; ++it) sweep(std::true_type{}, it & 1);
    } else {
        const int odd = D.iters & 1;                       // (the odd one first)
        if (odd) sweep(std::true_type{}, 1);
        for (int it = odd; it < D.iters; it += 2) {
            sweep(std::true_type{}, 0);
            sweep(std::false_type{}, 1);
        }
    }
    double* const Dw = ONE ? D.out + (size_t)img * npix + (size_t)r0 * D.nu + c0 : nullptr;
#pragma unroll
    for (int k = 0; k < R; ++k)
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int y = r0 + k, x = c0 + c;
            if (ONE) {
                Dw[(size_t)k * D.nu + c] = (double)s[k][c];
                continue;
            }
            if (!WHOLE && (y < vy0 || y >= vy1 || x < ux0 || x >= ux1)) continue;
            const size_t p = (size_t)img * npix + (size_t)y * D.nu + x;
            if (WHOLE || D.out) D.out[p] = (double)s[k][c];
            else D.s_out[p] = s[k][c];
        }
}

// N = alpha ((Phat - P) + (Shat - S)) and the projection P + S + N, per pixel.
struct NoiseParams {
    const double* phat;       // image k at phat + k * phat_stride
    long long phat_stride;
    const double* p;          // [n][npix]
    const double* shat;       // image k at shat + k * shat_stride
    long long shat_stride;
    const double* s;          // [n][npix]
    double alpha;
    double* noise;            // [n][npix] or null
    double* image;            // [n][npix] or null
    long long npix, n;        // pixels per image, images
};

__global__ __launch_bounds__(256) void noise_kernel(NoiseParams Q) {
    const long long total = Q.npix * Q.n;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const long long k = i / Q.npix, q = i - k * Q.npix;
        const double ph = Q.phat[k * Q.phat_stride + q], sh = Q.shat[k * Q.shat_stride + q];
        const double pp = Q.p[i], ss = Q.s[i];
        const double nn = Q.alpha * ((ph - pp) + (sh - ss));
        if (Q.noise) Q.noise[i] = nn;
        if (Q.image) Q.image[i] = (pp + ss) + nn;
    }
}

}  // namespace gdrr
