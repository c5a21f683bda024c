// Host side of libgdrr: argument checks, workspace layout, launch plans,
// the cached HIP graph of a batch, and the C ABI of include/gdrr.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "gdrr.h"
#include "gdrr_kernels.h"
#include "gdrr_raytrace.h"
#include "gdrr_denoise.h"

using namespace gdrr;

namespace {

thread_local std::string g_err;

int fail(int code, const std::string& msg) {
    g_err = msg;
    return code;
}

#define GDRR_HIP(call)                                                                   \
    do {                                                                                 \
        hipError_t e_ = (call);                                                          \
        if (e_ != hipSuccess) return fail(GDRR_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

// --------------------------------------------------------------------------
// Device properties, read once per device.
// --------------------------------------------------------------------------
struct DevInfo {
    int cus = 0;
    size_t lds_max = 0;      // per workgroup
    bool ok = false;
};

std::mutex g_dev_mu;
DevInfo g_dev[64];

int device_info(DevInfo& out) {
    int dev = 0;
    GDRR_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(GDRR_ENOTSUP, "device index out of range");
    std::lock_guard<std::mutex> lk(g_dev_mu);
    if (!g_dev[dev].ok) {
        hipDeviceProp_t prop;
        GDRR_HIP(hipGetDeviceProperties(&prop, dev));
        g_dev[dev].cus = prop.multiProcessorCount;
        g_dev[dev].lds_max = prop.sharedMemPerBlock;
        g_dev[dev].ok = true;
    }
    out = g_dev[dev];
    return GDRR_OK;
}

// --------------------------------------------------------------------------
// Workspace carving: the same walk sizes the workspace (base == nullptr) and
// lays it out.
// --------------------------------------------------------------------------
struct Carver {
    char* base;
    size_t off = 0;
    explicit Carver(void* b) : base((char*)b) {}
    template <class T>
    T* take(size_t n) {
        off = (off + 255) & ~(size_t)255;
        T* p = base ? (T*)(base + off) : nullptr;
        off += n * sizeof(T);
        return p;
    }
};

// Workgroups of 1024 lanes for the rows of a source's spectrum table (a launch has fewer than 2^32
// lanes, a table up to 2^24 rows).
constexpr int kRowBlocks = 4096;

// Rows of a source's spectrum table (one, or one per detector column); -1 if invalid.
int spec_rows(const gdrr_source& s) {
    if (s.spec_rows == 0 || s.spec_rows == 1) return 1;
    return s.spec_rows == s.fu && s.fu > 1 ? s.spec_rows : -1;
}

uint32_t guide_size(int n) {
    uint32_t k = 1;
    while ((int)k < n && k < (1u << 20)) k <<= 1;
    return k;
}

// --------------------------------------------------------------------------
// Argument checks.
// --------------------------------------------------------------------------
int check_volume(const gdrr_volume* v) {
    if (!v) return fail(GDRR_EINVAL, "volume is NULL");
    if (v->nx < 1 || v->ny < 1 || v->nz < 1) return fail(GDRR_EINVAL, "volume dimensions must be >= 1");
    if ((long long)v->nx * v->ny * v->nz >= (1ll << 31)) return fail(GDRR_EINVAL, "volume has 2^31 voxels or more");
    // cell records are indexed in 32-bit arithmetic
    if ((long long)(v->nx + 1) * (v->ny + 1) * (v->nz + 1) >= (1ll << 31))
        return fail(GDRR_EINVAL, "volume has 2^31 interpolation cells or more ((nx+1)(ny+1)(nz+1))");
    if (!(v->dx_mm > 0 && v->dy_mm > 0 && v->dz_mm > 0)) return fail(GDRR_EINVAL, "voxel sizes must be > 0");
    if (!v->density || !v->material) return fail(GDRR_EINVAL, "volume density/material pointer is NULL");
    if (v->macro < 0 || v->macro > 256) return fail(GDRR_EINVAL, "volume macro must be in [0, 256]");
    if (v->macro > 0 && (!(v->macro_margin >= 0.0f) || !std::isfinite(v->macro_margin)))
        return fail(GDRR_EINVAL, "volume macro_margin must be finite and >= 0");
    if (v->macro > 0 && (!(v->macro_rho_min >= 0.0f) || !std::isfinite(v->macro_rho_min)))
        return fail(GDRR_EINVAL, "volume macro_rho_min must be finite and >= 0");
    return GDRR_OK;
}

int cubes(int n, int m) { return (n + m - 1) / m; }
size_t cubes_of(const gdrr_volume& v, int m) {
    return (size_t)cubes(v.nx, m) * (size_t)cubes(v.ny, m) * (size_t)cubes(v.nz, m);
}

// The end of the workspace, which the queries count and calls run without too (a call is refused
// only for want of what its layout needs): the chunk dispensers, and the records of the screening
// cubes of a launch's single-majorant volumes.
constexpr size_t kDispBytes = (size_t)kDispensers * kDispStride * sizeof(unsigned long long);
// (16 KiB of LDS.  1e7 photons, ms with 512, 1024, 2048, 4096, 8192 cubes: 64x64x64 2.41 2.23 2.12 2.01 1.98,
// 128x128x96 2.51 2.18 2.15 2.02 2.00, 256x256x160 2.25 2.23 1.96 1.92 1.96, 512x512x256 2.30 2.10 2.03 1.99 2.03)
constexpr size_t kScreenCubes = 4096;
constexpr size_t kExtraBytes = kDispBytes + kScreenCubes * sizeof(uint2) + 512;

// The smallest cube edge (2 voxels or more) that cuts the volume into at most `most` cubes.
int screen_cube_of(const gdrr_volume& v, size_t most) {
    int m = 2;
    while (cubes_of(v, m) > most) ++m;
    return m;
}

#ifndef GDRR_MACRO_LDS_MAX
#define GDRR_MACRO_LDS_MAX (32 << 10)
#endif
constexpr size_t kMacroLdsMax = GDRR_MACRO_LDS_MAX;   // bytes of cube records staged in LDS
constexpr size_t kPaddedLdsMax = 112 << 10;            // the same with the padding of all-local grids

int check_physics(const gdrr_physics* p) {
    if (!p) return fail(GDRR_EINVAL, "physics is NULL");
    if (p->n_mat < 1 || p->n_mat > GDRR_MAX_MATERIALS) return fail(GDRR_EINVAL, "n_mat must be in [1, 16]");
    if (p->n_e < 2 || p->n_e > 1024) return fail(GDRR_EINVAL, "n_e must be in [2, 1024]");
    if (!(p->de_kev > 0) || !(p->e0_kev > 0)) return fail(GDRR_EINVAL, "energy grid must have e0 > 0 and de > 0");
    if (!p->mu_mass) return fail(GDRR_EINVAL, "mu_mass is NULL");
    if (!(p->e_cut_kev >= p->e0_kev)) return fail(GDRR_EINVAL, "e_cut must be >= e0");
    if (!(p->rayleigh_x0_invA > 0)) return fail(GDRR_EINVAL, "rayleigh x0 must be > 0");
    return GDRR_OK;
}

int check_source(const gdrr_source* s) {
    if (!s) return fail(GDRR_EINVAL, "source is NULL");
    if (s->n_spec < 1 || s->n_spec > 4096) return fail(GDRR_EINVAL, "n_spec must be in [1, 4096]");
    if (!s->spec_e_kev || !s->spec_prob || !s->fluence) return fail(GDRR_EINVAL, "source pointer is NULL");
    if (s->fu < 1 || s->fv < 1 || (long long)s->fu * s->fv > (1ll << 24))
        return fail(GDRR_EINVAL, "fluence grid must have 1 <= fu*fv <= 2^24");
    if (spec_rows(*s) < 0) return fail(GDRR_EINVAL, "spec_rows must be 0, 1 or fu");
    if ((long long)spec_rows(*s) * s->n_spec > (1ll << 24)) return fail(GDRR_EINVAL, "spec_rows * n_spec must be <= 2^24");
    return GDRR_OK;
}

int check_geometry(const gdrr_geometry* g, const gdrr_volume* v, const gdrr_source* s) {
    if (!g) return fail(GDRR_EINVAL, "geometry is NULL");
    if (!(g->sad_mm > 0 && g->aid_mm > 0)) return fail(GDRR_EINVAL, "SAD and AID must be > 0");
    if (g->nu < 1 || g->nv < 1 || !(g->du_mm > 0 && g->dv_mm > 0)) return fail(GDRR_EINVAL, "bad detector grid");
    if (!std::isfinite(g->phi_rad) || !std::isfinite(g->theta_rad)) return fail(GDRR_EINVAL, "angles must be finite");
    if (s && (s->fu != g->nu || s->fv != g->nv))
        return fail(GDRR_EINVAL, "the fluence grid must be the detector's pixel grid (fu = nu, fv = nv)");
    if (v) {
        const double hx = 0.5 * v->nx * v->dx_mm, hy = 0.5 * v->ny * v->dy_mm;
        const double r = std::sqrt(hx * hx + hy * hy);
        if (!(r < g->aid_mm) || !(r < g->sad_mm))
            return fail(GDRR_EINVAL, "the phantom must lie between the source and the detector at every angle");
    }
    return GDRR_OK;
}

// --------------------------------------------------------------------------
// Timing hook: HIP events around the transport kernel, on the call's stream.
// --------------------------------------------------------------------------
struct TimeEvents {
    hipEvent_t a = nullptr, b = nullptr;
    bool recorded = false;
};

std::mutex g_time_mu;
bool g_timing = false;
TimeEvents g_tev[64];

int timing_events(TimeEvents** out) {
    int dev = 0;
    GDRR_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(GDRR_ENOTSUP, "device index out of range");
    TimeEvents& t = g_tev[dev];
    if (!t.a) GDRR_HIP(hipEventCreate(&t.a));
    if (!t.b) GDRR_HIP(hipEventCreate(&t.b));
    *out = &t;
    return GDRR_OK;
}

// --------------------------------------------------------------------------
// Launch list: every kernel takes one parameter struct by value, so a launch
// is (function, grid, block, LDS bytes, argument bytes).  The list runs either
// directly or as a HIP graph.
// --------------------------------------------------------------------------
struct Launch {
    const void* func;
    dim3 grid, block;
    size_t shmem;
    std::vector<char> args;
};

template <class P>
Launch make_launch(const void* f, dim3 g, dim3 b, size_t sh, const P& p) {
    Launch L{f, g, b, sh, std::vector<char>(sizeof(P))};
    std::memcpy(L.args.data(), &p, sizeof(P));
    return L;
}

// Launches [timed, timed_last] are bracketed with `ev` (timed = -1: none;
// timed_last = -1: the single launch `timed`).
int run_direct(std::vector<Launch>& ls, hipStream_t st, int timed = -1, TimeEvents* ev = nullptr,
               int timed_last = -1) {
    if (timed_last < 0) timed_last = timed;
    for (size_t i = 0; i < ls.size(); ++i) {
        Launch& L = ls[i];
        void* a[1] = {L.args.data()};
        if ((int)i == timed) GDRR_HIP(hipEventRecord(ev->a, st));
        GDRR_HIP(hipLaunchKernel(L.func, L.grid, L.block, a, L.shmem, st));
        if (timed >= 0 && (int)i == timed_last) {
            GDRR_HIP(hipEventRecord(ev->b, st));
            ev->recorded = true;
        }
    }
    return GDRR_OK;
}

std::vector<char> launch_key(const std::vector<Launch>& ls) {
    std::vector<char> k;
    for (auto& L : ls) {
        const char* f = (const char*)&L.func;
        k.insert(k.end(), f, f + sizeof(L.func));
        unsigned dims[7] = {L.grid.x, L.grid.y, L.grid.z, L.block.x, L.block.y, L.block.z, (unsigned)L.shmem};
        k.insert(k.end(), (const char*)dims, (const char*)dims + sizeof(dims));
        k.insert(k.end(), L.args.begin(), L.args.end());
    }
    return k;
}

struct GraphEntry {
    int device = -1;
    std::vector<char> key;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

std::mutex g_graph_mu;
GraphEntry g_graphs[4];
int g_graph_next = 0;

int run_graph(std::vector<Launch>& ls, hipStream_t st, int timed = -1, TimeEvents* ev = nullptr) {
    int dev = 0;
    GDRR_HIP(hipGetDevice(&dev));
    std::vector<char> key = launch_key(ls);
    {
        const int t[1] = {timed};
        key.insert(key.end(), (const char*)t, (const char*)t + sizeof(t));
        const void* e[2] = {ev ? (const void*)ev->a : nullptr, ev ? (const void*)ev->b : nullptr};
        key.insert(key.end(), (const char*)e, (const char*)e + sizeof(e));
    }
    if (ev && timed >= 0) ev->recorded = true;
    std::lock_guard<std::mutex> lk(g_graph_mu);
    for (auto& e : g_graphs)
        if (e.exec && e.device == dev && e.key == key) {
            GDRR_HIP(hipGraphLaunch(e.exec, st));
            return GDRR_OK;
        }
    GraphEntry& e = g_graphs[g_graph_next];
    g_graph_next = (g_graph_next + 1) % 4;
    if (e.exec) { (void)hipGraphExecDestroy(e.exec); e.exec = nullptr; }
    if (e.graph) { (void)hipGraphDestroy(e.graph); e.graph = nullptr; }
    GDRR_HIP(hipGraphCreate(&e.graph, 0));
    hipGraphNode_t prev = nullptr;
    for (size_t i = 0; i < ls.size(); ++i) {
        Launch& L = ls[i];
        if ((int)i == timed) {
            hipGraphNode_t en;
            GDRR_HIP(hipGraphAddEventRecordNode(&en, e.graph, prev ? &prev : nullptr, prev ? 1 : 0, ev->a));
            prev = en;
        }
        hipKernelNodeParams kp{};
        void* a[1] = {L.args.data()};
        kp.func = const_cast<void*>(L.func);
        kp.gridDim = L.grid;
        kp.blockDim = L.block;
        kp.sharedMemBytes = (unsigned)L.shmem;
        kp.kernelParams = a;
        kp.extra = nullptr;
        hipGraphNode_t node;
        GDRR_HIP(hipGraphAddKernelNode(&node, e.graph, prev ? &prev : nullptr, prev ? 1 : 0, &kp));
        prev = node;
        if ((int)i == timed) {
            hipGraphNode_t en;
            GDRR_HIP(hipGraphAddEventRecordNode(&en, e.graph, &prev, 1, ev->b));
            prev = en;
        }
    }
    GDRR_HIP(hipGraphInstantiate(&e.exec, e.graph, nullptr, nullptr, 0));
    e.device = dev;
    e.key = std::move(key);
    GDRR_HIP(hipGraphLaunch(e.exec, st));
    return GDRR_OK;
}

// --------------------------------------------------------------------------
// A batch plan: host-side tables and the workspace layout.
// --------------------------------------------------------------------------
struct SrcArea {
    double* spec_cdf;
    uint32_t* spec_guide;
    double* flu_cdf;
    uint32_t* flu_guide;
    uint32_t spec_k, flu_k;
};

struct Layout {
    unsigned long long* counter;      // [8]: dispenser, error word
    unsigned long long* chunk_prefix; // [n_jobs + 1]
    DJob* jobs;                       // [n_jobs]
    long long* out_off;               // [n_jobs]
    float* majorants;                 // [n_vols][n_e - 1] (when computed)
    unsigned int* rho_max;            // [n_vols][256]
    unsigned int* present;            // [n_vols][256]
    SrcArea src[GDRR_MAX_SOURCES];
    CellRec* cells[GDRR_MAX_VOLUMES]; // per-volume cell records
    uint2* macro[GDRR_MAX_VOLUMES];   // per-volume local majorants (volumes with macro > 0)
    unsigned long long* tally;        // fixed-point tallies
    size_t tally_elems;
    size_t bytes;
};

size_t cell_count(const gdrr_volume& v) {
    return (size_t)(v.nx + 1) * (size_t)(v.ny + 1) * (size_t)(v.nz + 1);
}

Layout carve(void* ws, const gdrr_volume* vols, const gdrr_physics* phys, const gdrr_source* srcs, int n_srcs,
             int n_jobs, int n_vols, size_t tally_elems, bool need_majorant) {
    Carver c(ws);
    Layout L{};
    L.counter = c.take<unsigned long long>(8);
    L.chunk_prefix = c.take<unsigned long long>((size_t)n_jobs + 1);
    L.jobs = c.take<DJob>((size_t)n_jobs);
    L.out_off = c.take<long long>((size_t)n_jobs);
    L.majorants = need_majorant ? c.take<float>((size_t)n_vols * (phys->n_e - 1)) : nullptr;
    L.rho_max = c.take<unsigned int>((size_t)n_vols * 256);
    L.present = c.take<unsigned int>((size_t)n_vols * 256);
    for (int s = 0; s < n_srcs; ++s) {
        const int npix = srcs[s].fu * srcs[s].fv;
        L.src[s].spec_k = guide_size(srcs[s].n_spec);
        L.src[s].flu_k = guide_size(npix);
        const size_t rows = (size_t)spec_rows(srcs[s]);
        L.src[s].spec_cdf = c.take<double>(rows * srcs[s].n_spec);
        L.src[s].spec_guide = c.take<uint32_t>(rows * L.src[s].spec_k);
        L.src[s].flu_cdf = c.take<double>((size_t)npix);
        L.src[s].flu_guide = c.take<uint32_t>(L.src[s].flu_k);
    }
    for (int v = 0; v < n_vols; ++v) L.cells[v] = c.take<CellRec>(cell_count(vols[v]));
    for (int v = 0; v < n_vols; ++v) {
        const gdrr_volume& V = vols[v];
        L.macro[v] = V.macro > 0 ? c.take<uint2>((size_t)cubes(V.nx, V.macro) * cubes(V.ny, V.macro) *
                                                 cubes(V.nz, V.macro))
                                 : nullptr;
    }
    L.tally = c.take<unsigned long long>(tally_elems);
    L.tally_elems = tally_elems;
    L.bytes = c.off + 256;
    return L;
}

size_t tally_elems_of(const gdrr_job* jobs, int n_jobs, const gdrr_source* srcs) {
    size_t e = 0;
    for (int k = 0; k < n_jobs; ++k) e += 4 * (size_t)jobs[k].geom.nu * jobs[k].geom.nv;
    (void)srcs;
    return e;
}

// The tables that a call's host code makes for its kernels, with the gaps that the workspace
// leaves between them: one copy, or none where they fit a kernel's arguments.
struct TableImage {
    char* dev;                                 // the first table
    std::vector<char>& host;
    TableImage(void* first, void* end, std::vector<char>& staging) : dev((char*)first), host(staging) {
        host.assign(((size_t)((char*)end - dev) + 3) & ~(size_t)3, 0);
    }
    void put(const void* table, const void* src, size_t bytes) { std::memcpy(host.data() + ((const char*)table - dev), src, bytes); }
};

// Clears `fills` and writes the tables (by the kernel if they fit its arguments and by_kernel
// says so: a cached graph's kernels keep their arguments).
int add_setup(std::vector<Launch>& ls, const std::vector<FillParams>& fills, const TableImage& t, bool by_kernel, hipStream_t st) {
    SetupParams p{};
    size_t most = 1;
    for (const FillParams& f : fills) {
        if (f.n <= 0) continue;
        p.f[p.fills++] = f;
        most = std::max(most, (size_t)f.n);
    }
    by_kernel = by_kernel && t.host.size() <= sizeof(p.image);
    if (by_kernel) {
        p.tables = (uint32_t*)t.dev;
        p.words = (int)(t.host.size() / 4);
        std::memcpy(p.image, t.host.data(), t.host.size());
    }
    ls.push_back(make_launch((const void*)&setup_kernel, dim3((unsigned)std::min<size_t>(4096, (most + 255) / 256)), dim3(256), 0, p));
    if (!by_kernel) GDRR_HIP(hipMemcpyAsync(t.dev, t.host.data(), t.host.size(), hipMemcpyHostToDevice, st));
    return GDRR_OK;
}

// A pass over a volume: its cell records (if cells is not null) and the maxima of its densities.
Launch voxels_launch(const gdrr_volume& V, int n_mat, bool interp, int cus, CellRec* cells, bool maxima,
                     unsigned int* rho_max, unsigned int* present, unsigned int* status) {
    const size_t columns = (size_t)(V.nx + 1) * (size_t)(V.ny + 1), blocks = (columns + 255) / 256;
    int seg_log = 8;
    while (seg_log > 2 && ((size_t)1 << (seg_log - 1)) >= columns) --seg_log;
    // 2 cells in z per workgroup, so that the workgroups in flight write a few planes and not
    // columns all over the records (512 x 512 x 256: 560 us; 4 cells 619, 8 cells 648, 65 cells
    // 692); 4 with the maxima, which every workgroup has to hand in (64^3, no records: 8.7 us
    // against 10.9 with 2); more where the grid's 65535 in y would not do
    const int planes = std::max(maxima ? 4 : 2, (int)(((size_t)V.nz + 65535) / 65535));
    const VoxelParams p{V.density, V.material, V.nx, V.ny, V.nz, n_mat, planes, seg_log, cells, status, rho_max, present};
    const void* const f = !cells  ? (interp ? (const void*)&voxels_kernel<false, 2> : (const void*)&voxels_kernel<false, 1>)
                          : !maxima ? (const void*)&voxels_kernel<true, 0>
                          : interp  ? (const void*)&voxels_kernel<true, 2>
                                    : (const void*)&voxels_kernel<true, 1>;
    return make_launch(f, dim3((unsigned)blocks, (unsigned)((V.nz / planes + (256 >> seg_log)) >> (8 - seg_log))), dim3(256), 0, p);
}

// Lanes per cube of the local majorants and the screening: large cubes are few (13 x 13 x 7 of 40^3
// voxels: 1183 workgroups, 118 us with 1024 lanes, 315 with 256), small ones have no work for more
// than 256 lanes.  A call of 64 photons on 512x512x256 voxels, us with 256 and 1024 lanes at edges of
// 4, 8, 12, 14, 20, 40 and 64: 2474 5936, 1388 1592, 1053 1076, 1036 1064, 955 984, 899 864, 1024 834; on
// 256x256x160 617 1164, 367 416, 293 305, 269 268, 312 309, 309 282, 484 339.
unsigned macro_block(int cube) { return cube > 12 ? 1024u : 256u; }

struct Batch {
    const gdrr_volume* vols;
    int n_vols;
    const gdrr_physics* phys;
    const gdrr_source* srcs;
    int n_srcs;
    const gdrr_job* jobs;
    int n_jobs;
    const float* majorants;     // caller's, or null
    uint64_t seed;
    uint32_t flags;
    const gdrr_tuning* tune;
    int mode;                   // kModeForward / kModeTrace / kModeBackward
    int only_volume;            // backward: jobs of this volume only (-1 = all)
    double* out;                // forward: caller tallies
    const double* adj;          // backward
    double* grad;               // backward
    int8_t* t_cls; int32_t* t_pixel; float* t_e; int32_t* t_steps; int32_t* t_nc; int32_t* t_nr;
    bool use_graph;
    bool tables_by_kernel = false;   // one job: its tables as kernel arguments, no host copy, no timing
};

// Host staging of the per-call tables.  It is pageable memory: a host-to-device
// hipMemcpyAsync from pageable memory returns only once the source has been
// copied out (into the runtime's own staging for the DMA), so the buffer can be
// refilled by the next call while the previous copy is still in flight.
thread_local std::vector<char> g_staging;

// Geometry part of a job record (Sec. 2.1), evaluated in double and stored as float.
DJob djob_of(const gdrr_job& J) {
    const gdrr_geometry& g = J.geom;
    const double phi = g.phi_rad, th = g.theta_rad;
    const double cq = std::cos(phi + th), sq = std::sin(phi + th);
    DJob d{};
    d.Sx = (float)(-g.sad_mm * std::cos(phi));
    d.Sy = (float)(-g.sad_mm * std::sin(phi));
    d.Sz = 0.0f;
    d.Px = (float)(g.aid_mm * cq);
    d.Py = (float)(g.aid_mm * sq);
    d.Pz = 0.0f;
    d.nx = (float)cq; d.ny = (float)sq; d.nz = 0.0f;
    d.ux = (float)(-sq); d.uy = (float)cq; d.uz = 0.0f;
    d.du = g.du_mm; d.dv = g.dv_mm;
    d.idu = (float)(1.0 / g.du_mm); d.idv = (float)(1.0 / g.dv_mm);
    d.nu = g.nu; d.nv = g.nv;
    d.src = J.source; d.vol = J.volume;
    d.job_id = J.job_id;
    return d;
}

int check_batch(const Batch& B) {
    if (B.n_vols < 1 || B.n_vols > GDRR_MAX_VOLUMES) return fail(GDRR_EINVAL, "n_vols must be in [1, 8]");
    if (B.n_srcs < 1 || B.n_srcs > GDRR_MAX_SOURCES) return fail(GDRR_EINVAL, "n_srcs must be in [1, 8]");
    if (B.n_jobs < 1 || B.n_jobs > (1 << 20)) return fail(GDRR_EINVAL, "n_jobs must be in [1, 2^20]");
    if (!B.vols || !B.srcs || !B.jobs) return fail(GDRR_EINVAL, "NULL array argument");
    int rc;
    if ((rc = check_physics(B.phys))) return rc;
    for (int v = 0; v < B.n_vols; ++v)
        if ((rc = check_volume(&B.vols[v]))) return rc;
    for (int s = 0; s < B.n_srcs; ++s)
        if ((rc = check_source(&B.srcs[s]))) return rc;
    for (int k = 0; k < B.n_jobs; ++k) {
        const gdrr_job& J = B.jobs[k];
        if (J.volume < 0 || J.volume >= B.n_vols) return fail(GDRR_EINVAL, "job volume index out of range");
        if (J.source < 0 || J.source >= B.n_srcs) return fail(GDRR_EINVAL, "job source index out of range");
        if (J.n_photons >= (1ull << 32) || (uint64_t)J.first_photon + J.n_photons >= (1ull << 32))
            return fail(GDRR_EINVAL, "a job's photon indices must stay below 2^32 (first_photon + n_photons)");
        if (J.tally_offset < 0) return fail(GDRR_EINVAL, "negative tally offset");
        if ((rc = check_geometry(&J.geom, &B.vols[J.volume], &B.srcs[J.source]))) return rc;
    }
    if (B.tune) {
        const gdrr_tuning& t = *B.tune;
        if (t.block && (t.block % 64 || t.block < 64 || t.block > 1024)) return fail(GDRR_EINVAL, "tune.block must be a multiple of 64 in [64, 1024]");
        if (t.chunk && (t.chunk % 64 || t.chunk < 64)) return fail(GDRR_EINVAL, "tune.chunk must be a positive multiple of 64");
        if (t.defer < 0 || t.defer > 64) return fail(GDRR_EINVAL, "tune.defer must be in [0, 64]");
        if (t.blocks_per_cu < 0 || t.blocks_per_cu > 64) return fail(GDRR_EINVAL, "tune.blocks_per_cu must be in [0, 64]");
        if (t.coll_defer < 0 || t.coll_defer > 64) return fail(GDRR_EINVAL, "tune.coll_defer must be in [0, 64]");
    }
    return GDRR_OK;
}

// local: 0 single majorants, 1 local majorants with records in global memory, 2 with records in LDS,
// 3 (4) every traced volume with local majorants and records in LDS, interpolated (nearest) density,
// 5 every traced volume with a single majorant, screened (forward and trace: the adjoint visits null
// collisions too); block: threads of a workgroup
template <int MODE>
const void* mc_func(int local, int block) {
    if constexpr (MODE == kModeBackward)
        return local == 4 ? reinterpret_cast<const void*>(&mc_adjoint_kernel<4>)
             : local == 3 && block > 768 ? reinterpret_cast<const void*>(&mc_adjoint_kernel<3, 8>)
             : local == 3 ? reinterpret_cast<const void*>(&mc_adjoint_kernel<3>)
             : local == 2 ? reinterpret_cast<const void*>(&mc_adjoint_kernel<2>)
             : local == 1 ? reinterpret_cast<const void*>(&mc_adjoint_kernel<1>)
                          : reinterpret_cast<const void*>(&mc_adjoint_kernel<0>);
    else
        return local == 5 ? reinterpret_cast<const void*>(&mc_kernel<MODE, 5>)
             : local == 4 ? reinterpret_cast<const void*>(&mc_kernel<MODE, 4>)
             : local == 3 ? reinterpret_cast<const void*>(&mc_kernel<MODE, 3>)
             : local == 2 ? reinterpret_cast<const void*>(&mc_kernel<MODE, 2>)
             : local == 1 ? reinterpret_cast<const void*>(&mc_kernel<MODE, 1>)
                          : reinterpret_cast<const void*>(&mc_kernel<MODE, 0>);
}

const void* mc_func_for(int mode, int local, int block) {
    return mode == kModeForward ? mc_func<kModeForward>(local, block)
         : mode == kModeTrace ? mc_func<kModeTrace>(local, block) : mc_func<kModeBackward>(local, block);
}

// Does some job of the launch trace photons in volume v?
bool batch_uses(const Batch& B, int v) {
    for (int k = 0; k < B.n_jobs; ++k)
        if (B.jobs[k].volume == v && B.jobs[k].n_photons > 0 && (B.only_volume < 0 || v == B.only_volume))
            return true;
    return false;
}

int run_batch(const Batch& B, void* ws, size_t ws_bytes, hipStream_t st) {
    int rc = check_batch(B);
    if (rc) return rc;
    const gdrr_physics* phys = B.phys;
    const bool need_maj = B.majorants == nullptr;
    const Layout L0 = carve(nullptr, B.vols, phys, B.srcs, B.n_srcs, B.n_jobs, B.n_vols,
                            tally_elems_of(B.jobs, B.n_jobs, B.srcs), need_maj);
    if (!ws || ws_bytes < L0.bytes)
        return fail(GDRR_EINVAL, "workspace too small: need " + std::to_string(L0.bytes) + " bytes");
    DevInfo dev;
    if ((rc = device_info(dev))) return rc;
    char* wsa = (char*)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    const Layout L = carve(wsa, B.vols, phys, B.srcs, B.n_srcs, B.n_jobs, B.n_vols, L0.tally_elems, need_maj);
    const bool has_extra = ws_bytes >= L.bytes + kExtraBytes;
    char* const extra = wsa + ((L.bytes + 255) & ~(size_t)255);
    const bool interp = (B.flags & GDRR_INTERP_DENSITY) != 0;

    // ---- host tables: jobs, chunk prefix, output offsets ----
    gdrr_tuning tune{};
    if (B.tune) tune = *B.tune;
    unsigned long long total_photons = 0;
    for (int k = 0; k < B.n_jobs; ++k)
        if (B.only_volume < 0 || B.jobs[k].volume == B.only_volume) total_photons += B.jobs[k].n_photons;
    bool local = false;
    for (int v = 0; v < B.n_vols; ++v) local |= B.vols[v].macro > 0;
    // the single-majorant tables are staged only if some traced volume tracks with them
    bool any_single = false;
    for (int v = 0; v < B.n_vols; ++v) any_single |= batch_uses(B, v) && B.vols[v].macro <= 0;
    const int n_maj = any_single ? B.n_vols : 0;
    const int n_mat = phys->n_mat;
    // Local majorants go to LDS (after the tables) while the records of all volumes that the
    // launch traces fit in kMacroLdsMax.  All-local launches (every traced volume has local
    // majorants) keep one word per cube in a grid padded with words that
    // end a walk (outside_stride), at most kPaddedLdsMax bytes (8192 cubes in a grid of one slab
    // take 105 KB); where tables leave no room for it, or an axis has over 512 cubes, they take
    // the unpadded 8-byte records, or global memory.  A cube's bound is the same number everywhere.
    int macro_lds[GDRR_MAX_VOLUMES];
    int macro_lds_n = 0;
    int local_kind = 0;
    const size_t one_wave = (size_t)(tune.block ? tune.block : 256) / 64;      // least slots of a launch
    const auto fits = [&](int kind, size_t records) {
        return slots_offset_bytes(table_floats2(n_mat, phys->n_e, n_maj) * 8 + records * lds_record_bytes(kind)) +
               one_wave * kMinSlots * slot_bytes(kind) <= dev.lds_max;
    };
    if (local) {
        size_t n = 0, padded = 0;
        bool small_grids = true;
        for (int v = 0; v < B.n_vols; ++v)
            if (B.vols[v].macro > 0 && batch_uses(B, v)) {
                const gdrr_volume& V = B.vols[v];
                const int cx = cubes(V.nx, V.macro), cy = cubes(V.ny, V.macro), cz = cubes(V.nz, V.macro);
                n += (size_t)cx * cy * cz;
                small_grids &= cx <= 512 && cy <= 512 && cz <= 512;
                padded += (size_t)outside_stride(cx, cy) * ((size_t)cz + 2);
            }
        if (n > 0 && !any_single && small_grids && n * lds_record_bytes(3) <= kMacroLdsMax &&
            padded * lds_record_bytes(3) <= kPaddedLdsMax && fits(3, padded))
            local_kind = interp ? 3 : 4;
        else if (n > 0 && n * lds_record_bytes(2) <= kMacroLdsMax && fits(2, n))
            local_kind = 2;
        else
            local_kind = 1;
    }
    // Screening of a single majorant: cubes as small as kScreenCubes in the launch allow (2 voxels at
    // least), their records after everything else in the workspace; without room there or in LDS,
    // launches run unscreened.
    int screen_cube[GDRR_MAX_VOLUMES] = {};
    uint2* screen_rec[GDRR_MAX_VOLUMES] = {};
    if (!local && any_single && B.mode != kModeBackward) {
        int used = 0;
        for (int v = 0; v < B.n_vols; ++v) used += batch_uses(B, v);
        size_t n = 0;
        for (int v = 0; v < B.n_vols; ++v)
            if (batch_uses(B, v)) {
                screen_cube[v] = screen_cube_of(B.vols[v], kScreenCubes / used);
                screen_rec[v] = (uint2*)(extra + kDispBytes) + n;
                n += cubes_of(B.vols[v], screen_cube[v]);
            }
        // (and where the cubes' records would leave a caller's small workgroups fewer than 16 wavefronts
        // per compute unit, and fewer than without: 256 lanes, waits 32, 6e6 photons of 64^3 voxels of 9
        // materials 3.08 ms with 12 wavefronts screened, 2.55 with 20 unscreened; of 4 materials 2.14 with 16, 2.37)
        const size_t threads = tune.block ? tune.block : B.mode == kModeTrace ? 256 : 1024;
        const auto waves = [&](int kind, size_t records) {
            const size_t bytes = slots_offset_bytes(table_floats2(n_mat, phys->n_e, n_maj) * 8 + records * lds_record_bytes(kind)) +
                                 threads / 64 * kMinSlots * slot_bytes(kind);
            return bytes > dev.lds_max ? 0 : dev.lds_max / ((bytes + kLdsGranule - 1) / kLdsGranule * kLdsGranule) * (threads / 64);
        };
        if (has_extra && fits(5, n) && (waves(5, n) >= 16 || waves(5, n) >= waves(0, 0))) local_kind = 5;
    }
    for (int v = 0; v < GDRR_MAX_VOLUMES; ++v) {
        macro_lds[v] = -1;
        if (local_kind == 5 && v < B.n_vols && screen_cube[v]) {
            macro_lds[v] = macro_lds_n;
            macro_lds_n += (int)cubes_of(B.vols[v], screen_cube[v]);
        }
        if (v >= B.n_vols || local_kind < 2 || B.vols[v].macro <= 0 || !batch_uses(B, v)) continue;
        const gdrr_volume& V = B.vols[v];
        const int cx = cubes(V.nx, V.macro), cy = cubes(V.ny, V.macro), cz = cubes(V.nz, V.macro);
        // (all-local: the offset of cube (0, 0, 0), after the padding below the grid)
        macro_lds[v] = macro_lds_n + (local_kind >= 3 ? outside_stride(cx, cy) : 0);
        macro_lds_n += local_kind >= 3 ? outside_stride(cx, cy) * (cz + 2) : cx * cy * cz;
    }
    // Default shape.  All-local and screened launches are bound by VALU issue: they gain from early
    // refills and from 1024-thread workgroups, two per compute unit, which share the tables and cube
    // records and so keep 8 wavefronts per SIMD.  All-local (2e7 photons of a 256x256x160
    // phantom): 2.50 ms against 4.46 at 256 threads, waits 32.  Screened (1e7 photons), ms at 256/32/32,
    // 512/16/16, 1024/16/16, 1024/8/12: 64x64x64 3.43 2.16 1.93 1.86, 128x128x96 3.76 2.13 2.00 1.91,
    // 256x256x160 3.76 2.31 1.92 1.86, 512x512x256 3.96 2.41 2.03 1.98; 1e5 photons 217 to 251 us at
    // 256/32/32, 205 to 231 at 1024/8/12.  Launches that take neither path wait on their gathers,
    // where late refills do best (512x512x256, unscreened: 3.21 ms against 3.50).
    // (The trace kernel runs 7 wavefronts per SIMD, which 1024-thread workgroups would cut to 4.)
    const bool wide = local_kind >= 3 && B.mode != kModeTrace;
    int block = tune.block ? tune.block : (wide ? 1024 : 256);
    // Rows for the material sets of cubes: all-local and screened launches, at most 8 materials (screened
    // ones have a row of all materials for the sets beyond, and for any with more materials).
    const int sets = local_kind >= 3 && n_mat <= 8 ? std::min((1 << n_mat) - 1 - n_mat, (int)kNoRow - n_mat)   // of two or more
                                                   : local_kind == 5;
    const auto plan_for = [&](int threads, LdsPlan& plan) -> int {
        int most = 0;
        GDRR_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&most, mc_func_for(B.mode, local_kind, threads), threads, 0));
        plan = plan_lds(table_floats2(n_mat, phys->n_e, n_maj) * 8 + (size_t)macro_lds_n * lds_record_bytes(local_kind),
                        (size_t)phys->n_e * 8, sets, local_kind == 5, threads / 64, slot_bytes(local_kind), dev.lds_max, std::max(most, 1),
                        tune.blocks_per_cu);
        return GDRR_OK;
    };
    LdsPlan plan{};
    // All-local adjoint: the widest of the workgroups that keep 6 wavefronts per SIMD (1.8e8 histories of 256x256x160 voxels: 768 lanes 25.6 ms, 512 25.5, 1024 of 64 VGPRs with spills 28.4);
    // 1024 only where the LDS leaves the others fewer lanes than that.
    if (wide && !tune.block && B.mode == kModeBackward) {
        plan = {};
        int lanes = 0;
        for (const int b : {768, 512, 1024}) {
            LdsPlan p{};
            if ((rc = plan_for(b, p))) return rc;
            if (std::min(p.per_cu * b, 1536) > lanes) {
                lanes = std::min(p.per_cu * b, 1536);
                plan = p;
                block = b;
            }
        }
    } else if ((rc = plan_for(block, plan))) {
        return rc;
    }
    // (the library's own workgroups shrink where they do not fit)
    while (!tune.block && block > 256 && plan.per_cu == 0) {
        block /= 2;
        if ((rc = plan_for(block, plan))) return rc;
    }
    const size_t lds = plan.bytes;
    if (lds > dev.lds_max) return fail(GDRR_ENOTSUP, "tables exceed the LDS of a workgroup");
    const int mask_rows = plan.rows, per_cu = tune.blocks_per_cu ? tune.blocks_per_cu : plan.per_cu;
    const unsigned grid = (unsigned)(dev.cus * per_cu);
    const unsigned long long waves = (unsigned long long)grid * (block / 64);
    int chunk = tune.chunk;
    if (!chunk) {
        unsigned long long c = total_photons / (waves * 8ull);
        c = std::max<unsigned long long>(64, std::min<unsigned long long>(4096, c));
        chunk = (int)(c / 64 * 64);
    }
    const int defer = tune.defer ? tune.defer : (wide ? 8 : 32);
    const int cdefer = tune.coll_defer ? tune.coll_defer : (wide && !tune.defer ? 12 : defer);

    const size_t n_jobs = (size_t)B.n_jobs;
    const size_t job_bytes = sizeof(unsigned long long) * (n_jobs + 1);       // of the chunk prefix
    std::vector<unsigned long long> prefix(n_jobs + 1);
    std::vector<DJob> dj(n_jobs);
    std::vector<long long> out_off(n_jobs);
    unsigned long long chunks = 0;
    size_t toff = 0;
    for (size_t k = 0; k < n_jobs; ++k) {
        const gdrr_job& J = B.jobs[k];
        const gdrr_geometry& g = J.geom;
        DJob d = djob_of(J);
        const bool run = B.only_volume < 0 || J.volume == B.only_volume;
        const unsigned long long n = run ? J.n_photons : 0ull;
        d.n_lo = (uint32_t)J.n_photons;
        d.n_hi = (uint32_t)(J.n_photons >> 32);
        d.first = J.first_photon;
        d.index = (uint32_t)k;
        d.tally_off = (long long)toff;
        d.adj_off = (long long)(2 * (size_t)g.nu * g.nv * k);
        toff += 4 * (size_t)g.nu * g.nv;
        dj[k] = d;
        out_off[k] = J.tally_offset;
        prefix[k] = chunks;
        chunks += (n + (unsigned long long)chunk - 1) / (unsigned long long)chunk;
    }
    prefix[n_jobs] = chunks;

    // The volume order of the dispenser: jobs are taken in array order; a
    // wavefront drains before it changes phantom, so callers group jobs by volume.
    std::vector<Launch> ls;
    TableImage tables(L.chunk_prefix, L.out_off + n_jobs, g_staging);
    tables.put(L.chunk_prefix, prefix.data(), job_bytes);
    tables.put(L.jobs, dj.data(), sizeof(DJob) * n_jobs);
    tables.put(L.out_off, out_off.data(), sizeof(long long) * n_jobs);
    if (B.tables_by_kernel && tables.host.size() > sizeof(SetupParams::image))
        return fail(GDRR_EINVAL, "internal: the tables do not fit a kernel's arguments");

    unsigned int* status = (unsigned int*)(L.counter + 1);    // input-error bits of this call
    const bool resume = B.mode == kModeForward && (B.flags & GDRR_RESUME);
    // ---- clear counters, tallies (unless resuming), the gradient and the majorant scratch ----
    {
        std::vector<FillParams> fills = {{L.counter, 8}};
        if (has_extra) fills.push_back({(unsigned long long*)extra, (long long)(kDispBytes / 8)});
        if (!resume) fills.push_back({L.tally, (long long)L.tally_elems});
        if (B.mode == kModeBackward && !(B.flags & GDRR_ACCUMULATE)) {
            const gdrr_volume& V = B.vols[B.only_volume];
            fills.push_back({(unsigned long long*)B.grad, (long long)V.nx * V.ny * V.nz});       // (the bits of 0.0)
        }
        if (need_maj) {
            fills.push_back({(unsigned long long*)L.rho_max, (long long)B.n_vols * 128});   // 256 u32 per volume
            fills.push_back({(unsigned long long*)L.present, (long long)B.n_vols * 128});
        }
        if ((rc = add_setup(ls, fills, tables, !B.use_graph, st))) return rc;
    }
    // ---- cell records of every volume that has photons; the maxima for the majorants, if they
    // are not the caller's and any volume is tracked by one (all volumes are checked then) ----
    for (int v = 0; v < B.n_vols; ++v) {
        const bool cells = batch_uses(B, v);
        if (!cells && !need_maj) continue;
        const gdrr_volume& V = B.vols[v];
        ls.push_back(voxels_launch(V, phys->n_mat, interp, dev.cus, cells ? L.cells[v] : nullptr, need_maj && (n_maj || !cells),
                                   L.rho_max + 256 * v, L.present + 256 * v, status));
        if (need_maj && n_maj) {
            MajFinParams fp{L.rho_max + 256 * v, L.present + 256 * v, phys->mu_mass, phys->n_mat, phys->n_e,
                            1.0 + (double)(1.0f / 1048576.0f), L.majorants + (size_t)v * (phys->n_e - 1),
                            status};
            ls.push_back(make_launch((const void*)&majorant_kernel, dim3((phys->n_e + 254) / 256), dim3(256), 0, fp));
        }
        if (!cells) continue;
        if (local_kind == 5) {
            const int m = screen_cube[v];
            MacroParams mp{V.density, V.material, V.nx, V.ny, V.nz, m, cubes(V.nx, m), cubes(V.ny, m), cubes(V.nz, m),
                           phys->n_mat, kScreenScale, 0.0f, screen_rec[v]};
            ls.push_back(make_launch((const void*)&macro_kernel, dim3((unsigned)cubes_of(V, m)), dim3(macro_block(m)), 0, mp));
        }
        if (L.macro[v]) {
            MacroParams mp{V.density, V.material, V.nx, V.ny, V.nz, V.macro, cubes(V.nx, V.macro),
                           cubes(V.ny, V.macro), cubes(V.nz, V.macro), phys->n_mat,
                           1.0 + (double)V.macro_margin, V.macro_rho_min, L.macro[v]};
            const size_t nm = (size_t)mp.mnx * mp.mny * mp.mnz;
            // one workgroup per cube
            ls.push_back(make_launch((const void*)&macro_kernel,
                                     dim3((unsigned)std::max<size_t>(1, std::min<size_t>((size_t)dev.cus * 16, nm))),
                                     dim3(macro_block(V.macro)), 0, mp));
        }
    }
    // ---- sources: CDFs and guide tables ----
    for (int s = 0; s < B.n_srcs; ++s) {
        const gdrr_source& S = B.srcs[s];
        const SrcArea& A = L.src[s];
        const int rows = spec_rows(S);
        const CdfTable flu{S.fluence, S.fu * S.fv, 1, A.flu_cdf, A.flu_guide, (int)A.flu_k};
        const int row_blocks = std::min(rows, kRowBlocks);
        const SrcPrepParams sp{{{S.spec_prob, S.n_spec, rows, A.spec_cdf, A.spec_guide, (int)A.spec_k}, flu}, row_blocks, status};
        const bool is_long = flu.n > kLongTable;
        const unsigned blocks = is_long ? kSegs / kSegBlock : 1;
        ls.push_back(make_launch((const void*)&cdf_kernel, dim3(row_blocks + blocks), dim3(kSegs), 0, sp));
        if (!is_long) continue;
        ls.push_back(make_launch((const void*)&long_cdf_kernel, dim3(blocks), dim3(kSegs), 0, LongCdfParams{flu, status}));
        ls.push_back(make_launch((const void*)&guide_kernel, dim3((A.flu_k + 255) / 256), dim3(256), 0, flu));
    }
    // ---- the persistent transport kernel ----
    KParams kp{};
    for (int v = 0; v < B.n_vols; ++v) {
        const gdrr_volume& V = B.vols[v];
        DVolume& d = kp.vol[v];
        d.density = V.density;
        d.material = V.material;
        d.cells = L.cells[v];
        d.cx = V.nx + 1;
        d.cxy = (V.nx + 1) * (V.ny + 1);
        d.nx = V.nx; d.ny = V.ny; d.nz = V.nz; d.nxy = V.nx * V.ny;
        d.lox = (float)(-0.5 * V.nx * V.dx_mm); d.hix = -d.lox;
        d.loy = (float)(-0.5 * V.ny * V.dy_mm); d.hiy = -d.loy;
        d.loz = (float)(-0.5 * V.nz * V.dz_mm); d.hiz = -d.loz;
        d.idx = (float)(1.0 / V.dx_mm); d.idy = (float)(1.0 / V.dy_mm); d.idz = (float)(1.0 / V.dz_mm);
        d.lds_majorant = n_maj ? v * (phys->n_e - 1) : -1;
        d.macro = L.macro[v];
        const int mc = local_kind == 5 ? screen_cube[v] : V.macro;
        if (local_kind == 5 && mc > 0) d.screen = screen_rec[v];
        if (mc > 0) {
            d.mnx = cubes(V.nx, mc); d.mny = cubes(V.ny, mc); d.mnz = cubes(V.nz, mc);
            d.mcube = mc;
            d.mlx = (float)(d.mnx - 1); d.mly = (float)(d.mny - 1); d.mlz = (float)(d.mnz - 1);
            d.msy = d.mnx + 1; d.msz = outside_stride(d.mnx, d.mny);
            d.mex = (float)((double)mc * V.dx_mm);
            d.mey = (float)((double)mc * V.dy_mm);
            d.mez = (float)((double)mc * V.dz_mm);
            d.imx = (float)(1.0 / ((double)mc * V.dx_mm));
            d.imy = (float)(1.0 / ((double)mc * V.dy_mm));
            d.imz = (float)(1.0 / ((double)mc * V.dz_mm));
        }
    }
    for (int s = 0; s < B.n_srcs; ++s) {
        DSource& d = kp.src[s];
        d.spec_e = B.srcs[s].spec_e_kev;
        d.spec_cdf = L.src[s].spec_cdf;
        d.spec_guide = L.src[s].spec_guide;
        d.flu_cdf = L.src[s].flu_cdf;
        d.flu_guide = L.src[s].flu_guide;
        d.n_spec = B.srcs[s].n_spec;
        d.spec_rows = spec_rows(B.srcs[s]);
        d.spec_k = (int)L.src[s].spec_k;
        d.npix = B.srcs[s].fu * B.srcs[s].fv;
        d.flu_k = (int)L.src[s].flu_k;
    }
    kp.jobs = L.jobs;
    kp.chunk_prefix = L.chunk_prefix;
    kp.counter = has_extra ? (unsigned long long*)extra : L.counter;
    kp.n_disp = has_extra ? kDispensers : 1;
    kp.tally = L.tally;
    kp.mu_mass = phys->mu_mass;
    kp.response = phys->response;
    kp.majorants = need_maj ? L.majorants : B.majorants;
    kp.total_chunks = chunks;
    kp.n_jobs = B.n_jobs;
    kp.n_vols = B.n_vols;
    kp.n_maj = n_maj;
    kp.n_mat = phys->n_mat;
    kp.tot_rows = phys->n_mat + mask_rows;
    kp.mask_rows = mask_rows;
    kp.n_e = phys->n_e;
    kp.e0 = phys->e0_kev;
    kp.inv_de = (float)(1.0 / phys->de_kev);
    kp.e_max = (float)(phys->e0_kev + (double)phys->de_kev * (phys->n_e - 1));
    kp.e_cut = phys->e_cut_kev;
    kp.x0 = phys->rayleigh_x0_invA;
    kp.mhx0 = -0.5f * phys->rayleigh_x0_invA;
    kp.k0 = (uint32_t)B.seed;
    kp.k1 = (uint32_t)(B.seed >> 32);
    kp.flags = B.flags;
    kp.chunk = chunk;
    kp.defer = defer;
    kp.cdefer = cdefer;
    kp.t_cls = B.t_cls; kp.t_pixel = B.t_pixel; kp.t_e = B.t_e;
    kp.t_steps = B.t_steps; kp.t_nc = B.t_nc; kp.t_nr = B.t_nr;
    kp.adj = B.adj;
    kp.grad = B.grad;
    for (int v = 0; v < kMaxVol; ++v) kp.macro_lds[v] = v < GDRR_MAX_VOLUMES ? macro_lds[v] : -1;
    kp.macro_lds_n = macro_lds_n;
    kp.n_slots = plan.slots;
    const void* mf = mc_func_for(B.mode, local_kind, block);
    int timed = -1;
    if (chunks > 0) {
        timed = (int)ls.size();
        ls.push_back(make_launch(mf, dim3(grid), dim3(block), lds, kp));
    }
    // ---- finalize ----
    if (B.mode == kModeForward) {
        int maxpix = 1;
        for (int k = 0; k < B.n_jobs; ++k) maxpix = std::max(maxpix, B.jobs[k].geom.nu * B.jobs[k].geom.nv);
        FinParams fp{L.jobs, B.n_jobs, L.tally, B.out, L.out_off, B.flags & (GDRR_TALLY_SUMSQ | GDRR_ACCUMULATE | GDRR_RESUME)};
        ls.push_back(make_launch((const void*)&finalize_kernel,
                                 dim3((unsigned)std::min(1024, (4 * maxpix + 255) / 256), (unsigned)B.n_jobs), dim3(256), 0, fp));
    }
    TimeEvents* ev = nullptr;
    if (!B.tables_by_kernel) {
        std::lock_guard<std::mutex> lk(g_time_mu);
        if (g_timing && timed >= 0 && (rc = timing_events(&ev))) return rc;
    }
    if (!ev) timed = -1;
    return B.use_graph ? run_graph(ls, st, timed, ev) : run_direct(ls, st, timed, ev);
}

size_t batch_bytes(const gdrr_volume* vols, int n_vols, const gdrr_physics* phys, const gdrr_source* srcs,
                   int n_srcs, const gdrr_job* jobs, int n_jobs, bool need_maj) {
    if (!vols || !phys || !srcs || !jobs || n_srcs < 1 || n_srcs > GDRR_MAX_SOURCES || n_jobs < 1 || n_vols < 1 ||
        n_vols > GDRR_MAX_VOLUMES)
        return 0;
    for (int v = 0; v < n_vols; ++v)
        if (vols[v].nx < 1 || vols[v].ny < 1 || vols[v].nz < 1) return 0;
    for (int s = 0; s < n_srcs; ++s)
        if (srcs[s].n_spec < 1 || spec_rows(srcs[s]) < 0) return 0;
    return carve(nullptr, vols, phys, srcs, n_srcs, n_jobs, n_vols, tally_elems_of(jobs, n_jobs, srcs), need_maj).bytes +
           256;
}

// The bytes that the queries return.
size_t batch_bytes_all(const gdrr_volume* vols, int n_vols, const gdrr_physics* phys, const gdrr_source* srcs,
                       int n_srcs, const gdrr_job* jobs, int n_jobs) {
    const size_t bytes = batch_bytes(vols, n_vols, phys, srcs, n_srcs, jobs, n_jobs, true);
    return bytes ? bytes + kExtraBytes : 0;
}

// --------------------------------------------------------------------------
// Ray-tracing primary (Eq. 1): workspace layout and launch.
// --------------------------------------------------------------------------
struct RtLayout {
    unsigned long long* head;            // [8] status block (word 1: input-error bits)
    DJob* jobs;                          // [n_jobs]
    int* unit_job;                       // [max units]
    unsigned int* unit_first;
    unsigned int* unit_pref;
    long long* out_off;                  // [n_jobs]
    float* coef[GDRR_MAX_SOURCES];       // [rows][n_spec]
    float* tab[GDRR_MAX_SOURCES];        // [n_spec][n_mat]
    double* inv_wsum[GDRR_MAX_SOURCES];  // [1]
    Plane* planes[GDRR_MAX_VOLUMES];     // volumes that some job uses
    uint16_t* codes[GDRR_MAX_VOLUMES];   // (their corners' materials)
    size_t bytes;
};

bool volume_used(const gdrr_job* jobs, int n_jobs, int v) {
    for (int k = 0; k < n_jobs; ++k)
        if (jobs[k].volume == v) return true;
    return false;
}


unsigned long long rt_tiles(const gdrr_geometry& g) {
    return (unsigned long long)((g.nu + 15) / 16) * (unsigned long long)((g.nv + 15) / 16);
}

// Work units: pieces of one tile row of one job, `run` tiles long (whole
// rows once there are enough of them to fill every XCD several times).
unsigned long long rt_run_length(const gdrr_job* jobs, int n_jobs) {
    unsigned long long total = 0, widest = 1;
    for (int k = 0; k < n_jobs; ++k) {
        total += rt_tiles(jobs[k].geom);
        widest = std::max(widest, (unsigned long long)((jobs[k].geom.nu + 15) / 16));
    }
    return std::min(widest, std::max<unsigned long long>(4, total / (8ull * kXcds)));
}

template <bool SMALL>
const void* rt_kernel(int lanes, int n_mat) {
    return lanes == 4    ? (const void*)&raytrace_kernel<4, false, SMALL>
           : lanes == 16 ? (const void*)&raytrace_kernel<16, false, SMALL>
           : n_mat > kPlaneLook ? (const void*)&raytrace_kernel<1, true, SMALL>
                                : (const void*)&raytrace_kernel<1, false, SMALL>;
}

unsigned long long rt_row_units(const gdrr_geometry& g, unsigned long long run) {
    return (unsigned long long)((g.nv + 15) / 16) * (((unsigned long long)((g.nu + 15) / 16) + run - 1) / run);
}

size_t rt_max_units(const gdrr_job* jobs, int n_jobs) {
    const unsigned long long run = rt_run_length(jobs, n_jobs);
    size_t u = 0;
    for (int k = 0; k < n_jobs; ++k) u += (size_t)rt_row_units(jobs[k].geom, run);
    return u;
}

RtLayout rt_carve(void* ws, const gdrr_volume* vols, int n_vols, const gdrr_physics* phys, const gdrr_source* srcs,
                  int n_srcs, const gdrr_job* jobs, int n_jobs) {
    Carver c(ws);
    RtLayout L{};
    L.head = c.take<unsigned long long>(8);
    L.jobs = c.take<DJob>((size_t)n_jobs);
    const size_t units = rt_max_units(jobs, n_jobs);
    L.unit_job = c.take<int>(units);
    L.unit_first = c.take<unsigned int>(units);
    L.unit_pref = c.take<unsigned int>(units);
    L.out_off = c.take<long long>((size_t)n_jobs);
    for (int s = 0; s < n_srcs; ++s) {
        L.coef[s] = c.take<float>((size_t)spec_rows(srcs[s]) * srcs[s].n_spec);
        L.tab[s] = c.take<float>((size_t)srcs[s].n_spec * phys->n_mat);
        L.inv_wsum[s] = c.take<double>(1);
    }
    for (int v = 0; v < n_vols; ++v)
        if (volume_used(jobs, n_jobs, v)) {
            // 18 bytes a plane of a column in the room of records of whole cells, 32 bytes each and
            // one fewer per column: the size that callers know
            const size_t n = plane_count(vols[v].nx, vols[v].ny, vols[v].nz);
            L.planes[v] = (Plane*)c.take<CellRec>(cell_count(vols[v]));
            L.codes[v] = L.planes[v] ? (uint16_t*)(L.planes[v] + n) : nullptr;
        }
    L.bytes = c.off + 256;
    return L;
}

// Lanes per ray for a number of 16 x 16 tiles.  Measured (us, 1 / 4 / 16 lanes, 256x256x160 voxels): 192 tiles
// 329 / 138 / 204, 384 tiles 340 / 188 / 365, 576 tiles 393 / 319 / 582, 768 tiles 408 / 510 / 1078 (images of
// 256x192); 12 tiles 432 / 156 / 91, 48 tiles 460 / 165 / 111, 96 tiles 449 / 169 / 132 (of 64x48): the lines
// could lie up to half as far again to the right.
int rt_lanes(unsigned long long tiles) { return tiles <= 64 ? 16 : tiles <= 512 ? 4 : 1; }

constexpr unsigned kRtMaxTiles = (1u << 24) - 1024u;    // grid * block stays below 2^32 work-items

int check_rt(const gdrr_volume* vols, int n_vols, const gdrr_physics* phys, const gdrr_source* srcs, int n_srcs,
             const gdrr_job* jobs, int n_jobs, uint32_t flags) {
    if (n_vols < 1 || n_vols > GDRR_MAX_VOLUMES) return fail(GDRR_EINVAL, "n_vols must be in [1, 8]");
    if (n_srcs < 1 || n_srcs > GDRR_MAX_SOURCES) return fail(GDRR_EINVAL, "n_srcs must be in [1, 8]");
    if (n_jobs < 1 || n_jobs > (1 << 20)) return fail(GDRR_EINVAL, "n_jobs must be in [1, 2^20]");
    if (!vols || !srcs || !jobs) return fail(GDRR_EINVAL, "NULL array argument");
    if (flags & ~(GDRR_INTERP_DENSITY | GDRR_ACCUMULATE))
        return fail(GDRR_EINVAL, "gdrr_primary takes only GDRR_INTERP_DENSITY and GDRR_ACCUMULATE");
    int rc;
    if ((rc = check_physics(phys))) return rc;
    for (int v = 0; v < n_vols; ++v)
        if ((rc = check_volume(&vols[v]))) return rc;
    for (int s = 0; s < n_srcs; ++s)
        if ((rc = check_source(&srcs[s]))) return rc;
    for (int k = 0; k < n_jobs; ++k) {
        const gdrr_job& J = jobs[k];
        if (J.volume < 0 || J.volume >= n_vols) return fail(GDRR_EINVAL, "job volume index out of range");
        if (J.source < 0 || J.source >= n_srcs) return fail(GDRR_EINVAL, "job source index out of range");
        if (J.tally_offset < 0) return fail(GDRR_EINVAL, "negative output offset");
        if ((rc = check_geometry(&J.geom, &vols[J.volume], &srcs[J.source]))) return rc;
    }
    return GDRR_OK;
}

int run_primary(const gdrr_volume* vols, int n_vols, const gdrr_physics* phys, const gdrr_source* srcs, int n_srcs,
                const gdrr_job* jobs, int n_jobs, float step_mm, uint32_t flags, double* out, void* ws,
                size_t ws_bytes, hipStream_t st) {
    int rc = check_rt(vols, n_vols, phys, srcs, n_srcs, jobs, n_jobs, flags);
    if (rc) return rc;
    if (!out) return fail(GDRR_EINVAL, "out is NULL");
    if (!std::isfinite(step_mm)) return fail(GDRR_EINVAL, "step_mm must be finite");
    const RtLayout L0 = rt_carve(nullptr, vols, n_vols, phys, srcs, n_srcs, jobs, n_jobs);
    if (!ws || ws_bytes < L0.bytes)
        return fail(GDRR_EINVAL, "workspace too small: need " + std::to_string(L0.bytes) + " bytes");
    RtParams rp{};
    for (int v = 0; v < n_vols; ++v) {
        const gdrr_volume& V = vols[v];
        const double edge = std::min(V.dx_mm, std::min(V.dy_mm, V.dz_mm));
        const double dl = step_mm > 0.0f ? (double)step_mm : 0.5 * edge;
        const double diag = std::sqrt((double)V.nx * V.dx_mm * V.nx * V.dx_mm + (double)V.ny * V.dy_mm * V.ny * V.dy_mm +
                                      (double)V.nz * V.dz_mm * V.nz * V.dz_mm);
        if (volume_used(jobs, n_jobs, v) && diag / dl > (double)(1 << 20))
            return fail(GDRR_EINVAL, "step_mm too small: more than 2^20 intervals across a phantom");
        rp.dl[v] = (float)dl;
    }
    const size_t lds = (size_t)phys->n_mat * kRtBlock * sizeof(float);
    DevInfo dev;
    if ((rc = device_info(dev))) return rc;
    if (lds > dev.lds_max) return fail(GDRR_ENOTSUP, "per-material accumulators exceed the LDS of a workgroup");
    char* wsa = (char*)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    const RtLayout L = rt_carve(wsa, vols, n_vols, phys, srcs, n_srcs, jobs, n_jobs);
    const bool interp = (flags & GDRR_INTERP_DENSITY) != 0;

    const size_t nj = (size_t)n_jobs;
    std::vector<DJob> dj(nj);
    std::vector<long long> off(nj);
    unsigned long long tiles = 0;
    for (size_t k = 0; k < nj; ++k) {
        dj[k] = djob_of(jobs[k]);
        dj[k].index = (uint32_t)k;
        off[k] = jobs[k].tally_offset;
        tiles += rt_tiles(jobs[k].geom);
        if (tiles > kRtMaxTiles) return fail(GDRR_EINVAL, "too many pixels in one call (2^32 lanes)");
    }
    const int lanes = rt_lanes(tiles);
    // Units in row-band order: for each phantom, tile row by tile row, that
    // row of every job on the phantom, dealt to the XCDs in turn.  All XCDs
    // then work through the same band of detector rows -- the same slab of
    // the phantom -- across all its projections at once, so the slab is read
    // from HBM about once and served from the last-level cache after that.
    const unsigned long long run = rt_run_length(jobs, n_jobs);
    std::vector<int> u_job[kXcds];
    std::vector<unsigned int> u_first[kXcds];
    std::vector<std::vector<int>> band[GDRR_MAX_VOLUMES];    // [volume][tile row] -> jobs in order
    for (size_t k = 0; k < nj; ++k) {
        std::vector<std::vector<int>>& b = band[jobs[k].volume];
        const size_t rows = (size_t)((jobs[k].geom.nv + 15) / 16);
        if (b.size() < rows) b.resize(rows);
        for (size_t r = 0; r < rows; ++r) b[r].push_back((int)k);
    }
    int deal = 0;
    for (int v = 0; v < n_vols; ++v)
        for (size_t r = 0; r < band[v].size(); ++r)
            for (const int k : band[v][r]) {
                const unsigned long long tu = (unsigned long long)((jobs[k].geom.nu + 15) / 16);
                for (unsigned long long c = 0; c < tu; c += run) {
                    u_job[deal].push_back(k);
                    u_first[deal].push_back((unsigned int)(r * tu + c));
                    deal = (deal + 1) % kXcds;
                }
            }
    std::vector<int> ujob;
    std::vector<unsigned int> ufirst, upref;
    unsigned int most = 0;
    for (int x = 0; x < kXcds; ++x) {
        rp.xcd_start[x] = (unsigned int)ujob.size();
        unsigned int acc = 0;
        for (size_t i = 0; i < u_job[x].size(); ++i) {
            const int k = u_job[x][i];
            ujob.push_back(k);
            ufirst.push_back(u_first[x][i]);
            upref.push_back(acc);
            const unsigned long long tu = (unsigned long long)((jobs[k].geom.nu + 15) / 16);
            acc += (unsigned int)std::min<unsigned long long>(run, tu - u_first[x][i] % tu);
        }
        rp.xcd_tiles[x] = acc;
        most = std::max(most, acc);
    }
    rp.xcd_start[kXcds] = (unsigned int)ujob.size();
    const size_t nu_ = ujob.size();
    const size_t b_u = sizeof(unsigned int) * nu_;
    TableImage tables(L.jobs, L.out_off + nj, g_staging);
    tables.put(L.jobs, dj.data(), sizeof(DJob) * nj);
    tables.put(L.unit_job, ujob.data(), b_u);
    tables.put(L.unit_first, ufirst.data(), b_u);
    tables.put(L.unit_pref, upref.data(), b_u);
    tables.put(L.out_off, off.data(), sizeof(long long) * nj);

    std::vector<Launch> ls;
    unsigned int* status = (unsigned int*)(L.head + 1);
    if ((rc = add_setup(ls, {{L.head, 8}}, tables, true, st))) return rc;
    bool small = true;                         // every index and stride of the plane records below 2^24
    for (int v = 0; v < n_vols; ++v) {
        const gdrr_volume& V = vols[v];
        small = small && std::max(std::max((long long)V.nx, (long long)V.ny), (long long)(V.nx + 1) * (V.nz + 2)) < (1ll << 24) - 1;
        DVolume& d = rp.vol[v];
        d.density = V.density;
        d.material = V.material;
        rp.planes[v] = interp ? L.planes[v] : nullptr;
        rp.codes[v] = interp ? L.codes[v] : nullptr;
        d.cx = V.nx + 1;
        d.cxy = (V.nx + 1) * (V.ny + 1);
        d.nx = V.nx; d.ny = V.ny; d.nz = V.nz; d.nxy = V.nx * V.ny;
        d.lox = (float)(-0.5 * V.nx * V.dx_mm); d.hix = -d.lox;
        d.loy = (float)(-0.5 * V.ny * V.dy_mm); d.hiy = -d.loy;
        d.loz = (float)(-0.5 * V.nz * V.dz_mm); d.hiz = -d.loz;
        d.idx = (float)(1.0 / V.dx_mm); d.idy = (float)(1.0 / V.dy_mm); d.idz = (float)(1.0 / V.dz_mm);
        if (interp && L.planes[v]) {
            const int tx = (V.nx + 1 + kPlX - 1) / kPlX, tzs = (V.nz + 2 + kPlZ - 1) / kPlZ;
            const unsigned n = (unsigned)((size_t)tx * tzs * (V.ny + 1));     // (below 2^30)
            PlaneParams cp{V.density, V.material, V.nx, V.ny, V.nz, phys->n_mat, tx, tzs, (V.nz + 2 + tzs - 1) / tzs, n,
                           L.planes[v], L.codes[v], status};
            // (a launch has fewer than 2^32 lanes)
            ls.push_back(make_launch((const void*)&planes_kernel, dim3(std::min(n, 1u << 23)), dim3(256), 0, cp));
        } else if (volume_used(jobs, n_jobs, v)) {
            const long long nv = (long long)V.nx * V.ny * V.nz;
            VolCheckParams vc{V.density, V.material, nv, phys->n_mat, status};
            ls.push_back(make_launch((const void*)&volume_check_kernel,
                                     dim3((unsigned)std::max<long long>(1, std::min<long long>((long long)dev.cus * 8, (nv + 255) / 256))),
                                     dim3(256), 0, vc));
        }
    }
    for (int s = 0; s < n_srcs; ++s) {
        const gdrr_source& S = srcs[s];
        RtPrepParams pp{S.spec_e_kev, S.spec_prob, S.fluence, S.n_spec, S.fu * S.fv, spec_rows(S), phys->mu_mass, phys->response,
                        phys->n_mat, phys->n_e, (double)phys->e0_kev, (double)phys->de_kev, L.coef[s], L.tab[s],
                        L.inv_wsum[s], status};
        ls.push_back(make_launch((const void*)&raytrace_prep_kernel, dim3(std::min(spec_rows(S), kRowBlocks) + 1), dim3(kRtPrepBlock), 0, pp));
        rp.src[s] = RtSource{S.fluence, L.coef[s], L.tab[s], L.inv_wsum[s], S.n_spec, spec_rows(S)};
    }
    rp.jobs = L.jobs;
    rp.unit_job = L.unit_job;
    rp.unit_first = L.unit_first;
    rp.unit_pref = L.unit_pref;
    rp.out_off = L.out_off;
    rp.out = out;
    rp.n_mat = phys->n_mat;
    rp.interp = interp ? 1 : 0;
    rp.accumulate = (flags & GDRR_ACCUMULATE) ? 1 : 0;
    const unsigned long long grid = (unsigned long long)kXcds * most * lanes;
    if (grid * kRtBlock >= (1ull << 32)) return fail(GDRR_EINVAL, "too many pixels in one call (2^32 lanes)");
    const int timed = (int)ls.size();
    const void* const f = small ? rt_kernel<true>(lanes, phys->n_mat) : rt_kernel<false>(lanes, phys->n_mat);
    // Nearest voxel, one lane per ray: seven workgroups per compute unit (by their LDS), not the eight that
    // the registers allow.  Their lines of the voxel arrays are shared through L1 and L2, which eight
    // overflow (us with 7 and 8, 4 images of 512x384 or 16 of 256x192: 512x512x256 voxels seen along x 2297 2805,
    // 256x256x160 907 960 and 1126 1185, along y 719 689; 6 workgroups 2266, 964, 1228, 870).
    const size_t rt_lds = lanes == 1 && !interp ? std::max(lds, 18 * kLdsGranule) : lds / lanes;
    ls.push_back(make_launch(f, dim3((unsigned)grid), dim3(kRtBlock), rt_lds, rp));
    TimeEvents* ev = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_time_mu);
        if (g_timing && (rc = timing_events(&ev))) return rc;
    }
    return run_direct(ls, st, ev ? timed : -1, ev);
}

// --------------------------------------------------------------------------
// Denoising (Eq. 5) and noise assembly (Sec. 2.6).
// --------------------------------------------------------------------------
bool ranges_overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + b_bytes && b0 < a0 + a_bytes;
}

size_t dn_buffer_bytes(int n_img, int nv, int nu) {
    return ((size_t)n_img * nv * nu * sizeof(float) + 255) & ~(size_t)255;
}

// How a stack of images is denoised: tiles of 64 C columns by R rows per wavefront, or whole
// images in one workgroup each.
struct DnPlan {
    const void* kernel;
    int tiles_u, tiles_v, halo, waves, passes, sweeps;   // a pass takes up to `sweeps`
    double us;                                           // the estimate that it was chosen by
};

// The plan is the one that this estimate finds cheapest: a pass takes 2 us and 3e-4 us per
// pixel that a CU loads and stores, a sweep 0.25 us (barrier and LDS round trip) and 7.5e-5 us
// per pixel of a CU's regions, halos included.  Fitted to 1 to 60 images of 512 x 384 in each
// configuration at halos of 8, 16 and 24; it decides between them as measured: one such image,
// 256 sweeps, halo 16: 182 us with regions of 64 x 56, 216 with 64 x 80, 364 with 128 x 96; 60
// images, 64 sweeps: 734, 707 and 575 at a halo of 8.
template <int C, int R>
void dn_try_tiles(int max_waves, int n_img, int nv, int nu, int iters, bool sel, int cus, DnPlan& best) {
    const int waves = std::min(max_waves, (nv + R - 1) / R), cols = 64 * C, rows = R * waves;
    const bool edge = nu < cols || nv < rows;
    for (const int k : {8, 12, 16, 24}) {
        if ((nu > cols && 2 * k >= cols) || (nv > rows && 2 * k >= rows)) break;
        const int du = cols - 2 * k, dv = rows - 2 * k;
        const int tu = nu <= cols ? 1 : (nu - 2 * k + du - 1) / du, tv = nv <= rows ? 1 : (nv - 2 * k + dv - 1) / dv;
        const bool one = tu == 1 && tv == 1;
        const int sweeps = one ? iters : k, passes = one ? 1 : std::max(1, (iters + k - 1) / k);
        const double px = std::ceil((double)n_img * tu * tv / cus) * cols * rows;
        const double us = passes * (2.0 + 3e-4 * px) + iters * (0.25 + 7.5e-5 * px);
        if (!(us < best.us)) continue;
        best = {edge ? (sel ? (const void*)&denoise_tile_kernel<C, R, 0, true, true> : (const void*)&denoise_tile_kernel<C, R, 0, true, false>)
                     : (sel ? (const void*)&denoise_tile_kernel<C, R, 0, false, true> : (const void*)&denoise_tile_kernel<C, R, 0, false, false>),
                tu, tv, k, waves, passes, sweeps, us};
    }
}

DnPlan dn_plan_tiles(int n_img, int nv, int nu, int iters, bool sel, int cus) {
    DnPlan p{};
    p.us = INFINITY;
    dn_try_tiles<1, 7>(8, n_img, nv, nu, iters, sel, cus, p);
    dn_try_tiles<1, 7>(16, n_img, nv, nu, iters, sel, cus, p);
    dn_try_tiles<1, 5>(16, n_img, nv, nu, iters, sel, cus, p);
    dn_try_tiles<2, 6>(16, n_img, nv, nu, iters, sel, cus, p);
    return p;
}

// Whole images go in rounds of one per CU, with no halo, but a lone one has a single CU; the
// same estimate, with the cost of a pixel measured for each width (a wavefront's share of the
// rows costs more moves in narrow ones, and fewer than 4 wavefronts leave SIMDs idle): 90
// images of 256 x 192, 100 sweeps, 428 us against 409 in tiles, 200 images, 30 sweeps, 155
// against 152; 360 images, 256 sweeps, 2140 against 3460 or more.
DnPlan dn_plan_images(int n_img, int nv, int nu, int iters, bool sel, int cus) {
    DnPlan p{};
    int rows = 0;
    if (nu == 256 && nv % 12 == 0) {
        rows = 12;
        p.kernel = sel ? (const void*)&denoise_tile_kernel<4, 12, 6, false, true> : (const void*)&denoise_tile_kernel<4, 12, 6, false, false>;
    } else if (nu == 128 && nv % 24 == 0) {
        rows = 24;
        p.kernel = sel ? (const void*)&denoise_tile_kernel<2, 24, 12, false, true> : (const void*)&denoise_tile_kernel<2, 24, 12, false, false>;
    } else if (nu == 64 && nv % 48 == 0) {
        rows = 48;
        p.kernel = sel ? (const void*)&denoise_tile_kernel<1, 48, 24, false, true> : (const void*)&denoise_tile_kernel<1, 48, 24, false, false>;
    }
    p.us = INFINITY;
    if (!rows || nv / rows > kDnMaxWaves) return p;
    const int waves = nv / rows;
    const double px = (double)nv * nu, per_px = (rows == 12 ? 8.4e-5 : rows == 24 ? 1.0e-4 : 1.1e-4) * std::max(1.0, 4.0 / waves);
    return {p.kernel, 1, 1, 0, waves, 1, iters, std::ceil((double)n_img / cus) * (2.0 + 3e-4 * px + iters * (0.25 + per_px * px))};
}

int run_denoise(const double* shat, long long stride, int n_img, int nv, int nu, float beta, float omega, int iters,
                float s_floor, double* out, void* ws, size_t ws_bytes, hipStream_t st) {
    if (!shat || !out) return fail(GDRR_EINVAL, "shat / out is NULL");
    if (n_img < 1 || nv < 1 || nu < 1) return fail(GDRR_EINVAL, "n_img, nv and nu must be >= 1");
    const long long npix = (long long)nv * nu;
    if (stride == 0) stride = npix;
    if (stride < npix) return fail(GDRR_EINVAL, "shat_stride must be 0 or >= nv * nu");
    if (!(beta > 0.0f) || !std::isfinite(beta)) return fail(GDRR_EINVAL, "beta must be finite and > 0");
    if (!(omega > 0.0f && omega < 2.0f)) return fail(GDRR_EINVAL, "omega must be in (0, 2)");
    if (iters < 0 || iters > (1 << 20)) return fail(GDRR_EINVAL, "iters must be in [0, 2^20]");
    if (!(s_floor > 0.0f) || !std::isfinite(s_floor)) return fail(GDRR_EINVAL, "s_floor must be finite and > 0");
    if ((long long)n_img * ((nu + 47) / 48) * ((nv + 63) / 64) >= (1ll << 31)) return fail(GDRR_EINVAL, "too many tiles in one call");
    const size_t in_bytes = ((size_t)(n_img - 1) * (size_t)stride + (size_t)npix) * sizeof(double);
    const size_t out_bytes = (size_t)n_img * (size_t)npix * sizeof(double);
    if (ranges_overlap(shat, in_bytes, out, out_bytes)) return fail(GDRR_EINVAL, "out must not overlap shat");
    const size_t buf = dn_buffer_bytes(n_img, nv, nu);
    if (!ws || ws_bytes < 2 * buf + 256) return fail(GDRR_EINVAL, "workspace too small: need " + std::to_string(2 * buf + 256) + " bytes");
    char* wsa = (char*)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    float* pp[2] = {(float*)wsa, (float*)(wsa + buf)};
    // Shat as float32, kept by the first pass for the others (counted by the query; without it
    // every pass reads the doubles)
    float* const hf = ws_bytes >= 3 * buf + 256 ? (float*)(wsa + 2 * buf) : nullptr;
    DevInfo dev;
    int rc;
    if ((rc = device_info(dev))) return rc;
    const bool sel = s_floor < 1.17549435e-38f;            // (the least normal number)
    DnPlan plan = dn_plan_tiles(n_img, nv, nu, iters, sel, dev.cus);
    if (const DnPlan whole = dn_plan_images(n_img, nv, nu, iters, sel, dev.cus); whole.us < plan.us) plan = whole;
    if ((long long)n_img * plan.tiles_u * plan.tiles_v >= (1ll << 31)) return fail(GDRR_EINVAL, "too many tiles in one call");
    std::vector<Launch> ls;
    DnParams d{};
    d.shat = shat;
    d.shat_stride = stride;
    d.n_img = n_img; d.nv = nv; d.nu = nu;
    d.omega = omega;
    d.inv_beta = 1.0f / beta;
    d.s_floor = s_floor;
    d.tiles_u = plan.tiles_u; d.tiles_v = plan.tiles_v; d.halo = plan.halo;
    // (a launch has fewer than 2^32 lanes)
    const long long lanes = 64ll * plan.waves * plan.tiles_u * plan.tiles_v;
    const int most = (int)std::max(1ll, std::min((long long)n_img, ((1ll << 32) - 1) / lanes));
    for (int first = 0; first < n_img; first += std::min(most, n_img - first)) {
        const size_t at = (size_t)first * (size_t)npix;
        d.n_img = std::min(most, n_img - first);
        d.shat = shat + (size_t)first * (size_t)stride;
        for (int p = 0; p < plan.passes; ++p) {
            const bool last = p + 1 == plan.passes;
            d.h_in = p > 0 && hf ? hf + at : nullptr;
            d.h_out = p == 0 && !last && hf ? hf + at : nullptr;
            d.s_in = p == 0 ? nullptr : pp[p & 1] + at;
            d.s_out = last ? nullptr : pp[(p + 1) & 1] + at;
            d.out = last ? out + at : nullptr;
            d.iters = std::min(plan.sweeps, iters - p * plan.sweeps);
            ls.push_back(make_launch(plan.kernel, dim3((unsigned)(d.n_img * plan.tiles_u * plan.tiles_v)), dim3(64 * plan.waves), 0, d));
        }
    }
    TimeEvents* ev = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_time_mu);
        if (g_timing && (rc = timing_events(&ev))) return rc;
    }
    return run_direct(ls, st, ev ? 0 : -1, ev, ev ? (int)ls.size() - 1 : -1);
}

// --------------------------------------------------------------------------
// Scratch of gdrr_mc_project_static: one array per device in the code object.
// Host code never passes `scratch` itself (in host code the name stands for a
// host-side shadow); it passes the device address that hipGetSymbolAddress
// returns for the current device, looked up once per device.
// --------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[GDRR_STATIC_SCRATCH_BYTES];

std::mutex g_scratch_mu;
void* g_scratch_ptr[64];

int static_scratch(void** out) {
    int dev = 0;
    GDRR_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(GDRR_ENOTSUP, "device index out of range");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        GDRR_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(GDRR_EHIP, "hipGetSymbolAddress returned NULL for the static scratch");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return GDRR_OK;
}

gdrr_job single_job(const gdrr_geometry* geom, uint64_t n, uint32_t job_id) {
    gdrr_job j{};
    j.volume = 0;
    j.source = 0;
    j.geom = *geom;
    j.n_photons = n;
    j.job_id = job_id;
    j.tally_offset = 0;
    return j;
}

}  // namespace

extern "C" {

const char* gdrr_last_error(void) { return g_err.c_str(); }

const char* gdrr_version(void) { return "gdrr-mi355x 0.1"; }

int gdrr_init(void) {
    DevInfo d;
    int rc = device_info(d);
    if (rc) return rc;
    void* p = nullptr;
    return static_scratch(&p);
}

int gdrr_enable_timing(int enable) {
    std::lock_guard<std::mutex> lk(g_time_mu);
    g_timing = enable != 0;
    return GDRR_OK;
}

int gdrr_last_kernel_ms(float* ms) {
    if (!ms) return fail(GDRR_EINVAL, "ms is NULL");
    int dev = 0;
    GDRR_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_time_mu);
    if (dev < 0 || dev >= 64 || !g_tev[dev].recorded) return fail(GDRR_EINVAL, "no timed launch on this device");
    GDRR_HIP(hipEventSynchronize(g_tev[dev].b));
    GDRR_HIP(hipEventElapsedTime(ms, g_tev[dev].a, g_tev[dev].b));
    return GDRR_OK;
}

int gdrr_default_tuning(gdrr_tuning* out) {
    if (!out) return fail(GDRR_EINVAL, "out is NULL");
    out->block = 256;
    out->blocks_per_cu = 0;
    out->chunk = 0;
    out->defer = 32;
    out->coll_defer = 0;
    return GDRR_OK;
}

size_t gdrr_majorant_workspace(void) { return 4096; }

int gdrr_majorant(const gdrr_volume* vol, const gdrr_physics* phys, uint32_t flags, float margin, float* out,
                  void* workspace, size_t ws_bytes, void* stream) {
    int rc;
    if ((rc = check_volume(vol)) || (rc = check_physics(phys))) return rc;
    if (!out) return fail(GDRR_EINVAL, "out is NULL");
    if (!(margin >= 0.0f) || !std::isfinite(margin)) return fail(GDRR_EINVAL, "margin must be finite and >= 0");
    if (!workspace || ws_bytes < gdrr_majorant_workspace()) return fail(GDRR_EINVAL, "workspace too small");
    DevInfo dev;
    if ((rc = device_info(dev))) return rc;
    hipStream_t st = (hipStream_t)stream;
    // the status block first (as in every workspace; word 1 holds the input-error bits), then the
    // per-material maxima and presence flags
    unsigned long long* head = (unsigned long long*)(((uintptr_t)workspace + 255) & ~(uintptr_t)255);
    unsigned int* err = (unsigned int*)(head + 1);
    unsigned int* rmax = (unsigned int*)(head + 8);
    unsigned int* pres = rmax + 256;
    std::vector<Launch> ls;
    FillParams f{head, 8 + 256};
    ls.push_back(make_launch((const void*)&fill_zero_kernel, dim3(2), dim3(256), 0, f));
    ls.push_back(voxels_launch(*vol, phys->n_mat, (flags & GDRR_INTERP_DENSITY) != 0, dev.cus, nullptr, true, rmax, pres, err));
    MajFinParams fp{rmax, pres, phys->mu_mass, phys->n_mat, phys->n_e, 1.0 + (double)margin, out, err};
    ls.push_back(make_launch((const void*)&majorant_kernel, dim3((phys->n_e + 254) / 256), dim3(256), 0, fp));
    return run_direct(ls, st);
}

size_t gdrr_mc_project_workspace(const gdrr_volume* vol, const gdrr_physics* phys, const gdrr_source* src,
                                 const gdrr_geometry* geom) {
    if (!geom) return 0;
    gdrr_job j = single_job(geom, 0, 0);
    return batch_bytes_all(vol, 1, phys, src, 1, &j, 1);
}

int gdrr_mc_project(const gdrr_volume* vol, const gdrr_physics* phys, const gdrr_source* src,
                    const gdrr_geometry* geom, const float* majorant, uint64_t seed, uint64_t n_photons,
                    uint32_t job_id, uint32_t flags, double* tally, void* workspace, size_t ws_bytes,
                    void* stream) {
    if (!geom) return fail(GDRR_EINVAL, "geometry is NULL");
    if (!tally) return fail(GDRR_EINVAL, "tally is NULL");
    gdrr_job j = single_job(geom, n_photons, job_id);
    Batch B{vol, 1, phys, src, 1, &j, 1, majorant, seed, flags, nullptr, kModeForward, -1, tally,
            nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, false};
    return run_batch(B, workspace, ws_bytes, (hipStream_t)stream);
}

int gdrr_mc_project_static(const gdrr_volume* vol, const gdrr_physics* phys, const gdrr_source* src,
                           const gdrr_geometry* geom, const float* majorant, uint64_t seed, uint64_t n_photons,
                           uint32_t job_id, uint32_t flags, double* tally, void* stream) {
    if (!geom) return fail(GDRR_EINVAL, "geometry is NULL");
    if (!tally) return fail(GDRR_EINVAL, "tally is NULL");
    if (flags & GDRR_RESUME) return fail(GDRR_EINVAL, "gdrr_mc_project_static does not resume (GDRR_RESUME)");
    gdrr_job j = single_job(geom, n_photons, job_id);
    Batch B{vol, 1, phys, src, 1, &j, 1, majorant, seed, flags, nullptr, kModeForward, -1, tally,
            nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, false};
    B.tables_by_kernel = true;
    int rc = check_batch(B);
    if (rc) return rc;
    const size_t need = batch_bytes(vol, 1, phys, src, 1, &j, 1, majorant == nullptr);
    if (need > GDRR_STATIC_SCRATCH_BYTES)
        return fail(GDRR_EINVAL, "gdrr_mc_project_static: the call needs " + std::to_string(need) +
                                 " bytes of scratch; the static scratch holds " +
                                 std::to_string((size_t)GDRR_STATIC_SCRATCH_BYTES) + " (use gdrr_mc_project)");
    void* ws = nullptr;
    if ((rc = static_scratch(&ws))) return rc;
    return run_batch(B, ws, GDRR_STATIC_SCRATCH_BYTES, (hipStream_t)stream);
}

size_t gdrr_mc_project_batch_workspace(const gdrr_volume* vols, int32_t n_vols, const gdrr_physics* phys,
                                       const gdrr_source* srcs, int32_t n_srcs, const gdrr_job* jobs,
                                       int32_t n_jobs) {
    return batch_bytes_all(vols, n_vols, phys, srcs, n_srcs, jobs, n_jobs);
}

int gdrr_mc_project_batch(const gdrr_volume* vols, int32_t n_vols, const gdrr_physics* phys,
                          const gdrr_source* srcs, int32_t n_srcs, const gdrr_job* jobs, int32_t n_jobs,
                          const float* majorants, uint64_t seed, uint32_t flags, const gdrr_tuning* tune,
                          double* tallies, void* workspace, size_t ws_bytes, void* stream) {
    if (!tallies) return fail(GDRR_EINVAL, "tallies is NULL");
    Batch B{vols, n_vols, phys, srcs, n_srcs, jobs, n_jobs, majorants, seed, flags, tune, kModeForward, -1,
            tallies, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, true};
    return run_batch(B, workspace, ws_bytes, (hipStream_t)stream);
}

int gdrr_mc_backward(const gdrr_volume* vols, int32_t n_vols, const gdrr_physics* phys, const gdrr_source* srcs,
                     int32_t n_srcs, const gdrr_job* jobs, int32_t n_jobs, int32_t volume, const float* majorants,
                     uint64_t seed, uint32_t flags, const gdrr_tuning* tune, const double* adj,
                     double* grad_density, void* workspace, size_t ws_bytes, void* stream) {
    if (!majorants) return fail(GDRR_EINVAL, "the adjoint needs the forward's majorants");
    if (!adj || !grad_density) return fail(GDRR_EINVAL, "adj / grad_density is NULL");
    if (volume < 0 || volume >= n_vols) return fail(GDRR_EINVAL, "volume index out of range");
    // (the gradient is cleared by run_batch's launch list, after every argument check)
    Batch B{vols, n_vols, phys, srcs, n_srcs, jobs, n_jobs, majorants, seed, flags, tune, kModeBackward, volume,
            nullptr, adj, grad_density, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, false};
    return run_batch(B, workspace, ws_bytes, (hipStream_t)stream);
}

size_t gdrr_primary_workspace(const gdrr_volume* vols, int32_t n_vols, const gdrr_physics* phys,
                              const gdrr_source* srcs, int32_t n_srcs, const gdrr_job* jobs, int32_t n_jobs) {
    if (!vols || !phys || !srcs || !jobs || n_vols < 1 || n_vols > GDRR_MAX_VOLUMES || n_srcs < 1 ||
        n_srcs > GDRR_MAX_SOURCES || n_jobs < 1)
        return 0;
    for (int k = 0; k < n_jobs; ++k)
        if (jobs[k].volume < 0 || jobs[k].volume >= n_vols) return 0;
    for (int v = 0; v < n_vols; ++v)
        if (vols[v].nx < 1 || vols[v].ny < 1 || vols[v].nz < 1) return 0;
    for (int s = 0; s < n_srcs; ++s)
        if (srcs[s].n_spec < 1 || spec_rows(srcs[s]) < 0) return 0;
    return rt_carve(nullptr, vols, n_vols, phys, srcs, n_srcs, jobs, n_jobs).bytes + 256;
}

int gdrr_primary(const gdrr_volume* vols, int32_t n_vols, const gdrr_physics* phys, const gdrr_source* srcs,
                 int32_t n_srcs, const gdrr_job* jobs, int32_t n_jobs, float step_mm, uint32_t flags, double* out,
                 void* workspace, size_t ws_bytes, void* stream) {
    return run_primary(vols, n_vols, phys, srcs, n_srcs, jobs, n_jobs, step_mm, flags, out, workspace, ws_bytes,
                       (hipStream_t)stream);
}

size_t gdrr_denoise_workspace(int32_t n_img, int32_t nv, int32_t nu) {
    if (n_img < 1 || nv < 1 || nu < 1) return 0;
    return 3 * dn_buffer_bytes(n_img, nv, nu) + 256;
}

int gdrr_denoise(const double* shat, int64_t shat_stride, int32_t n_img, int32_t nv, int32_t nu, float beta,
                 float omega, int32_t iters, float s_floor, double* out, void* workspace, size_t ws_bytes,
                 void* stream) {
    return run_denoise(shat, shat_stride, n_img, nv, nu, beta, omega, iters, s_floor, out, workspace, ws_bytes,
                       (hipStream_t)stream);
}

int gdrr_noise(int32_t n_img, int64_t npix, const double* phat, int64_t phat_stride, const double* p,
               const double* shat, int64_t shat_stride, const double* s, double alpha, double* noise,
               double* image, void* stream) {
    if (!phat || !p || !shat || !s) return fail(GDRR_EINVAL, "input pointer is NULL");
    if (n_img < 1 || npix < 1) return fail(GDRR_EINVAL, "n_img and npix must be >= 1");
    if (phat_stride == 0) phat_stride = npix;
    if (shat_stride == 0) shat_stride = npix;
    if (phat_stride < npix || shat_stride < npix) return fail(GDRR_EINVAL, "strides must be 0 or >= npix");
    if (!std::isfinite(alpha)) return fail(GDRR_EINVAL, "alpha must be finite");
    NoiseParams q{phat, phat_stride, p, shat, shat_stride, s, alpha, noise, image, npix, n_img};
    const long long total = npix * (long long)n_img;
    const unsigned grid = (unsigned)std::max<long long>(1, std::min<long long>(8192, (total + 255) / 256));
    void* a[1] = {&q};
    GDRR_HIP(hipLaunchKernel((const void*)&noise_kernel, dim3(grid), dim3(256), a, 0, (hipStream_t)stream));
    return GDRR_OK;
}

int gdrr_noise_scale(double n_sim, double zeta, double mas, double* alpha) {
    if (!alpha) return fail(GDRR_EINVAL, "alpha is NULL");
    if (!(n_sim > 0.0 && zeta > 0.0 && mas > 0.0) || !std::isfinite(n_sim) || !std::isfinite(zeta) ||
        !std::isfinite(mas))
        return fail(GDRR_EINVAL, "n_sim, zeta and mAs must be finite and > 0");
    *alpha = std::sqrt(n_sim / (zeta * mas));
    return GDRR_OK;
}

int gdrr_input_status(const void* workspace, void* stream) {
    if (!workspace) return fail(GDRR_EINVAL, "workspace is NULL");
    hipStream_t st = (hipStream_t)stream;
    const unsigned int* word = (const unsigned int*)((((uintptr_t)workspace + 255) & ~(uintptr_t)255) + 8);
    unsigned int bits = 0;
    GDRR_HIP(hipStreamSynchronize(st));
    GDRR_HIP(hipMemcpyAsync(&bits, word, sizeof(bits), hipMemcpyDeviceToHost, st));
    GDRR_HIP(hipStreamSynchronize(st));
    if (!bits) return GDRR_OK;
    std::string msg = "invalid device inputs:";
    if (bits & kErrDensity) msg += " densities negative, NaN or infinite (transported as 0);";
    if (bits & kErrMaterial) msg += " material indices >= n_mat (transported as n_mat - 1);";
    if (bits & kErrWeights) msg += " spectrum or fluence weights negative, non-finite or summing to 0;";
    msg.pop_back();
    return fail(GDRR_EINVAL, msg);
}

int gdrr_mc_trace(const gdrr_volume* vol, const gdrr_physics* phys, const gdrr_source* src,
                  const gdrr_geometry* geom, const float* majorant, uint64_t seed, uint64_t n_photons,
                  uint32_t job_id, uint32_t flags, int8_t* cls, int32_t* pixel, float* e_final, int32_t* steps,
                  int32_t* n_compton, int32_t* n_rayleigh, void* workspace, size_t ws_bytes, void* stream) {
    if (!geom) return fail(GDRR_EINVAL, "geometry is NULL");
    gdrr_job j = single_job(geom, n_photons, job_id);
    Batch B{vol, 1, phys, src, 1, &j, 1, majorant, seed, flags, nullptr, kModeTrace, -1, nullptr, nullptr,
            nullptr, cls, pixel, e_final, steps, n_compton, n_rayleigh, false};
    return run_batch(B, workspace, ws_bytes, (hipStream_t)stream);
}

}  // extern "C"
