// Batched synthesis over many stars: every stage is one persistent launch
// whose workgroups take (star, item) work from a list spanning all stars.
// The opacity stage (dominant and skewed: stars differ in window length,
// line count and line density) pulls items from an atomic queue ordered by
// decreasing cost; the cheap, uniform stages stride over their lists.  The
// stage bodies are those of the per-star kernels (pz_stages.h), so each star
// gets bitwise the per-star result.  The host also hosts the autotuner.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "pz_stages.h"

namespace pz {
int set_error(int code, const char* msg);
int check_atmos(const pz_plan* plan, const pz_atmos* atm);
int check_params(const pz_params* par);
StarDev make_star(const pz_plan* p, const pz_atmos* atm, const pz_params* par);
}  // namespace pz

using namespace pz;

namespace {

enum Phase {
    PH_POP,        // (star, 512 (species, depth) pairs)
    PH_LINES,      // (star, 512 lines): per-line factors
    PH_PARAMS,     // (star, PARAM_ITEM (line, depth) pairs)
    PH_OP32,       // (star, tile) of stars with 32-pixel tiles, decreasing cost, atomic queue
    PH_OP64,       // ... 64-pixel tiles
    PH_OP128,      // ... 128-pixel tiles
    PH_SPLIT,      // (star, 32-pixel tile) of stars with split sums, decreasing cost
    PH_FAR2,       // (star, 32-pixel tile): far zone of stars with short grids
    PH_FAR4,       // (star, 64-pixel tile): ... with long ones
    PH_SEED,       // (star, 512 pixels): chi^2 seed for stars with a target
    PH_LOSS,       // (star): chi^2 value, one 1024-thread workgroup
    PH_FLUX,       // (star, ROW_ITEM pixels): transfer, one list for each transfer_list()
    PH_REVERSE = PH_FLUX + 10,   // ... its adjoint
    PH_REVERSE_END = PH_REVERSE + 9,
    PH_GATHER,     // (star, GATHER_ITEM lines), atomic queue
    PH_GSPLIT,     // (star, GATHER_ITEM lines) of stars with split sums, atomic queue
    PH_SCATTER,    // (star, 512 lines)
    PH_PARTIAL,    // (star, list b * n_rchunk + c)
    PH_FINAL,      // (star, list b)
    N_PHASE
};

constexpr int PARAM_ITEM = 512 * 32;
constexpr int N_COUNTER = 5;             // queues: opacity x 3 tile widths, gather, split gather
constexpr int GATHER_ITEM = 64;
constexpr int ROW_ITEM = 64;             // pixels of a transfer item: four passes of 16 by rows, one by columns
// Lists 2 (np - 2) + E2 by rows with np depths per lane, 8 + E2 by columns: what the star's own calls take.
int transfer_list(const pz::StarDev& s, bool reverse) {
    const bool e2 = s.quad == PZ_QUAD_E2;
    return (reverse ? PH_REVERSE : PH_FLUX) + (pz::columns_rule(s.N, s.D, s.quad, reverse) ? 8 : 2 * (pz::row_np(s.D) - 2)) + e2;
}

// Next item of an atomic queue for the whole workgroup (wavefront-uniform).
__device__ __forceinline__ int next_item(int* ctr, int* s_it) {
    if (threadIdx.x == 0) *s_it = atomicAdd(ctr, 1);
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(*s_it);
    __syncthreads();
    return it;
}

// The item of a workgroup, made wavefront-uniform so the star descriptor is
// read with scalar loads.
__device__ __forceinline__ int2 uniform_item(const int2* __restrict__ items, int it) {
    const int2 w = items[it];
    return make_int2(__builtin_amdgcn_readfirstlane(w.x), __builtin_amdgcn_readfirstlane(w.y));
}

__global__ void kb_reset(int* ctr, int n) {
    if ((int)threadIdx.x < n) ctr[threadIdx.x] = 0;
}

__global__ __launch_bounds__(512) void kb_pop(const StarDev* __restrict__ stars, const int2* __restrict__ items, int n) {
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = uniform_item(items, it);
        dev_populations(stars[w.x], w.y * 512 + threadIdx.x);
    }
}

__global__ __launch_bounds__(512) void kb_lines(const StarDev* __restrict__ stars, const int2* __restrict__ items, int n) {
    __shared__ double red[4 * 512];
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = uniform_item(items, it);
        const DampBounds bnd = damp_bounds(stars[w.x], red);
        dev_line_consts(stars[w.x], w.y * 512 + threadIdx.x, bnd);
    }
}

__global__ __launch_bounds__(512) void kb_params(const StarDev* __restrict__ stars, const int2* __restrict__ items, int n) {
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = uniform_item(items, it);
        const StarDev& s = stars[w.x];
        const long base = (long)w.y * PARAM_ITEM;
        for (int k = threadIdx.x; k < PARAM_ITEM; k += 512) dev_line_params(s, base + k);
    }
}

// ANYCT: some star of the batch uses the centre test (the LDS holds its rows);
// G: depth-group slots (at least D / (64 / WPX) for every star); FG: exactly
// D / (64 / WPX) for every star.
// NTH: threads per workgroup, 512 for a whole tile or a part of it (items are
// taken in parts then).
template <int WPX, bool ANYCT, int G, bool FG, int NTH>
__global__ __launch_bounds__(NTH) PZ_OPACITY_WAVES(WPX) void kb_opacity(const StarDev* __restrict__ stars, const int2* __restrict__ items, int n, int* ctr) {
    PZ_OPACITY_LDS(WPX, ANYCT, sm);
    __shared__ int s_it;
    load_pw_table(sm.pw, false);                       // visible after the first item fetch's barrier
    for (;;) {
        constexpr int PARTS = 512 / NTH;
        const int it = next_item(ctr, &s_it);
        if (it >= n * PARTS) return;
        const int2 w = uniform_item(items, it / PARTS);
        const StarDev& s = stars[w.x];
        dev_opacity_tile<WPX, false, ANYCT, G, false, FG, NTH>(s, w.y, it % PARTS, s.chunk, sm);
    }
}

// Adds the lines flagged wide_a (usually none) to every (star, tile) item.
template <int WPX, bool ANYCT>
__global__ __launch_bounds__(512) PZ_OPACITY_WAVES(WPX) void kb_opacity_wide(const StarDev* __restrict__ stars, const int2* __restrict__ items, int n) {
    PZ_OPACITY_LDS(WPX, ANYCT, sm);
    load_pw_table(sm.pw, false);
    __syncthreads();
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = uniform_item(items, it);
        const StarDev& s = stars[w.x];
        dev_opacity_tile<WPX, true, ANYCT, opacity_max_groups<WPX>(), false>(s, w.y, 0, s.chunk, sm);
    }
}

// Split sums: one workgroup per (star, tile) item; the far zone's form is the
// one that the star's own calls take.
__global__ __launch_bounds__(far_waves<2>() * WAVE) void kb_opacity_far2(const StarDev* __restrict__ stars, const int2* __restrict__ items) {
    __shared__ FarLds<2> lds;
    const int2 w = uniform_item(items, blockIdx.x);
    dev_opacity_far<2>(stars[w.x], w.y, lds);
}

__global__ __launch_bounds__(far_waves<4>() * WAVE) void kb_opacity_far4(const StarDev* __restrict__ stars, const int2* __restrict__ items) {
    __shared__ FarLds<4> lds;
    const int2 w = uniform_item(items, blockIdx.x);
    dev_opacity_far<4>(stars[w.x], w.y, lds);
}

// blockIdx.y: the depth groups of the tile (enough for the deepest star).
__global__ __launch_bounds__(256) void kb_opacity_near(const StarDev* __restrict__ stars, const int2* __restrict__ items) {
    __shared__ float4 near_tab[PZ_NEAR_N];
    __shared__ float4 pw[PZ_PW_LDS];
    const int2 w = uniform_item(items, blockIdx.x);
    const StarDev& s = stars[w.x];
    if ((int)blockIdx.y >= near_parts(s.D)) return;
    load_near_table(near_tab);
    load_pw_table(pw, false);
    __syncthreads();
    if (s.center)
        dev_opacity_near<NEAR_G, true>(s, w.y, blockIdx.y, near_tab, pw);
    else
        dev_opacity_near<NEAR_G, false>(s, w.y, blockIdx.y, near_tab, pw);
}

// Transfer (REV: its adjoint) of the stars with NP depths per lane and one
// quadrature: a kernel for all of them would take the registers of the largest
// everywhere (254, one wavefront per SIMD): the adjoint of eight stars took
// 0.36 ms so, 0.33 by one thread per pixel, and takes 0.24.
template <int NP, bool E2, bool REV>
__global__ __launch_bounds__(256) void kb_rows(const StarDev* __restrict__ stars, const int2* __restrict__ items) {
    const int2 w = uniform_item(items, blockIdx.x);
    const StarDev& s = stars[w.x];
#pragma unroll 1
    for (int k = 0; k < ROW_ITEM; k += 16) {
        const int i = w.y * ROW_ITEM + k + threadIdx.x / 16;
        if constexpr (REV && E2)
            dev_reverse_e2_row<NP>(s, i);
        else if constexpr (REV)
            dev_reverse_row<NP>(s, i);
        else
            dev_flux_e2_row<NP>(s, i);
    }
}

__global__ __launch_bounds__(256) void kb_flux(const StarDev* __restrict__ stars, const int2* __restrict__ items) {
    __shared__ FluxLds lds;
    const int2 w = uniform_item(items, blockIdx.x);
    const StarDev& s = stars[w.x];
#pragma unroll 1
    for (int k = w.y * ROW_ITEM; k < min((w.y + 1) * ROW_ITEM, s.N); k += FLUX_PX) dev_flux_block(s, k, lds);
}

// One thread per pixel; blockIdx.y: the branch.
template <bool E2>
__global__ __launch_bounds__(WAVE) void kb_flux_column(const StarDev* __restrict__ stars, const int2* __restrict__ items) {
    __shared__ float col[MAXD * WAVE];
    const int2 w = uniform_item(items, blockIdx.x);
    dev_flux_columns<E2>(stars[w.x], w.y * ROW_ITEM + threadIdx.x, blockIdx.y == 0, col + threadIdx.x);
}

template <bool E2>
__global__ __launch_bounds__(WAVE) void kb_reverse_column(const StarDev* __restrict__ stars, const int2* __restrict__ items) {
    __shared__ double col[MAXD * WAVE];
    const int2 w = uniform_item(items, blockIdx.x);
    dev_reverse_columns<E2>(stars[w.x], w.y * ROW_ITEM + threadIdx.x, col + threadIdx.x);
}
static_assert(ROW_ITEM == WAVE, "an item by columns is one wavefront");

__global__ __launch_bounds__(512) void kb_seed(const StarDev* __restrict__ stars, const int2* __restrict__ items, int n, const float* inv_s2,
                                               const float* const* ys) {
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = uniform_item(items, it);
        const StarDev& s = stars[w.x];
        dev_chi2_seed(s.N, s.F, s.Fc, ys[w.x], inv_s2[w.x], const_cast<float*>(s.dLdF), nullptr,
                      w.y * 512 + threadIdx.x);
    }
}

__global__ __launch_bounds__(1024) void kb_loss(const StarDev* __restrict__ stars, const int2* __restrict__ items, int n, const float* inv_s2,
                                                const float* const* ys, float* const* losses) {
    __shared__ float red[1024];
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = uniform_item(items, it);
        const StarDev& s = stars[w.x];
        dev_chi2_loss(s.N, s.F, s.Fc, ys[w.x], inv_s2[w.x], losses[w.x], red);
        __syncthreads();
    }
}

// NEAR: the near zone of the split sums, after kb_gather_far.
template <bool NEAR>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(8))) void kb_gather(const StarDev* __restrict__ stars, const int2* __restrict__ items, int n, int* ctr) {
    __shared__ int s_it;
    __shared__ float4 pw[2 * PZ_PW_LDS];
    __shared__ float4 lq[512 / WAVE][2 * MAXD];
    load_pw_table(pw, true);                           // visible after the first item fetch's barrier
    const int wave = threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
    for (;;) {
        const int it = next_item(ctr, &s_it);
        if (it >= n) return;
        const int2 w = uniform_item(items, it);
        const StarDev& s = stars[w.x];
        for (int q = wave; q < GATHER_ITEM; q += 512 / WAVE) {
            const int l = __builtin_amdgcn_readfirstlane(w.y * GATHER_ITEM + q);
            // the row is private to this wavefront: order its writes before the
            // reads and the previous line's reads before the writes
            __builtin_amdgcn_wave_barrier();
            stage_line_params(s, l, lane, lq[wave]);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            dev_gather<NEAR>(s, l, lane, pw, lq[wave]);
        }
    }
}

// Split sums: GATHER_ITEM lines per workgroup, by two pairs of wavefronts.
__global__ __launch_bounds__(256) void kb_gather_far(const StarDev* __restrict__ stars, const int2* __restrict__ items) {
    const int2 w = uniform_item(items, blockIdx.x);
    const StarDev& s = stars[w.x];
    __shared__ LineSums hand[2][GFAR_LINES];
    const int wave = threadIdx.x / WAVE;
    for (int q = 0; q < GATHER_ITEM; q += 2 * GFAR_LINES) {
        const int base = w.y * GATHER_ITEM + q + wave / 2 * GFAR_LINES;
        if (s.fam)
            dev_gather_far<true>(s, base, wave % 2, hand[wave / 2]);
        else
            dev_gather_far<false>(s, base, wave % 2, hand[wave / 2]);
        __syncthreads();
    }
}

__global__ __launch_bounds__(512) void kb_scatter(const StarDev* __restrict__ stars, const int2* __restrict__ items, int n) {
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = uniform_item(items, it);
        dev_scatter(stars[w.x], w.y * 512 + threadIdx.x);
    }
}

__global__ __launch_bounds__(256) void kb_partial(const StarDev* __restrict__ stars, const int2* __restrict__ items, int n) {
    __shared__ float red[256];
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = uniform_item(items, it);
        const StarDev& s = stars[w.x];
        dev_reduce_partial(s, w.y % s.n_rchunk, w.y / s.n_rchunk, red);
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void kb_final(const StarDev* __restrict__ stars, const int2* __restrict__ items, int n) {
    __shared__ float red[256];
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = uniform_item(items, it);
        dev_reduce_final(stars[w.x], w.y, red);
        __syncthreads();
    }
}

size_t align_up(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace

template <bool ANYCT>
static hipError_t batch_opacity_occupancy(int* occ) {
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ[0], kb_opacity<4, ANYCT, 4, true, 512>, 512, 0);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ[1], kb_opacity<8, ANYCT, 9, true, 512>, 512, 0);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ[2], kb_opacity<16, ANYCT, 19, false, 512>, 512, 0);
    return e;
}

struct pz_batch {
    int n_star;
    int device;
    bool has_target;
    bool any_center;      // some star uses the centre test
    int max_d;            // largest depth count of the stars
    int min_d;            // smallest depth count of the stars
    std::vector<StarDev> sc_stars;   // stars with continuum scattering (their own flux and reverse launches)
    std::vector<const pz_plan*> plans;
    int n_items[N_PHASE];
    int2* items[N_PHASE];
    StarDev* stars;
    float* inv_s2;
    const float** ys;
    float** losses;
    int* ctr;             // [N_COUNTER] queue counters: opacity (32, 64, 128), gather, split gather
    int grid512, grid256, grid1024, grid_op[3], grid_gather;
    bool halves64;        // 64-pixel opacity tiles in halves
    void* base;
};

// One phase's opacity launches: the main pass with the fewest depth-group
// slots that hold every star's D / (64 / WPX) groups (with no empty slot when
// every star has the same group count), then the wide pass.
template <int WPX, bool ANYCT, int NTH>
static void batch_opacity_main(const pz_batch* bt, int n, const int2* items, int* ctr, int grid, hipStream_t st) {
    constexpr int GB = opacity_max_groups<WPX>();
    const int ng = bt->max_d / (64 / WPX);             // <= GB: D <= MAXD
    const bool same = bt->min_d / (64 / WPX) == ng;
    if (ng == GB)
        same ? kb_opacity<WPX, ANYCT, GB, true, NTH><<<grid, NTH, 0, st>>>(bt->stars, items, n, ctr)
             : kb_opacity<WPX, ANYCT, GB, false, NTH><<<grid, NTH, 0, st>>>(bt->stars, items, n, ctr);
    else if (ng == GB - 1 && same)
        kb_opacity<WPX, ANYCT, GB - 1, true, NTH><<<grid, NTH, 0, st>>>(bt->stars, items, n, ctr);
    else
        kb_opacity<WPX, ANYCT, GB - 1, false, NTH><<<grid, NTH, 0, st>>>(bt->stars, items, n, ctr);
}

// Tiles in halves as in the per-star launches (the same bits either way).
// 64-pixel tiles gain where the heaviest one outlasts the chip's share of the
// rest: the items' costs add up to less than half of slots x the heaviest.
// Eight stars of unlike line densities (888 tiles, 0.44 of it) take 17.8 ms
// forward + backward in halves, 20.1 whole and 22.4 in quarters; alike stars
// of 440 tiles (0.53) 1132 us forward whole and 1246 in halves (40 depths).
template <int WPX, bool ANYCT>
static void batch_opacity_wpx(const pz_batch* bt, int n, const int2* items, int* ctr, int grid, hipStream_t st) {
    if (opacity_halves<WPX, ANYCT>(bt->halves64))
        batch_opacity_main<WPX, ANYCT, opacity_half_threads<WPX, ANYCT>()>(bt, n, items, ctr, 2 * grid, st);
    else
        batch_opacity_main<WPX, ANYCT, 512>(bt, n, items, ctr, grid, st);
    kb_opacity_wide<WPX, ANYCT><<<grid, 512, 0, st>>>(bt->stars, items, n);
}

template <bool ANYCT>
static void batch_opacity(const pz_batch* bt, hipStream_t st) {
    auto grid = [](int want, int n) { return std::max(1, std::min(want, n)); };
    const int* n = bt->n_items;
    int2* const* it = bt->items;
    if (n[PH_OP32]) batch_opacity_wpx<4, ANYCT>(bt, n[PH_OP32], it[PH_OP32], bt->ctr, grid(bt->grid_op[0], n[PH_OP32]), st);
    if (n[PH_OP64])
        batch_opacity_wpx<8, ANYCT>(bt, n[PH_OP64], it[PH_OP64], bt->ctr + 1, grid(bt->grid_op[1], n[PH_OP64]), st);
    if (n[PH_OP128])
        batch_opacity_wpx<16, ANYCT>(bt, n[PH_OP128], it[PH_OP128], bt->ctr + 2, grid(bt->grid_op[2], n[PH_OP128]), st);
}

template <bool REV>
static void batch_transfer(const pz_batch* bt, hipStream_t st) {
    constexpr int PH = REV ? PH_REVERSE : PH_FLUX;
    const int* n = bt->n_items + PH;
    int2* const* it = bt->items + PH;
    for (int np = 2; np <= 5; ++np)
        with_row_np(16 * np, [&](auto NP) {
            const int g = 2 * (np - 2), e = g + 1;
            if (n[g]) {
                if constexpr (REV)
                    kb_rows<NP.value, false, true><<<n[g], 256, 0, st>>>(bt->stars, it[g]);
                else
                    kb_flux<<<n[g], 256, 0, st>>>(bt->stars, it[g]);
            }
            if (n[e]) kb_rows<NP.value, true, REV><<<n[e], 256, 0, st>>>(bt->stars, it[e]);
        });
    if constexpr (REV) {
        if (n[8]) kb_reverse_column<false><<<n[8], WAVE, 0, st>>>(bt->stars, it[8]);
        if (n[9]) kb_reverse_column<true><<<n[9], WAVE, 0, st>>>(bt->stars, it[9]);
    } else {
        if (n[8]) kb_flux_column<false><<<dim3(n[8], 2), WAVE, 0, st>>>(bt->stars, it[8]);
        if (n[9]) kb_flux_column<true><<<dim3(n[9], 2), WAVE, 0, st>>>(bt->stars, it[9]);
    }
}

extern "C" {

int pz_batch_create(int32_t n_star, const pz_star* stars, pz_batch** out) {
    if (!out) return set_error(PZ_E_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (n_star < 1 || !stars) return set_error(PZ_E_INVALID_ARG, "need n_star >= 1 stars");
    std::vector<StarDev> sd(n_star);
    std::vector<float> inv_s2(n_star, 0.0f);
    std::vector<const float*> ys(n_star, nullptr);
    std::vector<float*> losses(n_star, nullptr);
    std::vector<std::vector<int2>> items(N_PHASE);
    bool has_target = false;
    for (int b = 0; b < n_star; ++b) {
        const pz_star& st = stars[b];
        if (!st.plan) return set_error(PZ_E_INVALID_ARG, "star without a plan");
        for (int c = 0; c < b; ++c)
            if (stars[c].plan == st.plan) return set_error(PZ_E_INVALID_ARG, "two stars share a plan");
        int rc = check_atmos(st.plan, &st.atm);
        if (rc) return rc;
        if ((rc = check_params(&st.par))) return rc;
        if (st.atm.sigma_c && !st.plan->scatter_ws)
            return set_error(PZ_E_INVALID_ARG,
                             "a star has sigma_c but its plan was built without PZ_FLAG_SCATTERING");
        if (!st.F || !st.Fc) return set_error(PZ_E_INVALID_ARG, "every star needs F and Fc");
        if (st.y && !(st.sigma > 0.0f)) return set_error(PZ_E_INVALID_ARG, "sigma must be > 0 with a target y");
        const pz_plan* p = st.plan;
        StarDev s = make_star(p, &st.atm, &st.par);
        s.F = st.F;
        s.Fc = st.Fc;
        s.dLdF = st.y ? p->seed : st.dL_dF;
        s.g_loggf = st.g_loggf;
        s.g_damp = st.g_damp;
        s.g_abund = st.g_abund;
        s.g_xi = st.g_xi;
        sd[b] = s;
        if (st.y) {
            has_target = true;
            inv_s2[b] = 1.0f / (st.sigma * st.sigma);
            ys[b] = st.y;
            losses[b] = st.loss;
        }
        const long nld = (long)s.L * s.D;
        for (int k = 0; k < (s.S * s.D + 511) / 512; ++k) items[PH_POP].push_back({b, k});
        for (int k = 0; k < (s.L + 511) / 512; ++k) items[PH_LINES].push_back({b, k});
        for (long k = 0; k < (nld + PARAM_ITEM - 1) / PARAM_ITEM; ++k) items[PH_PARAMS].push_back({b, (int)k});
        const int ph_op = s.split ? PH_SPLIT : s.tile_px == 32 ? PH_OP32 : (s.tile_px == 64 ? PH_OP64 : PH_OP128);
        for (int t = 0; t < (s.split ? s.n_t32 : s.n_tiles); ++t) items[ph_op].push_back({b, t});
        if (s.split) {
            const bool wide = far_wide(s.n_t32);
            for (int t = 0; t < (wide ? (s.n_t32 + 1) / 2 : s.n_t32); ++t) items[wide ? PH_FAR4 : PH_FAR2].push_back({b, t});
        }
        // a star with scattering runs its transfer and reverse transfer in launches of its own
        if (st.y)
            for (int k = 0; k < (s.N + 511) / 512; ++k) items[PH_SEED].push_back({b, k});
        if (!s.scatter)
            for (int k = 0; k < (s.N + ROW_ITEM - 1) / ROW_ITEM; ++k)
                for (bool rev : {false, true}) items[transfer_list(s, rev)].push_back({b, k});
        if (st.y && st.loss) items[PH_LOSS].push_back({b, 0});
        for (int k = 0; k < (s.L + GATHER_ITEM - 1) / GATHER_ITEM; ++k) items[s.split_gather ? PH_GSPLIT : PH_GATHER].push_back({b, k});
        for (int k = 0; k < (s.L + 511) / 512; ++k) items[PH_SCATTER].push_back({b, k});
        for (int k = 0; k < (s.S + 1) * s.n_rchunk; ++k) items[PH_PARTIAL].push_back({b, k});
        for (int k = 0; k < s.S + 1; ++k) items[PH_FINAL].push_back({b, k});
    }
    // opacity work: most expensive tiles first (longest-processing-time order)
    for (int ph : {PH_OP32, PH_OP64, PH_OP128, PH_SPLIT})
        std::stable_sort(items[ph].begin(), items[ph].end(), [&](const int2& x, const int2& y) {
            return stars[x.x].plan->tile_cost[x.y] > stars[y.x].plan->tile_cost[y.y];
        });

    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes);
        return o;
    };
    size_t o_items[N_PHASE];
    for (int ph = 0; ph < N_PHASE; ++ph) o_items[ph] = take(std::max<size_t>(items[ph].size(), 1) * sizeof(int2));
    const size_t o_st = take(n_star * sizeof(StarDev)), o_is = take(n_star * 4), o_ys = take(n_star * 8),
                 o_ls = take(n_star * 8), o_ctr = take(N_COUNTER * 4);
    pz_batch* bt = new (std::nothrow) pz_batch();
    if (!bt) return set_error(PZ_E_NOMEM, "host allocation failed");
    char* base = nullptr;
    if (hipGetDevice(&bt->device) != hipSuccess || hipMalloc((void**)&base, off) != hipSuccess) {
        (void)hipGetLastError();
        delete bt;
        return set_error(PZ_E_NOMEM, "device allocation for the batch failed");
    }
    bt->base = base;
    bt->n_star = n_star;
    bt->has_target = has_target;
    hipError_t e = hipSuccess;
    for (int ph = 0; ph < N_PHASE; ++ph) {
        bt->items[ph] = (int2*)(base + o_items[ph]);
        bt->n_items[ph] = (int)items[ph].size();
        if (e == hipSuccess && !items[ph].empty())
            e = hipMemcpy(bt->items[ph], items[ph].data(), items[ph].size() * sizeof(int2), hipMemcpyHostToDevice);
    }
    bt->stars = (StarDev*)(base + o_st);
    bt->inv_s2 = (float*)(base + o_is);
    bt->ys = (const float**)(base + o_ys);
    bt->losses = (float**)(base + o_ls);
    bt->ctr = (int*)(base + o_ctr);
    if (e == hipSuccess) e = hipMemcpy(bt->stars, sd.data(), n_star * sizeof(StarDev), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(bt->inv_s2, inv_s2.data(), n_star * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(bt->ys, ys.data(), n_star * 8, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(bt->losses, losses.data(), n_star * 8, hipMemcpyHostToDevice);
    int n_cu = 0, occ_op[3] = {0, 0, 0}, occ_g = 0;
    if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, bt->device);
    bt->any_center = false;
    bt->max_d = 0;
    bt->min_d = MAXD;
    for (int b = 0; b < n_star; ++b) {
        bt->any_center = bt->any_center || sd[b].center;
        bt->max_d = std::max(bt->max_d, sd[b].D);
        bt->min_d = std::min(bt->min_d, sd[b].D);
    }
    if (e == hipSuccess)
        e = bt->any_center ? batch_opacity_occupancy<true>(occ_op) : batch_opacity_occupancy<false>(occ_op);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ_g, kb_gather<false>, 512, 0);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        (void)hipFree(base);
        delete bt;
        return set_error(PZ_E_HIP, hipGetErrorString(e));
    }
    for (int k = 0; k < 3; ++k) bt->grid_op[k] = std::max(1, n_cu * std::max(occ_op[k], 1));
    bt->grid_gather = std::max(1, n_cu * std::max(occ_g, 1));
    double cost = 0.0, heaviest = 0.0;
    for (const int2& w : items[PH_OP64]) {
        const double c = (double)stars[w.x].plan->tile_cost[w.y];
        cost += c;
        heaviest = std::max(heaviest, c);
    }
    bt->halves64 = 2.0 * cost <= heaviest * bt->grid_op[1];
    bt->grid512 = std::max(1, n_cu * 4);
    bt->grid256 = std::max(1, n_cu * 8);
    bt->grid1024 = std::max(1, n_cu * 2);
    bt->plans.reserve(n_star);
    for (int b = 0; b < n_star; ++b) bt->plans.push_back(stars[b].plan);
    for (int b = 0; b < n_star; ++b)
        if (sd[b].scatter) bt->sc_stars.push_back(sd[b]);
    *out = bt;
    return PZ_OK;
}

void pz_batch_destroy(pz_batch* batch) {
    if (!batch) return;
    (void)hipDeviceSynchronize();
    (void)hipFree(batch->base);
    delete batch;
}

int synth_batch(const pz_batch* bt, int32_t mode, pz_stream stream) {
    if (!bt) return set_error(PZ_E_INVALID_ARG, "batch is NULL");
    if (mode != PZ_MODE_FWD && mode != PZ_MODE_FWD_BWD) return set_error(PZ_E_INVALID_ARG, "unknown mode");
    hipStream_t st = (hipStream_t)stream;
    auto grid = [](int want, int n) { return std::max(1, std::min(want, n)); };
    const int* n = bt->n_items;
    int2* const* it = bt->items;
    kb_reset<<<1, 64, 0, st>>>(bt->ctr, N_COUNTER);
    kb_pop<<<grid(bt->grid512, n[PH_POP]), 512, 0, st>>>(bt->stars, it[PH_POP], n[PH_POP]);
    if (n[PH_LINES]) kb_lines<<<grid(bt->grid512, n[PH_LINES]), 512, 0, st>>>(bt->stars, it[PH_LINES], n[PH_LINES]);
    kb_params<<<grid(bt->grid512, n[PH_PARAMS]), 512, 0, st>>>(bt->stars, it[PH_PARAMS], n[PH_PARAMS]);
    if (n[PH_SPLIT]) {
        if (n[PH_FAR4]) kb_opacity_far4<<<n[PH_FAR4], far_waves<4>() * WAVE, 0, st>>>(bt->stars, it[PH_FAR4]);
        if (n[PH_FAR2]) kb_opacity_far2<<<n[PH_FAR2], far_waves<2>() * WAVE, 0, st>>>(bt->stars, it[PH_FAR2]);
        kb_opacity_near<<<dim3(n[PH_SPLIT], near_parts(bt->max_d)), 256, 0, st>>>(bt->stars, it[PH_SPLIT]);
    }
    if (bt->any_center)
        batch_opacity<true>(bt, st);
    else
        batch_opacity<false>(bt, st);
    batch_transfer<false>(bt, st);
    for (const StarDev& s : bt->sc_stars) {
        const hipError_t e = launch_flux(s, st);
        if (e != hipSuccess) return set_error(PZ_E_HIP, hipGetErrorString(e));
    }
    if (n[PH_SEED])
        kb_seed<<<grid(bt->grid512, n[PH_SEED]), 512, 0, st>>>(bt->stars, it[PH_SEED], n[PH_SEED], bt->inv_s2, bt->ys);
    if (n[PH_LOSS])
        kb_loss<<<grid(bt->grid1024, n[PH_LOSS]), 1024, 0, st>>>(bt->stars, it[PH_LOSS], n[PH_LOSS], bt->inv_s2,
                                                                 bt->ys, bt->losses);
    if (mode == PZ_MODE_FWD_BWD) {
        batch_transfer<true>(bt, st);
        for (const StarDev& s : bt->sc_stars) {
            const hipError_t e = launch_reverse_scan(s, st);
            if (e != hipSuccess) return set_error(PZ_E_HIP, hipGetErrorString(e));
        }
        if (n[PH_GSPLIT]) {
            kb_gather_far<<<n[PH_GSPLIT], 256, 0, st>>>(bt->stars, it[PH_GSPLIT]);
            kb_gather<true><<<grid(bt->grid_gather, n[PH_GSPLIT]), 512, 0, st>>>(bt->stars, it[PH_GSPLIT], n[PH_GSPLIT],
                                                                                  bt->ctr + 4);
        }
        if (n[PH_GATHER])
            kb_gather<false><<<grid(bt->grid_gather, n[PH_GATHER]), 512, 0, st>>>(bt->stars, it[PH_GATHER], n[PH_GATHER],
                                                                                   bt->ctr + 3);
        kb_scatter<<<grid(bt->grid512, n[PH_SCATTER]), 512, 0, st>>>(bt->stars, it[PH_SCATTER], n[PH_SCATTER]);
        kb_partial<<<grid(bt->grid256, n[PH_PARTIAL]), 256, 0, st>>>(bt->stars, it[PH_PARTIAL], n[PH_PARTIAL]);
        kb_final<<<grid(bt->grid256, n[PH_FINAL]), 256, 0, st>>>(bt->stars, it[PH_FINAL], n[PH_FINAL]);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(PZ_E_HIP, hipGetErrorString(e));
    for (const pz_plan* p : bt->plans) {
        const_cast<pz_plan*>(p)->ws_valid = false;
        const_cast<pz_plan*>(p)->sc_ok = false;
    }
    return PZ_OK;
}

int pz_autotune(const pz_grid* grid, const pz_lines* lines, int32_t n_species, int32_t n_depth,
                const pz_options* base, const pz_atmos* atm, const pz_params* par, int32_t reps, pz_options* best,
                float* best_ms) {
    if (!grid || !lines || !base || !atm || !par || !best) return set_error(PZ_E_INVALID_ARG, "null argument");
    if (reps < 1) return set_error(PZ_E_INVALID_ARG, "reps must be >= 1");
    const int tiles[3] = {32, 64, 128};
    const int chunks[2] = {8, 16};
    float* F = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    float bms = 1e30f;
    pz_options bo = *base;
    int rc = PZ_OK;
    if (hipMalloc((void**)&F, (size_t)2 * std::max(grid->N, 1) * 4) != hipSuccess || hipEventCreate(&e0) != hipSuccess ||
        hipEventCreate(&e1) != hipSuccess) {
        rc = set_error(PZ_E_NOMEM, "autotune buffers");
    }
    bool split = false;                                // the pair has no effect: one is timed, the noise of six not ranked
    for (int ti = 0; ti < 3 && rc == PZ_OK && !split; ++ti) {
        for (int ci = 0; ci < 2 && rc == PZ_OK && !split; ++ci) {
            pz_options o = *base;
            o.tile_px = tiles[ti];
            o.lines_per_chunk = chunks[ci];
            pz_plan* p = nullptr;
            if ((rc = pz_plan_create(grid, lines, n_species, n_depth, &o, &p))) break;
            split = p->split;
            if (split) o.lines_per_chunk = 16;         // with 32 pixels what direct plans of these sizes take
            if ((rc = synth_forward(p, atm, par, F, F + grid->N, nullptr)) == PZ_OK) {
                (void)hipEventRecord(e0, nullptr);
                for (int r = 0; r < reps && rc == PZ_OK; ++r) rc = synth_forward(p, atm, par, F, F + grid->N, nullptr);
                (void)hipEventRecord(e1, nullptr);
                float ms = 0.0f;
                if (rc == PZ_OK && hipEventSynchronize(e1) == hipSuccess &&
                    hipEventElapsedTime(&ms, e0, e1) == hipSuccess) {
                    ms /= reps;
                    if (ms < bms) {
                        bms = ms;
                        bo = o;
                    }
                }
            }
            pz_plan_destroy(p);
        }
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (F) (void)hipFree(F);
    if (rc) return rc;
    *best = bo;
    if (best_ms) *best_ms = bms;
    return PZ_OK;
}

}  // extern "C"
