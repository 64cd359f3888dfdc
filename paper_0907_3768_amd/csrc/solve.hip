// Temperature solve, Eq. 7 (Section 4.3).
//
// Plain FP32: a workgroup takes a tile of 64 (or 16) cells x 4 grains.  The
// tile's heating (plus the extra term) is staged in LDS; each wave then solves
// one grain for the tile's cells (a cell per lane, or per four lanes), as the
// paper's third kernel gives a block one species, so the grain's Planck
// weights and the wavelength table are wave-uniform and come through the
// scalar cache.  Newton's first iterations run on the grain's table of ln P',
// which leaves one evaluation of the full sum as a rule.  T goes back through
// the same LDS slots; the iterations of the block are counted with one atomic.
// Mixed: four (cell, grain) pairs per thread, 256 apart in row-major order
// (coalesced H and T), each an O(1) lookup in the grain's inverse table
// ln T(ln H) (a cubic Hermite in FP64 between FP64 nodes, or in FP32 with the
// FP32 lookup), all four in flight together.
// Table-linear: the same layout, a bracketed search in the grain's table of
// powers at evenly spaced T and linear interpolation (Sections 2 and 5).
// Every form adds the optional extra heating Q to H first.
#include "device_common.h"

namespace dust {
namespace {

constexpr int PLAIN_GRAINS = 4;  // grains per workgroup: one per wave

// Plain: a workgroup takes 64 / R cells x 4 grains, a wave one grain for all
// the cells.  One grain per wave rather than several in turn: more workgroups
// hide the loads of the weights better and end more evenly (with vector loads,
// 32768 x 968 x 81: 655 us, 799 with four grains per wave).
// scaled: H holds the plan's scaled H' (the fused call's own).
// 32768 x 968 x 81: 1479 us with every iteration on the full sum, 382 with the
// first ones on the table and the weights as scalar loads; bound by the VALU
// and transcendental issue of the one evaluation of the full sum that is left
// (6.7e12 terms/s, a third of them in the cheaper forms).
template <int R>
__global__ __launch_bounds__(256) void solve_plain_kernel(PlanView v, int64_t C,
                                                          const float* H, int64_t ldh, float* T,
                                                          int64_t ldt, bool scaled,
                                                          dust_counters* cnt) {
    constexpr int CELLS = 64 / R;
    constexpr int ST = PLAIN_GRAINS + 1;  // odd: a grain's column falls on distinct banks
    __shared__ float sX[CELLS * ST];      // heating in, T out
    __shared__ int sEvals[4];
    const int64_t c0 = (int64_t)blockIdx.x * CELLS;
    const int g0 = blockIdx.y * PLAIN_GRAINS;
    const int G = (v.S - g0 < PLAIN_GRAINS) ? v.S - g0 : PLAIN_GRAINS;
    const int rows = (C - c0 < CELLS) ? (int)(C - c0) : CELLS;
    // (H may be T: every element is read here before its T is written)
    for (int i = threadIdx.x; i < rows * PLAIN_GRAINS; i += 256) {
        const int cc = i / PLAIN_GRAINS, sl = i - cc * PLAIN_GRAINS;
        if (sl >= G) continue;
        const int64_t c = c0 + cc;
        const float h = H[c * ldh + g0 + sl], q = v.q ? v.q[c * v.ldq + g0 + sl] : 0.0f;
        const float hscale = v.hscale[g0 + sl];
        sX[cc * ST + sl] = scaled ? h + q * hscale : (h + q) * hscale;
    }
    __syncthreads();
    const int cell = (threadIdx.x & 63) / R;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool live = cell < rows;
    int evals = 0;
    if (wave < G) {
        const int s = g0 + wave;  // wave-uniform: the grain's weights come as scalars
        const float t0 = (live && v.warm) ? T[(c0 + cell) * ldt + s] : 0.0f;
        const float t = solve_newton_wave<R>(v, s, live, live ? sX[cell * ST + wave] : 0.0f, t0,
                                             &evals, cnt);
        if (live) sX[cell * ST + wave] = t;  // (the R lanes of a cell hold the same)
    }
    if (cnt) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) evals += __shfl_xor(evals, off, 64);
        if ((threadIdx.x & 63) == 0) sEvals[wave] = evals;
    }
    __syncthreads();
    if (cnt && threadIdx.x == 0) {
        const int n = sEvals[0] + sEvals[1] + sEvals[2] + sEvals[3];
        if (n) atomicAdd(reinterpret_cast<unsigned long long*>(&cnt->n_newton_evals),
                         (unsigned long long)n);
    }
    for (int i = threadIdx.x; i < rows * PLAIN_GRAINS; i += 256) {
        const int cc = i / PLAIN_GRAINS, sl = i - cc * PLAIN_GRAINS;
        if (sl < G) T[(c0 + cc) * ldt + g0 + sl] = sX[cc * ST + sl];
    }
}

// Table-linear: one thread per (cell, grain) in row-major order.
__global__ __launch_bounds__(256) void solve_table_kernel(PlanView v, int64_t C,
                                                          const float* __restrict__ H,
                                                          int64_t ldh, float* __restrict__ T,
                                                          int64_t ldt, dust_counters* cnt) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= C * v.S) return;
    const int64_t c = i / v.S;
    const int s = (int)(i - c * v.S);
    float h = H[c * ldh + s];
    if (v.q) h += v.q[c * v.ldq + s];
    T[c * ldt + s] = table_linear_T(v, s, h * v.hscale[s], cnt);
}

// Mixed: each thread takes MIXED_PER pairs 256 apart in row-major order
// (coalesced H and T) and looks all of them up before it stores any, so that
// their dependent loads (H, then the grain's inverse-table nodes) overlap: a
// single lookup per thread leaves the kernel waiting on memory latency.  Pairs
// outside both tables go to an LDS list and are then solved exactly by the
// block's waves in turn (one pair per wave at a time, lanes over wavelength).
constexpr int MIXED_PER = 4;
constexpr int MIXED_BLOCK = 256 * MIXED_PER;  // pairs per workgroup

template <int MODE>
__device__ __forceinline__ int lookup_status(const PlanView& v, int s, float hs, float* T,
                                             bool active, dust_counters* cnt) {
    if constexpr (MODE == MODE_MIXED_POLISH) {
        if (!active) return LOOKUP_OK;
        return table_lookup_polish(v, s, hs, T, cnt) != 0 ? LOOKUP_PENDING : LOOKUP_OK;
    } else if constexpr (MODE == MODE_MIXED_F32) {
        return table_lookup_f32_nb(v, s, hs, T);
    } else {
        return table_lookup_f64_nb(v, s, hs, T);
    }
}

template <int MODE>
__global__ __launch_bounds__(256) void solve_mixed_kernel(PlanView v, int64_t C,
                                                          const float* __restrict__ H,
                                                          int64_t ldh, float* __restrict__ T,
                                                          int64_t ldt, dust_counters* cnt) {
    __shared__ int sCount;
    __shared__ int sList[MIXED_BLOCK];
    if (threadIdx.x == 0) sCount = 0;
    __syncthreads();
    const int64_t n = C * v.S;
    const int64_t base = (int64_t)blockIdx.x * MIXED_BLOCK + threadIdx.x;
    int64_t c[MIXED_PER];
    int s[MIXED_PER];
    float hs[MIXED_PER];
#pragma unroll
    for (int k = 0; k < MIXED_PER; ++k) {
        // past the end, read the last pair again (nothing is stored for it)
        const int64_t i = (base + k * 256 < n) ? base + k * 256 : n - 1;
        c[k] = i / v.S;
        s[k] = (int)(i - c[k] * v.S);
        float h = H[c[k] * ldh + s[k]];
        if (v.q) h += v.q[c[k] * v.ldq + s[k]];
        hs[k] = h * v.hscale[s[k]];
    }
    float t[MIXED_PER];
    int st[MIXED_PER];
#pragma unroll
    for (int k = 0; k < MIXED_PER; ++k)
        st[k] = lookup_status<MODE>(v, s[k], hs[k], &t[k], base + k * 256 < n, cnt);
    int nonfinite = 0;
#pragma unroll
    for (int k = 0; k < MIXED_PER; ++k) {
        if (base + k * 256 >= n) continue;
        if (MODE != MODE_MIXED_POLISH && st[k] == LOOKUP_PENDING &&
            cold_lookup(v, s[k], hs[k], &t[k], cnt))
            st[k] = LOOKUP_OK;
        if (st[k] == LOOKUP_PENDING) {
            sList[atomicAdd(&sCount, 1)] = threadIdx.x + k * 256;
        } else {
            nonfinite += st[k] == LOOKUP_NONFINITE;
            T[c[k] * ldt + s[k]] = t[k];
        }
    }
    if (cnt) wave_count_add(&cnt->n_nonfinite, nonfinite);
    __syncthreads();
    const int np = sCount;
    for (int e = threadIdx.x >> 6; e < np; e += blockDim.x >> 6) {
        const int64_t ip = (int64_t)blockIdx.x * MIXED_BLOCK + sList[e];
        const int64_t cp = ip / v.S;
        const int sp = (int)(ip - cp * v.S);
        float hf = H[cp * ldh + sp];
        if (v.q) hf += v.q[cp * v.ldq + sp];
        const double hp = (double)(hf * v.hscale[sp]);
        const float tp = wave_solve_pending(v, sp, hp, cnt);
        if ((threadIdx.x & 63) == 0) T[cp * ldt + sp] = tp;
    }
}

}  // namespace

hipError_t launch_solve(const PlanView& v, int64_t C, const float* H, int64_t ldh, float* T,
                        int64_t ldt, dust_counters* cnt, hipStream_t st) {
    if (C == 0) return hipSuccess;
    if (v.mode == DUST_MIXED) {
        const int64_t n = C * v.S;
        const unsigned blocks = (unsigned)((n + MIXED_BLOCK - 1) / MIXED_BLOCK);
        if (v.f32_lookup)
            hipLaunchKernelGGL(solve_mixed_kernel<MODE_MIXED_F32>,
                               dim3(blocks), dim3(256), 0, st, v, C, H, ldh, T, ldt, cnt);
        else if (v.polish)
            hipLaunchKernelGGL(solve_mixed_kernel<MODE_MIXED_POLISH>, dim3(blocks), dim3(256), 0,
                               st, v, C, H, ldh, T, ldt, cnt);
        else
            hipLaunchKernelGGL(solve_mixed_kernel<DUST_MIXED>, dim3(blocks), dim3(256), 0, st, v,
                               C, H, ldh, T, ldt, cnt);
    } else if (v.mode == DUST_TABLE_LINEAR) {
        const int64_t n = C * v.S;
        hipLaunchKernelGGL(solve_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                           st, v, C, H, ldh, T, ldt, cnt);
    } else {
        return launch_solve_plain(v, C, H, ldh, T, ldt, false, cnt, st);
    }
    return hipGetLastError();
}

// Four lanes per cell where the (64 cells, grain) waves leave SIMDs idle: 32 x
// 968 x 81 29.5 -> 9.9 us, 256 x 250 x 80 12.4 -> 8.4, 1024 x 968 x 81 (1296
// waves) 33.0 -> 29.2; at 2000 waves (1600 x 250 x 80) 13.9 against 15.6, at
// 3807 (3000 x 968 x 81) 51.6 against 72.1.
constexpr int64_t PLAIN_FEW_WAVES = 1536;

hipError_t launch_solve_plain(const PlanView& v, int64_t C, const float* H, int64_t ldh, float* T,
                              int64_t ldt, bool scaled, dust_counters* cnt, hipStream_t st) {
    if (C == 0) return hipSuccess;
    const unsigned gy = (unsigned)((v.S + PLAIN_GRAINS - 1) / PLAIN_GRAINS);
    if ((C + 63) / 64 * v.S <= PLAIN_FEW_WAVES)
        hipLaunchKernelGGL(solve_plain_kernel<4>, dim3((unsigned)((C + 15) / 16), gy), dim3(256), 0,
                           st, v, C, H, ldh, T, ldt, scaled, cnt);
    else
        hipLaunchKernelGGL(solve_plain_kernel<1>, dim3((unsigned)((C + 63) / 64), gy), dim3(256), 0,
                           st, v, C, H, ldh, T, ldt, scaled, cnt);
    return hipGetLastError();
}

}  // namespace dust
