// Temperature solve, Eq. 7 (Section 4.3).
//
// Plain FP32: a workgroup takes a tile of 64 (or 16) cells x 4 (or 16) grains.  The
// tile's heating (plus the extra term) is staged in LDS; each wave then solves
// one grain for the tile's cells (a cell per lane, or per four lanes), as the
// paper's third kernel gives a block one species, so the grain's Planck
// weights and the wavelength table are wave-uniform and come through the
// scalar cache.  Newton's first iterations run on the grain's table of ln P',
// which leaves one evaluation of the full sum as a rule.  T goes back through
// the same LDS slots; the iterations of the block are counted with one atomic.
// Mixed and table-linear: a workgroup takes 64 or 256 cells x 16 grains, a
// wave one grain at a time with a cell per lane (few grains of many cells: pairs
// in row-major order): an O(1) lookup in the grain's inverse table ln T(ln H) (a
// cubic Hermite in FP64 between FP64 nodes, or in FP32 with the FP32 lookup), or
// a bracketed search in its table of powers at evenly spaced T and linear
// interpolation (Sections 2 and 5).
// Every form adds the optional extra heating Q to H first.
#include "wave_heat.h"

namespace dust {
namespace {

// Plain: a workgroup takes 64 / R cells x GRAINS grains, a wave one grain at a
// time for all the cells.  One grain per wave (GRAINS = 4) rather than several in
// turn: more workgroups hide the loads of the weights better and end more evenly
// (with vector loads, 32768 x 968 x 81: 655 us, 799 with four grains per wave);
// on short rows of large calls four in turn (SHORT_ROWS).
// scaled: H holds the plan's scaled H' (the fused call's own).
// 32768 x 968 x 81: 1479 us with every iteration on the full sum, 382 with the
// first ones on the table and the weights as scalar loads; bound by the VALU
// and transcendental issue of the one evaluation of the full sum that is left
// (6.7e12 terms/s, a third of them in the cheaper forms).
template <int R, int GRAINS>
__global__ __launch_bounds__(256) void solve_plain_kernel(PlanView v, int64_t C,
                                                          const float* H, int64_t ldh, float* T,
                                                          int64_t ldt, bool scaled,
                                                          dust_counters* cnt) {
    constexpr int CELLS = 64 / R;
    constexpr int ST = GRAINS + 1;        // odd: a grain's column falls on distinct banks
    __shared__ float sX[CELLS * ST];      // heating in, T out
    __shared__ int sEvals[4];
    const int64_t c0 = (int64_t)blockIdx.x * CELLS;
    const int g0 = blockIdx.y * GRAINS;
    const int G = (v.S - g0 < GRAINS) ? v.S - g0 : GRAINS;
    const int rows = (C - c0 < CELLS) ? (int)(C - c0) : CELLS;
    // (H may be T: every element is read here before its T is written)
    for (int i = threadIdx.x; i < rows * GRAINS; i += 256) {
        const int cc = i / GRAINS, sl = i - cc * GRAINS;
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
    for (int sl = wave; sl < G; sl += 4) {
        const int s = g0 + sl;  // wave-uniform: the grain's weights come as scalars
        const float t0 = (live && v.warm) ? T[(c0 + cell) * ldt + s] : 0.0f;
        int ev;
        const float t = solve_newton_wave<R>(v, s, live, live ? sX[cell * ST + sl] : 0.0f, t0, &ev,
                                             cnt);
        if (live) sX[cell * ST + sl] = t;  // (the R lanes of a cell hold the same)
        evals += ev;
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
    for (int i = threadIdx.x; i < rows * GRAINS; i += 256) {
        const int cc = i / GRAINS, sl = i - cc * GRAINS;
        if (sl < G) T[(c0 + cc) * ldt + g0 + sl] = sX[cc * ST + sl];
    }
}

// The table forms: a workgroup takes 64 Q cells x 16 grains, its heating (plus
// the extra term) staged in LDS, and each wave four of the grains in turn, a
// cell per lane and Q lookups of one grain in flight.  A wave's gathers then
// fall into one grain's table (4 KB of inverse nodes), which L1 keeps for the
// tile's cells, and the grain's constants are scalars; pairs in row-major order
// gather 128-byte lines from every grain's table for each pair, and a 64-bit
// division per pair finds its grain.
// Pairs outside both tables are marked in LDS by the sign and, once the lookups
// are done, solved exactly by the tile's waves, a quarter each; a workgroup's
// blocks lie far apart, so that a cluster of such cells is spread over many
// workgroups.  Bound by the gathers and, at 64 cells, by the chain of dependent
// loads: 1048576 x 500 x 128 900 -> 553 us (H and T at copy rate: 225), the
// table-linear form 100003 x 301 x 45 87 -> 37 us.
constexpr int TABLE_GRAINS = 16;

template <int MODE, int Q>
__global__ __launch_bounds__(256) void solve_table_kernel(PlanView v, int64_t C,
                                                          const float* __restrict__ H, int64_t ldh,
                                                          float* __restrict__ T, int64_t ldt,
                                                          dust_counters* cnt) {
    constexpr int ST = TABLE_GRAINS + 1;  // odd: a grain's column falls on distinct banks
    constexpr int ROWS = 256 / TABLE_GRAINS, PER = 64 / ROWS;  // cells of one pass, passes of a block
    __shared__ float sX[64 * Q * ST];     // heating in, T out
    __shared__ int sPending;
    const int64_t nb = (C + 64 * Q - 1) / (64 * Q);  // workgroups along the cells
    const HeatTile ht = heat_tile<1>(blockIdx.x, v.Sp / 16);
    if (ht.c0 >= nb) return;
    const int g0 = TABLE_GRAINS * ht.tile;
    const int G = v.S - g0 < TABLE_GRAINS ? v.S - g0 : TABLE_GRAINS;
    // block k of the workgroup: 64 cells from this one on
    auto block = [&](int k) { return 64 * (ht.c0 + k * nb); };
    if (threadIdx.x == 0) sPending = 0;
    const int sl0 = threadIdx.x % TABLE_GRAINS, row = threadIdx.x / TABLE_GRAINS;
    {
        const float hscale = sl0 < G ? v.hscale[g0 + sl0] : 1.0f;
#pragma unroll
        for (int n = 0; n < PER * Q; ++n) {
            const int64_t c = block(n / PER) + ROWS * (n % PER) + row;
            float h = 0.0f;  // (pairs past the tile's end: T = 0, not stored)
            if (c < C && sl0 < G) {
                h = H[c * ldh + g0 + sl0];
                if (v.q) h += v.q[c * v.ldq + g0 + sl0];
            }
            sX[(ROWS * n + row) * ST + sl0] = h * hscale;
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int nonfinite = 0;
    for (int sl = wave; sl < G; sl += 4) {
        const int s = g0 + sl;  // wave-uniform
        float h[Q], t[Q];
        int st[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k) h[k] = sX[(64 * k + lane) * ST + sl];
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            if constexpr (MODE == DUST_MIXED) {
                st[k] = table_lookup_f64_nb(v, s, h[k], &t[k]);
            } else if constexpr (MODE == MODE_MIXED_F32) {
                st[k] = table_lookup_f32_nb(v, s, h[k], &t[k]);
            } else {
                st[k] = LOOKUP_OK;
                t[k] = 0.0f;
                if (block(k) + lane < C) {
                    if constexpr (MODE == MODE_MIXED_POLISH) {
                        if (table_lookup_polish(v, s, h[k], &t[k], cnt) != 0) st[k] = LOOKUP_PENDING;
                    } else {
                        t[k] = table_linear_T(v, s, h[k], cnt);
                    }
                }
            }
        }
        if constexpr (mixed_mode(MODE)) {
            bool pending = false;
#pragma unroll
            for (int k = 0; k < Q; ++k) {
                if (block(k) + lane >= C) st[k] = LOOKUP_OK;
                if (MODE != MODE_MIXED_POLISH && st[k] == LOOKUP_PENDING &&
                    cold_lookup(v, s, h[k], &t[k], cnt))
                    st[k] = LOOKUP_OK;
                nonfinite += st[k] == LOOKUP_NONFINITE;
                if (st[k] == LOOKUP_PENDING) {
                    t[k] = -h[k];
                    pending = true;
                }
            }
            if (pending) sPending = 1;
        }
#pragma unroll
        for (int k = 0; k < Q; ++k) sX[(64 * k + lane) * ST + sl] = t[k];
    }
    if (mixed_mode(MODE) && cnt) wave_count_add(&cnt->n_nonfinite, nonfinite);
    __syncthreads();
    if constexpr (mixed_mode(MODE)) {
        if (sPending) {  // uniform
            // wave w takes the pairs whose lane, block and grain add up to w mod 4
            // (a quarter of a cell's grains, and of a grain's cells)
            for (int sl = 0; sl < G; ++sl) {
                for (int k = 0; k < Q; ++k) {
                    float* x = &sX[(64 * k + lane) * ST + sl];
                    const float xl = ((lane + k + sl) & 3) == wave ? *x : 0.0f;
                    uint64_t mask = __ballot(__float_as_int(xl) < 0);
                    while (mask) {
                        const int src = __builtin_ctzll(mask);
                        mask &= mask - 1;
                        const float hp = -__int_as_float(
                            __builtin_amdgcn_readlane(__float_as_int(xl), src));
                        const float tp = wave_solve_pending(v, g0 + sl, (double)hp, cnt);
                        if (lane == src) *x = tp;
                    }
                }
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (int n = 0; n < PER * Q; ++n) {
        const int64_t c = block(n / PER) + ROWS * (n % PER) + row;
        if (c < C && sl0 < G) T[c * ldt + g0 + sl0] = sX[(ROWS * n + row) * ST + sl0];
    }
}

// The same for grids whose grains leave much of a 16-grain tile empty, and many
// cells: PER pairs per thread, 256 apart in row-major order, all looked up before
// any is stored (the table-linear search, with branches, takes one).  Pairs
// outside both tables go to an LDS list and are then solved exactly by the
// workgroup's waves in turn.
constexpr int pairs_per_thread(int mode) { return mixed_mode(mode) ? 4 : 1; }

template <int MODE>
__global__ __launch_bounds__(256) void solve_pairs_kernel(PlanView v, int64_t C,
                                                          const float* __restrict__ H, int64_t ldh,
                                                          float* __restrict__ T, int64_t ldt,
                                                          dust_counters* cnt) {
    constexpr int PER = pairs_per_thread(MODE), PAIRS_BLOCK = 256 * PER;
    __shared__ int sCount;
    __shared__ int sList[PAIRS_BLOCK];
    if (threadIdx.x == 0) sCount = 0;
    __syncthreads();
    const int64_t n = C * v.S;
    const int64_t base = (int64_t)blockIdx.x * PAIRS_BLOCK + threadIdx.x;
    int64_t c[PER];
    int s[PER];
    float hs[PER], t[PER];
    int st[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        // past the end, read the last pair again (nothing is stored for it)
        const int64_t i = (base + k * 256 < n) ? base + k * 256 : n - 1;
        c[k] = i / v.S;
        s[k] = (int)(i - c[k] * v.S);
        float h = H[c[k] * ldh + s[k]];
        if (v.q) h += v.q[c[k] * v.ldq + s[k]];
        hs[k] = h * v.hscale[s[k]];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if constexpr (MODE == DUST_MIXED) {
            st[k] = table_lookup_f64_nb(v, s[k], hs[k], &t[k]);
        } else if constexpr (MODE == MODE_MIXED_F32) {
            st[k] = table_lookup_f32_nb(v, s[k], hs[k], &t[k]);
        } else {
            st[k] = LOOKUP_OK;
            if (base + k * 256 < n) {
                if constexpr (MODE == MODE_MIXED_POLISH) {
                    if (table_lookup_polish(v, s[k], hs[k], &t[k], cnt) != 0) st[k] = LOOKUP_PENDING;
                } else {
                    t[k] = table_linear_T(v, s[k], hs[k], cnt);
                }
            }
        }
    }
    int nonfinite = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (base + k * 256 >= n) continue;
        if (mixed_mode(MODE) && MODE != MODE_MIXED_POLISH && st[k] == LOOKUP_PENDING &&
            cold_lookup(v, s[k], hs[k], &t[k], cnt))
            st[k] = LOOKUP_OK;
        if (st[k] == LOOKUP_PENDING) {
            sList[atomicAdd(&sCount, 1)] = threadIdx.x + k * 256;
        } else {
            nonfinite += st[k] == LOOKUP_NONFINITE;
            T[c[k] * ldt + s[k]] = t[k];
        }
    }
    if constexpr (mixed_mode(MODE)) {
        if (cnt) wave_count_add(&cnt->n_nonfinite, nonfinite);
        __syncthreads();
        const int np = sCount;
        for (int e = threadIdx.x >> 6; e < np; e += 4) {
            const int64_t ip = (int64_t)blockIdx.x * PAIRS_BLOCK + sList[e];
            const int64_t cp = ip / v.S;
            const int sp = (int)(ip - cp * v.S);
            float hf = H[cp * ldh + sp];
            if (v.q) hf += v.q[cp * v.ldq + sp];
            const float tp = wave_solve_pending(v, sp, (double)(hf * v.hscale[sp]), cnt);
            if ((threadIdx.x & 63) == 0) T[cp * ldt + sp] = tp;
        }
    }
}

// A launch holds fewer than 2^32 threads: f(view, first cell, cells) for slices
// of at most `most` cells.
template <typename F>
hipError_t in_slices(const PlanView& v, int64_t C, int64_t most, F&& f) {
    PlanView w = v;
    for (int64_t c = 0; c < C; c += most) {
        if (v.q) w.q = v.q + c * v.ldq;
        f(w, c, C - c < most ? C - c : most);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
constexpr int64_t MAX_BLOCKS = (1 << 24) - 1;  // of 256 threads

template <int MODE, int Q>
hipError_t launch_table(const PlanView& v, int64_t C, const float* H, int64_t ldh, float* T,
                        int64_t ldt, dust_counters* cnt, hipStream_t st) {
    const int tiles = v.Sp / 16;
    return in_slices(v, C, MAX_BLOCKS / (8 * tiles) * 8 * 64 * Q,
                     [&](const PlanView& w, int64_t c, int64_t n) {
        hipLaunchKernelGGL((solve_table_kernel<MODE, Q>), dim3(heat_blocks<64 * Q>(n, tiles)),
                           dim3(256), 0, st, w, n, H + c * ldh, ldh, T + c * ldt, ldt, cnt);
    });
}

template <int MODE>
hipError_t launch_pairs(const PlanView& v, int64_t C, const float* H, int64_t ldh, float* T,
                        int64_t ldt, dust_counters* cnt, hipStream_t st) {
    constexpr int PAIRS_BLOCK = 256 * pairs_per_thread(MODE);
    return in_slices(v, C, MAX_BLOCKS * PAIRS_BLOCK / v.S,
                     [&](const PlanView& w, int64_t c, int64_t n) {
        hipLaunchKernelGGL(solve_pairs_kernel<MODE>,
                           dim3((unsigned)((n * v.S + PAIRS_BLOCK - 1) / PAIRS_BLOCK)), dim3(256), 0,
                           st, w, n, H + c * ldh, ldh, T + c * ldt, ldt, cnt);
    });
}

// Whether pairs in row-major order beat 16-grain tiles: where few grains fill
// little of the last tile and the cells fill the GPU (below, more workgroups
// hide the gathers).  Tiles against pairs, mixed: 1500000 cells x 1 grain 35.3 us
// and 8.6, x 4 58 and 34, x 12 81 and 78, x 16 91 and 101, x 20 158 and 124, x 33
// 300 and 299 (FP32 lookup: 283 and 244), x 45 337 and 417; 400000 x 1 9.1 and
// 6.1, x 5 and x 8 equal, x 20 51 and 41; 100000 x 20 13.3 and 14.3.  The
// table-linear search, longer, is bound by its gathers from four grains on.
bool pairs_pay(const PlanView& v, int64_t C, int km) {
    if (C < 262144) return false;
    if (km == DUST_TABLE_LINEAR) return v.S <= 3;
    if (km == MODE_MIXED_F32) return v.S <= 36;  // (16 grains: 80 us against 74)
    return v.S <= 12 || (v.S > 16 && v.S <= 24);
}

// The branch-free lookups take 256 cells per workgroup, four of a grain in
// flight, once that leaves four workgroups per CU (100003 x 301 x 45: 21 us
// either way; 262144 x 250 x 80 71 us against 86 with 64 cells, 32768 x 250 x
// 80 13.1 with 64 cells, 15.4 with 256).  The polish and the table-linear
// search branch per pair, so more cells only lengthen a wave's chain (262144
// x 250 x 80 with 64 cells 136 and 154 us, with 256 140 and 160; 16384 cells
// 12 and 14, 24 and 25).
constexpr int64_t TABLE_BLOCKS = 1024;

template <int MODE>
hipError_t launch_table_mode(const PlanView& v, int64_t C, const float* H, int64_t ldh, float* T,
                             int64_t ldt, dust_counters* cnt, hipStream_t st) {
    if (pairs_pay(v, C, MODE)) return launch_pairs<MODE>(v, C, H, ldh, T, ldt, cnt, st);
    if constexpr (MODE == DUST_MIXED || MODE == MODE_MIXED_F32) {
        if ((C + 255) / 256 * (v.Sp / 16) >= TABLE_BLOCKS)
            return launch_table<MODE, 4>(v, C, H, ldh, T, ldt, cnt, st);
    }
    return launch_table<MODE, 1>(v, C, H, ldh, T, ldt, cnt, st);
}

}  // namespace

hipError_t launch_solve(const PlanView& v, int64_t C, const float* H, int64_t ldh, float* T,
                        int64_t ldt, dust_counters* cnt, hipStream_t st) {
    if (C == 0) return hipSuccess;
    if (!table_mode(v.mode)) return launch_solve_plain(v, C, H, ldh, T, ldt, false, cnt, st);
    switch (kernel_mode(v)) {
        case DUST_MIXED: return launch_table_mode<DUST_MIXED>(v, C, H, ldh, T, ldt, cnt, st);
        case MODE_MIXED_F32: return launch_table_mode<MODE_MIXED_F32>(v, C, H, ldh, T, ldt, cnt, st);
        case MODE_MIXED_POLISH:
            return launch_table_mode<MODE_MIXED_POLISH>(v, C, H, ldh, T, ldt, cnt, st);
        default: return launch_table_mode<DUST_TABLE_LINEAR>(v, C, H, ldh, T, ldt, cnt, st);
    }
}

// Four lanes per cell where the (64 cells, grain) waves leave SIMDs idle: 32 x
// 968 x 81 29.5 -> 9.9 us, 256 x 250 x 80 12.4 -> 8.4, 1024 x 968 x 81 (1296
// waves) 33.0 -> 29.2; at 2000 waves (1600 x 250 x 80) 13.9 against 15.6, at
// 3807 (3000 x 968 x 81) 51.6 against 72.1.
constexpr int64_t PLAIN_FEW_WAVES = 1536;
// Short rows of more pairs than the caches hold: four grains per workgroup are 16
// bytes of every row of H and T, and the sums are too short to hide that (2000000
// x 45: 3 wavelengths 4.34 ms with four grains, 4.11 with 16, 64 wavelengths 1.97
// and 1.74; 400000 x 80, 64 wavelengths 595 us and 583, 100 731 and 754; 50000 x 45
// fit the caches, 119 and 142 us at 3).
constexpr int SHORT_ROWS = 64;
constexpr int64_t SHORT_PAIRS = 30000000;

template <int R, int GRAINS>
hipError_t launch_plain(const PlanView& v, int64_t C, const float* H, int64_t ldh, float* T,
                        int64_t ldt, bool scaled, dust_counters* cnt, hipStream_t st) {
    const dim3 grid((unsigned)((C + 64 / R - 1) / (64 / R)),
                    (unsigned)((v.S + GRAINS - 1) / GRAINS));
    hipLaunchKernelGGL((solve_plain_kernel<R, GRAINS>), grid, dim3(256), 0, st, v, C, H, ldh, T, ldt,
                       scaled, cnt);
    return hipGetLastError();
}

hipError_t launch_solve_plain(const PlanView& v, int64_t C, const float* H, int64_t ldh, float* T,
                              int64_t ldt, bool scaled, dust_counters* cnt, hipStream_t st) {
    if (C == 0) return hipSuccess;
    const int64_t waves = (C + 63) / 64 * v.S;
    if (waves <= PLAIN_FEW_WAVES) return launch_plain<4, 4>(v, C, H, ldh, T, ldt, scaled, cnt, st);
    if (v.NL <= SHORT_ROWS && v.S >= 16 && C * v.S >= SHORT_PAIRS)
        return launch_plain<1, 16>(v, C, H, ldh, T, ldt, scaled, cnt, st);
    return launch_plain<1, 4>(v, C, H, ldh, T, ldt, scaled, cnt, st);
}

}  // namespace dust
