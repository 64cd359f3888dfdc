// Fused absorb -> solve -> emit (Eqs. 6, 7, 9-10) for a tile of 16 cells per
// workgroup.  The heating tile goes from the MFMA accumulators to LDS, is
// solved in place (LDS then holds 1/T), and feeds the emission loop: H never
// reaches device memory and T is written once.
#include "fused_body.h"
#include "wave_heat.h"

namespace dust {
namespace {

// Resident waves per SIMD: six (80 VGPRs) -- more tiles in flight keep the
// phases of different tiles overlapping.  Up to 128 grains the compiler
// spills only inside the exact fallback for out-of-table pairs, which tiles
// without such pairs branch over; measured 4 % faster than five, seven
// slower.  Above 128 grains (three or four grain tiles per wave, J in
// 64-wavelength chunks) a few heating values spill too, and six waves still
// measured 0.4-2.6 % faster than five.
// TAIL: the emission's odd last grain group is its own step (grids whose
// grain count leaves an odd number of 8-grain groups).
template <int MODE, int NTW, bool TAIL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6, 8))) void fused_kernel(
    PlanView v, int64_t C,
                                                   const float* __restrict__ J, int64_t ldj,
                                                   const float* __restrict__ m,
                                                   float* __restrict__ T, int64_t ldt,
                                                   float* __restrict__ L, int64_t ldl,
                                                   dust_counters* cnt) {
    extern __shared__ float sTile[];
    fused_tile<MODE, FUSED_TC, NTW, TAIL, fused_kc(NTW)>(v, (int64_t)blockIdx.x * FUSED_TC, C, J, ldj, m, T, ldt, L,
                                          ldl, cnt, sTile);
}

// Absorb + solve only (the first of the two-kernel form): T is written once
// and the emission kernel follows.
template <int MODE, int NTW>
__global__ __launch_bounds__(256) void absorb_solve_kernel(PlanView v, int64_t C,
                                                          const float* __restrict__ J,
                                                          int64_t ldj, float* __restrict__ T,
                                                          int64_t ldt, dust_counters* cnt) {
    extern __shared__ float lds[];  // sH [16][Sp], J staging, pending list
    char* sStage = reinterpret_cast<char*>(lds + FUSED_TC * v.Sp);
    const int64_t c0 = (int64_t)blockIdx.x * FUSED_TC;
    fused_absorb<MODE, NTW>(v, c0, C, J, ldj, lds, sStage);
    __syncthreads();
    fused_solve<MODE, FUSED_TC>(v, c0, C, T, ldt, cnt, lds,
                                reinterpret_cast<int*>(sStage + STAGE_BYTES));
}

// Absorb + solve for small calls: one wave per 16 cells x 16 grains, WAVES grain
// tiles of 16 cells per workgroup, the heating straight from device memory
// (heat_block) and the lookups straight from the accumulators, four pairs of
// one grain per lane.  Pairs the table does not take go to an LDS list, which
// the workgroup's waves (those past the last tile among them) solve exactly in
// turn.  The emission kernel follows.
template <int MODE, bool ALIGNED, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void heat_solve_kernel(PlanView v, int64_t C,
                                                         const float* __restrict__ J, int64_t ldj,
                                                         float* __restrict__ T, int64_t ldt,
                                                         dust_counters* cnt) {
    __shared__ int sCount;
    __shared__ float sHeat[256 * WAVES];     // the pending pairs' H' and
    __shared__ uint16_t sPair[256 * WAVES];  // 64 cell + grain of the workgroup's
    const int tiles = v.Sp / 16;
    const HeatTile ht = heat_tile<16>(blockIdx.x, (tiles + WAVES - 1) / WAVES);
    if (ht.c0 >= C) return;
    if constexpr (mixed_mode(MODE)) {
        if (threadIdx.x == 0) sCount = 0;
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = WAVES * ht.tile + wave;
    if (tile < tiles) {
        f32x4 hacc[1][1];
        heat_block<true, ALIGNED, 1, 1, 4>(v, ht.c0, C, tile, J, ldj, hacc);
        const f32x4 acc = hacc[0][0];
        const int s_raw = 16 * tile + (lane & 15);
        const int s = s_raw < v.S ? s_raw : v.S - 1;  // a lane past the last grain looks it up unused
        const int64_t cl = ht.c0 + 4 * (lane >> 4);
        float h[4], t[4];
        int st[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            h[r] = acc[r];
            if (v.q && s_raw < v.S && cl + r < C) h[r] += v.q[(cl + r) * v.ldq + s] * v.hscale[s];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool pair = s_raw < v.S && cl + r < C;
            if constexpr (MODE == DUST_MIXED) {
                st[r] = table_lookup_f64_nb(v, s, h[r], &t[r]);
                if (!pair)
                    st[r] = LOOKUP_OK;
                else if (st[r] == LOOKUP_PENDING && cold_lookup(v, s, h[r], &t[r], cnt))
                    st[r] = LOOKUP_OK;
            } else {  // (the fused kernel's lookup: the branch-free FP32 one rounds differently)
                st[r] = LOOKUP_OK;
                if (pair) {
                    if constexpr (mixed_mode(MODE)) {
                        if (mixed_lookup<MODE>(v, s, h[r], &t[r], cnt) != 0) st[r] = LOOKUP_PENDING;
                    } else {
                        t[r] = table_linear_T(v, s, h[r], cnt);
                    }
                }
            }
            if (pair && st[r] != LOOKUP_PENDING) T[(cl + r) * ldt + s] = t[r];
            if (mixed_mode(MODE) && st[r] == LOOKUP_PENDING) {
                const int e = atomicAdd(&sCount, 1);
                sHeat[e] = h[r];
                sPair[e] = (uint16_t)(64 * (4 * (lane >> 4) + r) + 16 * wave + (lane & 15));
            }
        }
        if (MODE == DUST_MIXED && cnt) {
            int bad = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) bad += st[r] == LOOKUP_NONFINITE;
            wave_count_add(&cnt->n_nonfinite, bad);
        }
    }
    if constexpr (mixed_mode(MODE)) {
        __syncthreads();
        const int np = sCount;
        for (int e = wave; e < np; e += WAVES) {
            const int sp = 16 * WAVES * ht.tile + (sPair[e] & 63);
            const float tp = wave_solve_pending(v, sp, (double)sHeat[e], cnt);
            if (lane == 0) T[(ht.c0 + (sPair[e] >> 6)) * ldt + sp] = tp;
        }
    }
}

// Grids of up to three grain tiles take four waves per workgroup, so that some
// are free to share a tile's exact solves (700 cells x 600 wavelengths x 16
// grains, every pair outside the table: 1.73 ms with one wave, 0.47 with four;
// 14.3 us either way with none); more tiles are waves enough, and spread better
// one by one (32 x 968 x 81 17.0 us against 19.8).
template <int MODE, bool ALIGNED>
hipError_t launch_heat_solve_mode(const PlanView& v, int64_t C, const float* J, int64_t ldj,
                                  float* T, int64_t ldt, dust_counters* cnt, hipStream_t st) {
    const int tiles = v.Sp / 16;
    if (mixed_mode(MODE) && tiles <= 3)
        hipLaunchKernelGGL((heat_solve_kernel<MODE, ALIGNED, 4>), dim3(heat_blocks<16>(C, 1)),
                           dim3(256), 0, st, v, C, J, ldj, T, ldt, cnt);
    else
        hipLaunchKernelGGL((heat_solve_kernel<MODE, ALIGNED, 1>), dim3(heat_blocks<16>(C, tiles)),
                           dim3(64), 0, st, v, C, J, ldj, T, ldt, cnt);
    return hipGetLastError();
}

template <bool ALIGNED>
hipError_t launch_heat_solve(const PlanView& v, int64_t C, const float* J, int64_t ldj, float* T,
                             int64_t ldt, dust_counters* cnt, hipStream_t st) {
    switch (kernel_mode(v)) {
        case DUST_MIXED:
            return launch_heat_solve_mode<DUST_MIXED, ALIGNED>(v, C, J, ldj, T, ldt, cnt, st);
        case MODE_MIXED_F32:
            return launch_heat_solve_mode<MODE_MIXED_F32, ALIGNED>(v, C, J, ldj, T, ldt, cnt, st);
        case MODE_MIXED_POLISH:
            return launch_heat_solve_mode<MODE_MIXED_POLISH, ALIGNED>(v, C, J, ldj, T, ldt, cnt, st);
        default:
            return launch_heat_solve_mode<DUST_TABLE_LINEAR, ALIGNED>(v, C, J, ldj, T, ldt, cnt, st);
    }
}

template <int NTW>
hipError_t launch_as_ntw(const PlanView& v, int64_t C, const float* J, int64_t ldj, float* T,
                         int64_t ldt, dust_counters* cnt, hipStream_t st) {
    const size_t lds = sizeof(float) * FUSED_TC * v.Sp + STAGE_BYTES + SOLVE_LDS_BYTES;
    const dim3 grid((unsigned)((C + FUSED_TC - 1) / FUSED_TC));
    const int km = kernel_mode(v);
    if (km == DUST_MIXED)
        hipLaunchKernelGGL((absorb_solve_kernel<DUST_MIXED, NTW>), grid, dim3(256), lds, st, v,
                           C, J, ldj, T, ldt, cnt);
    else if (km == MODE_MIXED_F32)
        hipLaunchKernelGGL((absorb_solve_kernel<MODE_MIXED_F32, NTW>), grid, dim3(256), lds,
                           st, v, C, J, ldj, T, ldt, cnt);
    else if (km == MODE_MIXED_POLISH)
        hipLaunchKernelGGL((absorb_solve_kernel<MODE_MIXED_POLISH, NTW>), grid, dim3(256), lds,
                           st, v, C, J, ldj, T, ldt, cnt);
    else if (v.mode == DUST_TABLE_LINEAR)
        hipLaunchKernelGGL((absorb_solve_kernel<DUST_TABLE_LINEAR, NTW>), grid, dim3(256), lds,
                           st, v, C, J, ldj, T, ldt, cnt);
    else
        hipLaunchKernelGGL((absorb_solve_kernel<DUST_PLAIN_FP32, NTW>), grid, dim3(256), lds, st,
                           v, C, J, ldj, T, ldt, cnt);
    return hipGetLastError();
}

template <int NTW, bool TAIL>
hipError_t launch_ntw(const PlanView& v, int64_t C, const float* J, int64_t ldj, const float* m,
                      float* T, int64_t ldt, float* L, int64_t ldl, dust_counters* cnt,
                      hipStream_t st) {
    const size_t lds = fused_lds_bytes(FUSED_TC, v.Sp, Stage<fused_kc(NTW)>::BYTES);
    const dim3 grid((unsigned)((C + FUSED_TC - 1) / FUSED_TC));
    const int km = kernel_mode(v);
    if (km == DUST_MIXED)
        hipLaunchKernelGGL((fused_kernel<DUST_MIXED, NTW, TAIL>), grid, dim3(256), lds, st, v, C,
                           J, ldj, m, T, ldt, L, ldl, cnt);
    else if (km == MODE_MIXED_F32)
        hipLaunchKernelGGL((fused_kernel<MODE_MIXED_F32, NTW, TAIL>), grid, dim3(256), lds, st,
                           v, C, J, ldj, m, T, ldt, L, ldl, cnt);
    else if (km == MODE_MIXED_POLISH)
        hipLaunchKernelGGL((fused_kernel<MODE_MIXED_POLISH, NTW, TAIL>), grid, dim3(256), lds,
                           st, v, C, J, ldj, m, T, ldt, L, ldl, cnt);
    else if (v.mode == DUST_TABLE_LINEAR)
        hipLaunchKernelGGL((fused_kernel<DUST_TABLE_LINEAR, NTW, TAIL>), grid, dim3(256), lds,
                           st, v, C, J, ldj, m, T, ldt, L, ldl, cnt);
    else
        hipLaunchKernelGGL((fused_kernel<DUST_PLAIN_FP32, NTW, TAIL>), grid, dim3(256), lds, st,
                           v, C, J, ldj, m, T, ldt, L, ldl, cnt);
    return hipGetLastError();
}

template <bool TAIL>
hipError_t launch_fused_as(const PlanView& v, int64_t C, const float* J, int64_t ldj,
                           const float* m, float* T, int64_t ldt, float* L, int64_t ldl,
                           dust_counters* cnt, hipStream_t st) {
    const int ntw = (v.Sp / 16 + 3) / 4;  // grain tiles per wave in one pass
    if (ntw <= 1) return launch_ntw<1, TAIL>(v, C, J, ldj, m, T, ldt, L, ldl, cnt, st);
    if (ntw <= 2) return launch_ntw<2, TAIL>(v, C, J, ldj, m, T, ldt, L, ldl, cnt, st);
    if (ntw <= 3) return launch_ntw<3, TAIL>(v, C, J, ldj, m, T, ldt, L, ldl, cnt, st);
    return launch_ntw<4, TAIL>(v, C, J, ldj, m, T, ldt, L, ldl, cnt, st);  // 4: several passes above
}

// Whether a call runs as heat_solve_kernel and the emission kernel instead of
// one fused kernel.  A fused workgroup takes 16 cells through every phase, so
// up to two workgroups per CU the call takes as long as one tile's chain
// whatever the cell count (968 wavelengths x 81 grains: 106 us for 32 cells,
// 118 for 4099), while the two kernels spread the same work over grain tiles
// and wavelength blocks: 17 us and 70.  At 8192 cells (512 tiles) 125 against
// 148 us, at 16384 228 against 219; 250 x 80 and 1000 x 240 cross at the same
// tile count, a short chain a little earlier (8192 x 200 x 40: 25.6 us fused,
// 26.6 split; 4096: 22.9, 18.1).  Below 6000 grain-wavelengths a tile's chain
// is shorter than the second launch is worth (120 x 20: 11.8 us fused, 14.3
// split; 120 x 40: 15.4 both).
constexpr int64_t SPLIT_TILES = 384, SPLIT_WORK = 6000;
constexpr int64_t SPLIT_TILES_LONG = 512, SPLIT_WORK_LONG = 16000;

bool split_pays(const PlanView& v, int64_t C) {
    const int64_t work = (int64_t)v.S * v.NL;
    return work >= SPLIT_WORK_LONG ? C <= 16 * SPLIT_TILES_LONG
                                   : C <= 16 * SPLIT_TILES && work >= SPLIT_WORK;
}

// Whether a plain call runs as the kernels of its three steps (launch_heat_newton)
// instead of one.  The one kernel's Newton sums, on vector loads, cost up to
// three times those of the solve kernel; the three pay their launches and the
// trips of H' and T through memory.  One kernel against three: 400000 x 80
// grains 857 and 927 us at 24 wavelengths, 937 and 950 at 32, 1145 and 1033 at
// 48; 6000 x 200 80 and 69 us at 24.  Up to 16 grains a tile's solve is one
// round of its threads: 6000 x 16 18.0 and 23.5 us at 100 wavelengths, 30.8 and
// 28.4 at 250; 700 x 16 16.3 and 17.1 at 100, 21.2 and 17.4 at 160; 50000 x 16 37
// and 42 at 32, 49 and 48 at 64; 400000 x 16 209 and 225 at 24, 226 and 223 at 32; x
// 5 156 and 139 at 8.  Few cells of more than 32 grains have
// rounds enough at any length: 40 x 80 28.8 and 21.1 us at 24 wavelengths, 700 x
// 40 18.8 and 17.0.
bool plain_split_pays(const PlanView& v, int64_t C) {
    if (v.S <= 16) return v.NL >= (C < 32768 ? 128 : (C < 262144 ? 64 : (v.S <= 8 ? 8 : 32)));
    return v.NL >= (v.S > 32 && C <= 4096 ? 8 : 32);
}

// The plain fused call as the kernels of its three steps, so that the Newton
// sums run on scalar weights (a fused tile's 16 cells give each lane its own
// grain's, through vector loads: 30001 x 251 x 77 1205 us in one kernel).  The
// scaled heating H' rests in the call's own output until the solve reads it:
// in T, solved in place, or, when T holds the start temperatures, in L.
hipError_t launch_heat_newton(const PlanView& v, int64_t C, const float* J, int64_t ldj, float* T,
                              int64_t ldt, float* L, int64_t ldl, dust_counters* cnt,
                              hipStream_t st) {
    float* H = v.warm ? L : T;
    const int64_t ldh = v.warm ? ldl : ldt;
    const hipError_t e = launch_absorb_scaled(v, C, J, ldj, H, ldh, st);
    return e != hipSuccess ? e : launch_solve_plain(v, C, H, ldh, T, ldt, true, cnt, st);
}

}  // namespace

hipError_t launch_fused(const PlanView& v, int64_t C, const float* J, int64_t ldj, const float* m,
                        float* T, int64_t ldt, float* L, int64_t ldl, dust_counters* cnt,
                        bool one_kernel, hipStream_t st) {
    if (C == 0) return hipSuccess;
    const int64_t nj = (C - 1) * ldj + v.NL, nt = (C - 1) * ldt + v.S, nl = (C - 1) * ldl + v.NL;
    const int64_t nq = (C - 1) * v.ldq + v.S;
    // (the one kernel stores a tile's T before its L, which stays where the two
    // share memory)
    one_kernel = one_kernel || share_memory(T, nt, L, nl);
    if (!one_kernel && !table_mode(v.mode) && plain_split_pays(v, C) &&
        (!v.warm || v.S <= v.NL) &&
        !share_memory(J, nj, T, nt) && !share_memory(J, nj, L, nl) &&
        !(v.q && (share_memory(v.q, nq, T, nt) || share_memory(v.q, nq, L, nl)))) {
        const hipError_t e = launch_heat_newton(v, C, J, ldj, T, ldt, L, ldl, cnt, st);
        return e != hipSuccess ? e : launch_emit(v, C, T, ldt, m, L, ldl, st);
    }
    if (!one_kernel && table_mode(v.mode) && split_pays(v, C) &&
        !share_memory(J, nj, T, nt)) {
        const hipError_t e = rows_aligned16(J, ldj)
                                 ? launch_heat_solve<true>(v, C, J, ldj, T, ldt, cnt, st)
                                 : launch_heat_solve<false>(v, C, J, ldj, T, ldt, cnt, st);
        return e != hipSuccess ? e : launch_emit(v, C, T, ldt, m, L, ldl, st);
    }
    if (((v.S + EMIT_GROUP - 1) / EMIT_GROUP) & 1)
        return launch_fused_as<true>(v, C, J, ldj, m, T, ldt, L, ldl, cnt, st);
    return launch_fused_as<false>(v, C, J, ldj, m, T, ldt, L, ldl, cnt, st);
}

hipError_t launch_absorb_solve(const PlanView& v, int64_t C, const float* J, int64_t ldj,
                               float* T, int64_t ldt, dust_counters* cnt, hipStream_t st) {
    if (C == 0) return hipSuccess;
    const int ntw = (v.Sp / 16 + 3) / 4;
    if (ntw <= 1) return launch_as_ntw<1>(v, C, J, ldj, T, ldt, cnt, st);
    if (ntw <= 2) return launch_as_ntw<2>(v, C, J, ldj, T, ldt, cnt, st);
    if (ntw <= 3) return launch_as_ntw<3>(v, C, J, ldj, T, ldt, cnt, st);
    if (ntw <= 4) return launch_as_ntw<4>(v, C, J, ldj, T, ldt, cnt, st);
    return launch_as_ntw<4>(v, C, J, ldj, T, ldt, cnt, st);  // several passes
}

}  // namespace dust
