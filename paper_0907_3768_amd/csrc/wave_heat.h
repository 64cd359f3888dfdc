// Heating of a few (16 cells, 16 grains) tiles by one wave, straight from device
// memory.
#pragma once

#include "device_common.h"

namespace dust {

// The (CELLS cells, grain tile) pairs of a call as a 1-D grid.  Workgroups go to
// the eight XCDs in turn, so workgroup b's cell block is taken from b mod 8:
// every grain tile of a cell block runs on one XCD and its J rows come from
// that L2 once.
struct HeatTile {
    int64_t c0;  // first cell
    int tile;    // grain tile
};
template <int CELLS>
__device__ __forceinline__ HeatTile heat_tile(unsigned b, int tiles) {
    const unsigned g = b >> 3;
    const unsigned j = g / (unsigned)tiles;
    return HeatTile{((int64_t)j * 8 + (b & 7)) * CELLS, (int)(g - j * (unsigned)tiles)};
}
template <int CELLS>
unsigned heat_blocks(int64_t C, int tiles) {
    return (unsigned)(((C + CELLS - 1) / CELLS + 7) / 8 * 8 * tiles);
}

// Heating of 16 MB cells x 16 NB grains by one wave, straight from device
// memory.  Element r of acc[mb][nb] in lane (row = lane mod 16, kq = lane / 16)
// is the scaled heating H' of cell c0 + 16 mb + 4 kq + r and grain
// 16 (tile + nb) + row.
//
// Lane (row, kq) loads wavelengths k0 + 8 kq .. + 7 of cell row `row` (two
// 16-byte loads where ALIGNED: J and its rows on 16 bytes) and its eight
// values of the weight fragment, U k-steps ahead of their MFMAs: with a
// wave or less per SIMD nothing else hides the loads.  The products and their
// order are those of fused_absorb, so H' is the same bit for bit.  Rows past
// the last cell read cell C - 1 again and tiles past the last grain tile read
// that one again; an MFMA's output depends on its own row and column of the
// inputs only, and those are not used.
template <bool BF, bool ALIGNED, int MB, int NB, int U>
__device__ __forceinline__ void heat_block(const PlanView& v, int64_t c0, int64_t C, int tile,
                                           const float* __restrict__ J, int64_t ldj,
                                           f32x4 (&acc)[MB][NB]) {
    const int lane = threadIdx.x & 63;
    const int row = lane & 15, kq = lane >> 4;
    const int nsteps = v.NLp / 32, nfull = v.NL / 32, tiles = v.Sp / 16;
    const float* jr[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int64_t c = c0 + 16 * m + row;
        jr[m] = J + (c < C ? c : C - 1) * ldj + 8 * kq;
    }
    struct Step {
        float x[MB][8];
        bf16x8 hi[NB], lo[NB];     // weights: bf16 hi and lo,
        float4 f0[NB], f1[NB];     // or FP32
    };
    auto load_k = [&](int step, Step& st) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const int t = tile + n < tiles ? tile + n : tiles - 1;
            const int64_t fr = (int64_t)t * nsteps + step;
            if constexpr (BF) {
                const int64_t o = (fr * 64 + lane) * 8;
                st.hi[n] = *reinterpret_cast<const bf16x8*>(v.khi + o);
                st.lo[n] = *reinterpret_cast<const bf16x8*>(v.klo + o);
            } else {
                const int64_t o = (fr * 128 + lane) * 4;
                st.f0[n] = *reinterpret_cast<const float4*>(v.kf + o);
                st.f1[n] = *reinterpret_cast<const float4*>(v.kf + o + 256);
            }
        }
    };
    auto load_full = [&](int step, Step& st) {  // step < nfull
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const float* p = jr[m] + 32 * step;
            if constexpr (ALIGNED) {
                const float4 a = *reinterpret_cast<const float4*>(p);
                const float4 b = *reinterpret_cast<const float4*>(p + 4);
                st.x[m][0] = a.x; st.x[m][1] = a.y; st.x[m][2] = a.z; st.x[m][3] = a.w;
                st.x[m][4] = b.x; st.x[m][5] = b.y; st.x[m][6] = b.z; st.x[m][7] = b.w;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) st.x[m][e] = p[e];
            }
        }
        load_k(step, st);
    };
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const Step& st) {
        if constexpr (BF) {
            bf16x8 ahi[MB], alo[MB];
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const __bf16 h = (__bf16)st.x[m][e];
                    ahi[m][e] = h;
                    alo[m][e] = (__bf16)(st.x[m][e] - (float)h);
                }
            // each product over every accumulator before the next: consecutive
            // MFMAs are independent
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[m], st.hi[n], acc[m][n], 0, 0, 0);
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[m], st.lo[n], acc[m][n], 0, 0, 0);
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo[m], st.hi[n], acc[m][n], 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int m = 0; m < MB; ++m)
#pragma unroll
                    for (int n = 0; n < NB; ++n) {
                        const float4 f = e < 4 ? st.f0[n] : st.f1[n];
                        const int q = e & 3;
                        const float b = q == 0 ? f.x : (q == 1 ? f.y : (q == 2 ? f.z : f.w));
                        acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(st.x[m][e], b, acc[m][n], 0, 0, 0);
                    }
        }
    };
    Step cur[U], nxt[U];
    const int groups = nfull / U;
    if (groups > 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) load_full(u, cur[u]);
    }
    for (int g = 0; g < groups; ++g) {
        // past the last group, that group again (in bounds, not used)
        const int s = (g + 1 < groups ? g + 1 : g) * U;
#pragma unroll
        for (int u = 0; u < U; ++u) load_full(s + u, nxt[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) multiply(cur[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) cur[u] = nxt[u];
    }
    // what is left: up to U - 1 full steps and a ragged one (J zero past NL)
    const int left = groups * U;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (left + u < nfull) {
            load_full(left + u, cur[u]);
        } else if (left + u < nsteps) {
            const int k = 32 * (left + u) + 8 * kq;
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    cur[u].x[m][e] = k + e < v.NL ? jr[m][32 * (left + u) + e] : 0.0f;
            load_k(left + u, cur[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (left + u < nsteps) multiply(cur[u]);
}

// Whether J's rows start on 16 bytes.
inline bool rows_aligned16(const float* J, int64_t ldj) {
    return ((uintptr_t)J & 15u) == 0 && (ldj & 3) == 0;
}

}  // namespace dust
