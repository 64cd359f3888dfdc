// Heating of 16 cells x 16 grains by one wave, straight from device memory.
#pragma once

#include "device_common.h"

namespace dust {

// The (CELLS cells, 16 grains) tiles of a call as a 1-D grid.  Workgroups go to
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

// Element r of the result in lane (row = lane mod 16, kq = lane / 16) is the
// scaled heating H' of cell c0 + 4 kq + r and grain 16 tile + row.
//
// Lane (row, kq) loads wavelengths k0 + 8 kq .. + 7 of cell row `row` (two
// 16-byte loads where ALIGNED: J and its rows on 16 bytes) and its eight
// values of the weight fragment, U k-steps ahead of their MFMAs: with a
// wave or less per SIMD nothing else hides the loads.  The products and their
// order are those of fused_absorb, so H' is the same bit for bit.  Rows past
// the last cell read cell C - 1 again; an MFMA's output row depends on its own
// input row only, and those rows are not used.
template <bool BF, bool ALIGNED, int U>
__device__ __forceinline__ f32x4 heat_wave(const PlanView& v, int64_t c0, int64_t C, int tile,
                                           const float* __restrict__ J, int64_t ldj) {
    const int lane = threadIdx.x & 63;
    const int row = lane & 15, kq = lane >> 4;
    const int nsteps = v.NLp / 32, nfull = v.NL / 32;
    const int64_t c = c0 + row < C ? c0 + row : C - 1;
    const float* jr = J + c * ldj + 8 * kq;
    struct Step {
        float x[8];
        bf16x8 hi, lo;     // weights: bf16 hi and lo,
        float4 f0, f1;     // or FP32
    };
    auto load_k = [&](int step, Step& st) {
        const int64_t fr = (int64_t)tile * nsteps + step;
        if constexpr (BF) {
            const int64_t o = (fr * 64 + lane) * 8;
            st.hi = *reinterpret_cast<const bf16x8*>(v.khi + o);
            st.lo = *reinterpret_cast<const bf16x8*>(v.klo + o);
        } else {
            const int64_t o = (fr * 128 + lane) * 4;
            st.f0 = *reinterpret_cast<const float4*>(v.kf + o);
            st.f1 = *reinterpret_cast<const float4*>(v.kf + o + 256);
        }
    };
    auto load_full = [&](int step, Step& st) {  // step < nfull
        const float* p = jr + 32 * step;
        if constexpr (ALIGNED) {
            const float4 a = *reinterpret_cast<const float4*>(p);
            const float4 b = *reinterpret_cast<const float4*>(p + 4);
            st.x[0] = a.x; st.x[1] = a.y; st.x[2] = a.z; st.x[3] = a.w;
            st.x[4] = b.x; st.x[5] = b.y; st.x[6] = b.z; st.x[7] = b.w;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) st.x[e] = p[e];
        }
        load_k(step, st);
    };
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const Step& st) {
        if constexpr (BF) {
            bf16x8 ahi, alo;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const __bf16 h = (__bf16)st.x[e];
                ahi[e] = h;
                alo[e] = (__bf16)(st.x[e] - (float)h);
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, st.hi, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, st.lo, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo, st.hi, acc, 0, 0, 0);
        } else {
            const float b[8] = {st.f0.x, st.f0.y, st.f0.z, st.f0.w,
                                st.f1.x, st.f1.y, st.f1.z, st.f1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(st.x[e], b[e], acc, 0, 0, 0);
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
            for (int e = 0; e < 8; ++e) cur[u].x[e] = k + e < v.NL ? jr[32 * (left + u) + e] : 0.0f;
            load_k(left + u, cur[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (left + u < nsteps) multiply(cur[u]);
    return acc;
}

// Whether J's rows start on 16 bytes.
inline bool rows_aligned16(const float* J, int64_t ldj) {
    return ((uintptr_t)J & 15u) == 0 && (ldj & 3) == 0;
}

}  // namespace dust
