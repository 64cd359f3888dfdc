// Cell SED, Eqs. 9-10 (Section 4.4):
//   L[c,l] = m[c] sum_s w_s C[s,l] B(lam_l, T[c,s]).
// A workgroup owns TC cells and a column of consecutive blocks of 32
// wavelengths; a wave takes one block at a time, its lanes 32 wavelengths x 2
// rows of grain groups, each lane TC partial sums (emit_block), and the rows'
// sums are added across lanes before the store.  The tile's 1/T sits in LDS;
// the emission weights em[s,l] are read once per grain and reused for the
// tile's cells.  An exact term is one multiply, v_exp_f32, one subtract,
// v_rcp_f32 and one FMA.  The order of every sum is the same whatever the
// tile and the column, so every form gives the same bits.
#include "device_common.h"

namespace dust {
namespace {

// Workgroups from which on a call's tiles are not split into wavelength columns
// (16 per CU; the fill of a tile's 1/T is shared by its whole column).
constexpr int64_t EMIT_WORKGROUPS = 4096;
// Grains up to which a column's work is short beside its start: two rounds of
// the waves at least, once such columns are three workgroups per CU (50000 x 250
// x 16 39.2 us in two columns, 37.3 in one; 6000 x 600 x 2 13.0 in five, 11.8 in
// three; but 6000 x 250 x 16 10.1 in two, 11.6 in one, and 3000 x 1000 x 16 13.0
// in eight, 15.1 in four).  Above 16 grains that holds up to 24 blocks (6000 x 600
// x 24 20.6 us in five columns, 19.2 in three; x 1000 27.5 in eight, 29.0 in four).
constexpr int EMIT_FEW_GRAINS = 32;
constexpr int64_t EMIT_FEW_WORKGROUPS = 768;

template <int TC, bool TAIL>
__global__ __launch_bounds__(256) void emit_kernel(PlanView v, int64_t C,
                                                   const float* __restrict__ T, int64_t ldt,
                                                   const float* __restrict__ m,
                                                   float* __restrict__ L, int64_t ldl, int bpc) {
    extern __shared__ float smem[];  // sInvT [TC][Sp], then sChunk [Sp/4][TC]
    float* sInvT = smem;
    uint32_t* sChunk = reinterpret_cast<uint32_t*>(smem + TC * v.Sp);
    const int64_t c0 = (int64_t)blockIdx.x * TC;
    for (int i = threadIdx.x; i < TC * v.Sp; i += 256) {
        const int cc = i / v.Sp, s = i - cc * v.Sp;
        sInvT[i] = (c0 + cc < C && s < v.S) ? inv_temperature(T[(c0 + cc) * ldt + s])
                                             : __builtin_inff();
    }
    __syncthreads();
    fill_chunk_min<TC>(sInvT, sChunk, v.Sp);
    __syncthreads();
    // Workgroup column y owns the wavelength blocks [y bpc, (y + 1) bpc); wave
    // w takes the column's blocks w, w + 4, ....  Grids with fewer than four
    // blocks (one column, 16-cell tiles) split the tile's cells over the waves.
    constexpr int LW = 64 / EMIT_ROWS;
    const int NB = (v.NL + LW - 1) / LW;
    if (TC < 16 || NB >= 4) {
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int b0 = (int)blockIdx.y * bpc;
        emit_tile<EMIT_ROWS, TC, TAIL>(v, c0, C, m, L, ldl, sInvT, sChunk, b0 + w, 4,
                                       b0 + bpc < NB ? b0 + bpc : NB);
    } else if constexpr (TC >= 16) {
        if (v.NL > 64)
            emit_cell_part<TC / 2, TC>(v, c0, C, m, L, ldl, sInvT, sChunk, 2);
        else
            emit_cell_part<TC / 4, TC>(v, c0, C, m, L, ldl, sInvT, sChunk, 1);
    }
}

// Blocks per column: as few columns as give EMIT_WORKGROUPS workgroups, each of
// whole rounds of the four waves.
int column_blocks(int64_t tiles, int NB, int S) {
    const int64_t want = (EMIT_WORKGROUPS + tiles - 1) / tiles;
    const int cols = want < NB ? (int)want : NB;
    const int bpc = ((NB + cols - 1) / cols + 3) / 4 * 4;
    const bool few = (S <= 16 || (S <= EMIT_FEW_GRAINS && NB <= 24)) &&
                     tiles * ((NB + 7) / 8) >= EMIT_FEW_WORKGROUPS;
    return few && bpc < 8 ? 8 : bpc;
}

template <int TC>
hipError_t launch_emit_tc(const PlanView& v, int64_t C, const float* T, int64_t ldt,
                          const float* m, float* L, int64_t ldl, int bpc, hipStream_t st) {
    const int64_t tiles = (C + TC - 1) / TC;
    const int NB = (v.NL + 31) / 32;
    const dim3 grid((unsigned)tiles, (unsigned)((NB + bpc - 1) / bpc));
    const size_t lds = emit_lds_bytes(TC, v.Sp);
    if (((v.S + EMIT_GROUP - 1) / EMIT_GROUP) & 1)
        hipLaunchKernelGGL((emit_kernel<TC, true>), grid, dim3(256), lds, st, v, C, T, ldt, m, L,
                           ldl, bpc);
    else
        hipLaunchKernelGGL((emit_kernel<TC, false>), grid, dim3(256), lds, st, v, C, T, ldt, m, L,
                           ldl, bpc);
    return hipGetLastError();
}

}  // namespace

// Cells per tile, by the number of (16 cells, 32 wavelengths) tasks a call
// has.  Where they do not fill the chip's 6144 wave slots (256 CUs x 4 SIMDs
// x 6) the call takes as long as one wave's chain of S x 16 cells, and smaller
// tiles shorten it: 32 cells x 968 wavelengths x 81 grains 36 us with 16-cell
// tiles in columns of eight blocks, 8.8 us with four-cell tiles (then bound by
// the launch); 4099 cells 58.7 -> 51 us, 2048 x 1000 x 240 103 -> 67 us.  Up
// to twelve rounds of the slots the last, partly filled round is what larger
// tiles lose: 20000 x 600 x 240 352 us with 16 cells, 326 with eight (323 with
// four), 32768 x 968 x 81 319 -> 311.  Beyond, 16 cells read the weights least
// (1048576 x 500 x 128: 7.05 ms in one column against 7.42 in two), and so do
// grids of few grains, whose chain is short and whose fill weighs more (20000
// x 150 x 12: 14.4 us, 15.6 with four cells).
constexpr int64_t EMIT_SLOTS = 6144;

hipError_t launch_emit(const PlanView& v, int64_t C, const float* T, int64_t ldt,
                       const float* m, float* L, int64_t ldl, hipStream_t st) {
    if (C == 0) return hipSuccess;
    const int NB = (v.NL + 31) / 32;
    const int64_t tasks = (C + 15) / 16 * NB;
    // T and L in one piece of memory (L over T, or rows side by side): a tile's
    // 256 wavelengths belong to one workgroup, which has read the tile's T
    // before it writes them
    if (share_memory(T, (C - 1) * ldt + v.S, L, (C - 1) * ldl + v.NL))
        return launch_emit_tc<16>(v, C, T, ldt, m, L, ldl, 256 / 32, st);
    if (NB >= 4 && v.S > 32 && tasks <= EMIT_SLOTS * 3 / 2)
        return launch_emit_tc<4>(v, C, T, ldt, m, L, ldl, column_blocks((C + 3) / 4, NB, v.S), st);
    if (NB >= 4 && v.S > 32 && tasks <= EMIT_SLOTS * 12)
        return launch_emit_tc<8>(v, C, T, ldt, m, L, ldl, column_blocks((C + 7) / 8, NB, v.S), st);
    return launch_emit_tc<16>(v, C, T, ldt, m, L, ldl, column_blocks((C + 15) / 16, NB, v.S), st);
}

}  // namespace dust
