// Plan-time kernels: the derived tables of a grid.
//
//  prep  (the paper's first kernel, Section 4.1): K = C dlam per grain and
//        wavelength, scaled per grain by an exact power of two, in FP32 and as
//        a bf16 hi+lo pair (both in MFMA fragment order); the solve weights K' c1 lam^-5; the emission
//        weights w C c1 lam^-5 (Eq. 10 without the mass); the wavelength
//        exponent table nu = -c2 log2(e) / lam.
//  ltab  (mixed mode): per grain, y_k = ln P'(T_k) at log-spaced T_k, in
//        FP64, with P'(T) = sum_l K'_l B(lam_l, T) the right side of Eq. 7 in
//        the plan's scaled units -- as an FP64 matrix product (MFMA) of the
//        grains' Planck weights with the Planck factors of the table
//        temperatures, which the product computes as it goes.
//  inv   (mixed mode): the inverse function ln T(y) and its derivative at
//        uniform steps of y, from Newton in FP64 on the forward table's
//        piecewise cubic, stored as FP64 nodes and as FP32 pairs of nodes (one
//        16-byte load per lookup).  A second, smaller pair of tables below the
//        range makes the lookups of colder grains.
//  plain: the same product at a few log-spaced T (y_k only), where Newton's
//        first iterations run.
//  table-linear mode: the same matrix product gives P'(T_k) itself at evenly
//        spaced T_k (the production table of Sections 2 and 5); kidx gives,
//        at uniform steps of ln P', the last table point below, so that a
//        lookup searches only a few points.
#include <math.h>

#include "device_common.h"

namespace dust {
namespace {

__device__ __forceinline__ void prep_body(const RefreshJob& j, int bx, int by) {
    const PlanView& v = j.v;
    const double* __restrict__ lam = j.lam;
    const double* __restrict__ dlam = j.dlam;
    const double* __restrict__ cabs = j.cabs;
    const double* __restrict__ w = j.w;
    const int* __restrict__ es = j.es;
    const int ge = j.ge;
    float* nu = j.nu; float* kf = j.kf; float* kb = j.kb; float* ku = j.ku; float* em = j.em;
    __bf16* khi = j.khi; __bf16* klo = j.klo;
    double* kdb = j.kdb; double* c2l = j.c2l;
    const int l = bx * blockDim.x + threadIdx.x;
    const int s = by;
    if (l >= v.NLp) return;
    const int64_t o = (int64_t)s * v.NLp + l;
    // The heating weights are stored in MFMA fragment order, so that one
    // wave's fragment of one grain tile and k-step is a contiguous 1 KB.
    const int64_t ob = kfrag_bf16(v, s, l), of = kfrag_f32(v, s, l);
    if (s == 0) {
        // (padding repeats the last: its terms have zero weight and stay finite)
        nu[l] = (float)(-RAD_C2 * LOG2E / lam[l < v.NL ? l : v.NL - 1]);
        if (l < v.NL) c2l[l] = RAD_C2 / lam[l];
    }
    if (s < v.S && l < v.NL) {
        const double C = cabs[(int64_t)s * v.NL + l];
        const double K = ldexp(C * dlam[l], es[s]);
        const double lm = lam[l];
        const double c1l5 = RAD_C1 / (lm * lm * lm * lm * lm);
        const float kff = (float)K;
        const __bf16 hi = (__bf16)kff;
        const __bf16 lo = (__bf16)(float)(K - (double)(float)hi);
        kf[of] = kff;
        khi[ob] = hi;
        klo[ob] = lo;
        kb[o] = (float)(K * c1l5);
        ku[o] = (float)(K * c1l5 * (RAD_C2 * LOG2E / lm));
        em[o] = (float)ldexp(w[s] * C * c1l5, -ge);
        kdb[(int64_t)s * v.NL + l] = K * c1l5;
    } else {
        kf[of] = 0.0f;
        khi[ob] = (__bf16)0.0f;
        klo[ob] = (__bf16)0.0f;
        kb[o] = 0.0f;
        ku[o] = 0.0f;
        em[o] = 0.0f;
    }
}

// The table is a matrix product:  P'[s,k] = sum_l W[s,l] F[k,l]  with
// W = K' c1 lam^-5 (per grain) and F[k,l] = 1 / (exp(c2 / (lam_l T_k)) - 1)
// (per table temperature, the same for every grain).

// y[s][k] = ln sum_l W[s][l] F[k][l] (table-linear: the sum itself): an FP64
// product on the matrix cores (v_mfma_f64_16x16x4_f64) whose F operand is
// computed in registers and never stored.  The 16-wavelength steps of a block of
// 16 points and up to LT_TILES grain tiles of 16 are split into shares (share w
// of n takes steps w, w + n, ...; n by the number of wavelengths) whose partial
// sums meet in LDS.  Per step, lane (row = lane mod 16, q = lane / 16)
// computes F for point row and wavelengths l0 + 4 q .. + 3 (four FP64
// exponentials), loads the same wavelengths of each grain tile's row of W
// (contiguous 32 bytes) and issues four MFMAs per tile; MFMA t takes the
// t-th wavelength of both operands (any assignment of wavelengths to k-slots
// gives the same sum when both operands use it).  Element j of a tile's
// accumulator in lane (col, q) holds grain row q + 4 j of point col (the
// FP64 form interleaves rows).
//
// What bounds it is a wave's chain of exponentials and dependent MFMAs (FP64
// ones, which take as long as the vector unit's), so a single plan's shares take
// a wave each, up to eight; there, and for a plan with many grains, a wave
// shares its exponentials among several tiles (product_tiles).  Where many plans
// share a launch workgroups have four waves as a rule (long_product), which take eight shares two by
// two, and fewer shares (up to LT_SHORT wavelengths each) leave waves to other
// point blocks: each wave's start (1/T, addresses, the sums' meeting) is as
// long as a step or two.  The sums are added in one order for each number of
// shares, so every launch makes the same table bit for bit.
// A refresh of all three stages, with four waves, 32 wavelengths a step and one
// tile, and now: 250 x 80 19.6 -> 15.8 us, 968 x 81 42 -> 27, 1000 x 240 62 -> 46,
// table-linear 1000 x 240 116 -> 62.  Many plans, with one wave that has the whole
// range and four tiles, with eight waves and eight shares whatever the length,
// and now: 64 of 100 - 600 wavelengths x 10 - 240 grains 372, 341, 331 us, 300 of
// 40 x 80 435, 648, 451, 700 of 130 x 16 334, 631, 447 (a wave with the whole
// range 381, but 250 x 80 alone 22.6; a sixth is the table below the range).
// Weights loaded before the exponentials cost the registers of a wave per SIMD
// (1000 x 240: 55 us).
constexpr int LT_WAVES = 8, LT_TILES = 4, LT_STEP = 16;
constexpr int LT_SHORT = 48;

// Shares of a product over NL wavelengths.
__host__ __device__ inline int product_shares(int NL) {
    return NL <= LT_SHORT ? 1 : (NL <= 2 * LT_SHORT ? 2 : (NL <= 4 * LT_SHORT ? 4 : LT_WAVES));
}
// Point blocks per workgroup: of four waves, each with a share of one.
__host__ __device__ inline int product_blocks(int NL) {
    const int n = product_shares(NL);
    return n < 4 ? 4 / n : 1;
}

// Grain tiles per workgroup of the product for `blocks` (16-point block, grain
// tile) pairs in one launch: one as long as the GPU has a place for each
// workgroup at once (two per CU).  A refresh of 968 x 81 (432 pairs) takes 30.3
// us with one, 29.4 with two, 36.7 with four; of 500 x 128 (576) 24.4 with two,
// 25.3 with four.
constexpr int64_t LT_PAIRS = 512;
int product_tiles(int64_t blocks) {
    return blocks <= LT_PAIRS ? 1 : (blocks <= 2 * LT_PAIRS ? 2 : LT_TILES);
}

// 1/T of table point k: the N points of the table's range, then the Nc points
// below it (mixed); 0 past the last.
__device__ __forceinline__ double point_inv_T(const RefreshJob& j, int k) {
    const PlanView& v = j.v;
    if (k >= v.N + j.Nc) return 0.0;
    if (k >= v.N) return exp(-(j.lnTmin_c + (k - v.N) * j.hstep_c));
    return v.mode == DUST_TABLE_LINEAR ? 1.0 / v.texp[k] : exp(-(v.lnTmin + k * v.hstep));
}

// The product's result for grain s and point k.
__device__ __forceinline__ void store_point(const RefreshJob& j, int s, int k, double P) {
    const PlanView& v = j.v;
    if (k < v.N)
        j.fwd[(int64_t)s * v.N + k] = v.mode == DUST_TABLE_LINEAR ? P : log(P);
    else
        j.fwd_c[(int64_t)s * j.Nc + (k - v.N)] = log(P);
}

template <int WAVES>
__device__ __forceinline__ void product_body(const RefreshJob& j, int bx, int by) {
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    constexpr int SLOTS = 4, NF = LT_STEP / 4;
    static_assert(LT_WAVES == 2 * SLOTS && (WAVES == SLOTS || WAVES == LT_WAVES), "eight shares");
    // (eight waves: four of them are left over where there are four shares or fewer)
    __shared__ f64x4 part[SLOTS][LT_TILES][64];
    const PlanView& v = j.v;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, q = lane >> 4;
    const int n = product_shares(v.NL);     // uniform
    const int per = n < SLOTS ? n : SLOTS;  // slots of a point block
    const int blocks = product_blocks(v.NL);
    const int tiles = (v.S + 15) / 16 - by * j.lt_tiles;
    const int nt = tiles < j.lt_tiles ? tiles : j.lt_tiles;
    const int s0 = by * j.lt_tiles * 16;
    f64x4 acc[LT_TILES];
    // the sums of share w for the 16 points from k0
    auto share = [&](int w, int k0) {
        const double invT = point_inv_T(j, k0 + row);
        const bool k_ok = k0 + row < v.N + j.Nc;
#pragma unroll
        for (int t = 0; t < LT_TILES; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
        for (int l0 = LT_STEP * w; l0 < v.NL; l0 += LT_STEP * n) {
            const int lq = l0 + NF * q;
            double f[NF];
#pragma unroll
            for (int t = 0; t < NF; ++t) {
                const int l = lq + t < v.NL ? lq + t : v.NL - 1;
                const double em = expm1_pos(v.c2l[l] * invT);
                // 0 once e^x overflows, and past the last wavelength or point
                f[t] = (em < __builtin_inf() && lq + t < v.NL && k_ok) ? rcp_f64(em) : 0.0;
            }
#pragma unroll
            for (int st = 0; st < LT_TILES; ++st) {
                if (st >= nt) break;  // uniform
                const int s = s0 + 16 * st + row;
                const double* wr = v.kdb + (int64_t)(s < v.S ? s : v.S - 1) * v.NL;
                double a[NF];
                if (l0 + LT_STEP <= v.NL) {  // uniform
#pragma unroll
                    for (int t = 0; t < NF; ++t) a[t] = wr[lq + t];
                } else {
#pragma unroll
                    for (int t = 0; t < NF; ++t) a[t] = wr[lq + t < v.NL ? lq + t : v.NL - 1];
                }
#pragma unroll
                for (int t = 0; t < NF; ++t)
                    acc[st] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], f[t], acc[st], 0, 0, 0);
            }
        }
    };
    auto put = [&](int slot) {
#pragma unroll
        for (int st = 0; st < LT_TILES; ++st)
            if (st < nt) part[slot][st][lane] = acc[st];
    };
    auto add = [&](int slot) {
#pragma unroll
        for (int st = 0; st < LT_TILES; ++st)
            if (st < nt) acc[st] += part[slot][st][lane];
    };
    // of eight shares, share w + 4 hands its sums to share w
    if (WAVES == LT_WAVES && n == LT_WAVES) {  // uniform
        share(wave, 16 * bx);
        if (wave >= SLOTS) put(wave - SLOTS);
        __syncthreads();
        if (wave < SLOTS) {
            add(wave);
            put(wave);
        }
    } else if (n > SLOTS) {  // (each lane meets its own values)
        share(wave + SLOTS, 16 * bx);
        put(wave);
        share(wave, 16 * bx);
        add(wave);
        put(wave);
    } else if (WAVES == SLOTS || wave < SLOTS) {
        share(wave & (n - 1), 16 * (bx * blocks + wave / n));
        put(wave);
    }
    __syncthreads();
    for (int i = wave; i < blocks * nt; i += WAVES) {
        const int pb = i / nt, st = i - pb * nt;
        const f64x4* p = &part[pb * per][st][lane];
        constexpr int NEXT = LT_TILES * 64;  // the next slot
        f64x4 sum = p[0];
        if (per > 1) sum += p[NEXT];
        if (per > 2) sum += p[2 * NEXT] + p[3 * NEXT];
        const int k = 16 * (bx * blocks + pb) + row;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const int sr = s0 + 16 * st + q + 4 * jj;
            if (sr < v.S && k < v.N + j.Nc) store_point(j, sr, k, sum[jj]);
        }
    }
}

// A grain's forward row for the searches below: in LDS up to FWD_LDS points
// (a search is ten or more reads, each waiting for the one before), in place
// above.  The caller's whole block takes part.
constexpr int FWD_LDS = 2048;

template <bool LOG>
__device__ __forceinline__ const double* stage_row(const double* f, int N, double* sF) {
    if (N > FWD_LDS) return f;  // uniform
    for (int i = threadIdx.x; i < N; i += blockDim.x) sF[i] = LOG ? log(f[i]) : f[i];
    __syncthreads();
    return sF;
}

// Table-linear: one thread per (grain, node); node j sits at
// ln P' = ylo + j (yhi - ylo) / (M - 1) and kidx[s][j] is the largest k in
// [0, N-2] with ln P'_k <= that value (0 if none).
__device__ __forceinline__ void kidx_body(const RefreshJob& job, int bx, int by, double* sF) {
    const PlanView& v = job.v;
    const double* __restrict__ fwd = job.fwd;
    int* kidx = job.kidx;
    double* ylo = job.ylo; double* yhi = job.yhi; double* dyinv = job.dyinv;
    const int j = bx * blockDim.x + threadIdx.x;
    const int s = by;
    const int N = v.N;
    const double* P = fwd + (int64_t)s * N;
    const double* y = stage_row<true>(P, N, sF);
    if (j >= v.M) return;
    const bool staged = N <= FWD_LDS;
    const double y0 = log(P[0]), y1 = log(P[N - 1]);
    const double dinv = (v.M - 1) / (y1 - y0);
    if (j == 0) {
        ylo[s] = y0;
        yhi[s] = y1;
        dyinv[s] = dinv;
    }
    const double yj = (j == v.M - 1) ? y1 : y0 + j / dinv;
    int lo = 0, hi = N - 2;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((staged ? y[mid] : log(P[mid])) <= yj) lo = mid; else hi = mid - 1;
    }
    kidx[(int64_t)s * v.M + j] = lo;
}

// ln T at y (>= f[0]) by Newton on the piecewise cubic through a forward table
// of N values f[0], f[ST], ... at ln T = lnT0 + k h, and d ln T / dy there.
template <int ST>
__device__ __forceinline__ double2 inverse_node(const double* __restrict__ f, int N, double lnT0,
                                                double h, double y) {
    // largest k in [0, N-2] with f_k <= y
    int lo = 0, hi = N - 2;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (f[ST * mid] <= y) lo = mid; else hi = mid - 1;
    }
    const int j0 = stencil_start(lo, N);
    const double a0 = f[ST * j0], a1 = f[ST * (j0 + 1)], a2 = f[ST * (j0 + 2)],
                 a3 = f[ST * (j0 + 3)];
    const double fl = f[ST * lo], fh = f[ST * (lo + 1)];
    double x = lo - j0 + (fh > fl ? (y - fl) / (fh - fl) : 0.0);
    double dp = 1.0;
    for (int it = 0; it < 4; ++it) {
        const double p = cubic4(x, a0, a1, a2, a3, &dp);
        x -= (p - y) / dp;
    }
    cubic4(x, a0, a1, a2, a3, &dp);
    return make_double2(lnT0 + ((double)j0 + x) * h, h / dp);
}

// One thread per (grain, inverse node): ln T at y_j = ylo + j dy and
// dy * d ln T / dy.
__device__ __forceinline__ void inv_body(const RefreshJob& job, int bx, int by, double* sF) {
    const PlanView& v = job.v;
    const int s = by, M = v.M, N = v.N;
    const int j = bx * blockDim.x + threadIdx.x;
    const double* f = stage_row<false>(job.fwd + (int64_t)s * N, N, sF);
    if (j >= M) return;
    const double y0 = f[0], y1 = f[N - 1];
    const double dinv = (M - 1) / (y1 - y0);
    if (j == 0) {
        job.ylo[s] = y0;
        job.yhi[s] = y1;
        job.dyinv[s] = dinv;
        job.ylof[s] = (float)y0;
        job.dyinvf[s] = (float)dinv;
    }
    const double yj = (j == M - 1) ? y1 : y0 + j / dinv;
    double2 node = inverse_node<1>(f, N, v.lnTmin, v.hstep, yj);
    node.y /= dinv;  // the derivative, scaled by the node spacing dy = 1 / dinv
    job.invd[(int64_t)s * M + j] = node;
    // the FP32 entries of the two intervals this node bounds
    const float2 nf = make_float2((float)node.x, (float)node.y);
    float2* row = job.invf + (int64_t)s * (M - 1) * 2;
    if (j < M - 1) row[2 * j] = nf;
    if (j > 0) row[2 * (j - 1) + 1] = nf;
}

// The same below the table's range, by one workgroup per grain: the nodes from
// every other forward point, then the table's ln T at the points between.
__device__ __forceinline__ void cold_inv_body(const RefreshJob& job, int s, double* sF) {
    static_assert(COLD_P + 2 * COLD_M <= FWD_LDS, "forward points and nodes in LDS");
    const int j = threadIdx.x;
    const double* f = stage_row<false>(job.fwd_c + (int64_t)s * COLD_P, COLD_P, sF);
    double2* nodes = reinterpret_cast<double2*>(sF + COLD_P + 1);
    const double y0 = f[0], y1 = f[COLD_P - 1];
    const double dinv = (COLD_M - 1) / (y1 - y0);
    if (j < COLD_M) {
        const double yj = (j == COLD_M - 1) ? y1 : y0 + j / dinv;
        double2 node = inverse_node<2>(f, COLD_N, job.lnTmin_c, 2.0 * job.hstep_c, yj);
        node.y /= dinv;
        nodes[j] = node;
        job.inv_c[(int64_t)s * COLD_M + j] = node;
    }
    __syncthreads();
    bool good = true;  // (a table that is not finite fails)
    if (j < COLD_N - 1) {
        const int k = 2 * j + 1;
        const double u = fmin(fmax((f[k] - y0) * dinv, 0.0), (double)(COLD_M - 1));
        const int i = (int)u < COLD_M - 2 ? (int)u : COLD_M - 2;
        good = fabs(hermite_lnT(nodes + i, u, i) - (job.lnTmin_c + k * job.hstep_c)) <= COLD_TOL;
    }
    const int bad = __syncthreads_or(!good);
    if (j == 0) {
        job.ylo_c[s] = y0;
        job.dyinv_c[s] = bad ? __builtin_nan("") : dinv;
    }
}

// The stages of a refresh (0 prep, 2 table product, 3 inverse table or search
// brackets; stage 1 is empty since the product computes its Planck factors
// itself): one block of a stage's grid.
template <int STAGE, int WAVES>
__device__ __forceinline__ void refresh_stage(const RefreshJob& j, int bx, int by) {
    if constexpr (STAGE == 0) {
        prep_body(j, bx, by);
    } else if constexpr (STAGE == 2) {
        product_body<WAVES>(j, bx, by);
    } else {
        __shared__ __align__(16) double sF[FWD_LDS];
        if (j.v.mode == DUST_TABLE_LINEAR) kidx_body(j, bx, by, sF);
        else if (bx == j.gx[3] - 1) cold_inv_body(j, by, sF);
        else inv_body(j, bx, by, sF);
    }
}

// One plan: the job by value, the stage's 2-D grid.
template <int STAGE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void refresh_kernel(RefreshJob j) {
    refresh_stage<STAGE, WAVES>(j, blockIdx.x, blockIdx.y);
}

// Many plans in one launch: the flat block index is located among the plans'
// consecutive ranges (starts[p] = first block of plan p, ascending) and
// unfolded into that plan's 2-D grid of x extent gx.
template <int STAGE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void refresh_batched_kernel(
    const RefreshJob* __restrict__ jobs, const int* __restrict__ starts, int n_jobs) {
    const int b = blockIdx.x;
    int lo = 0, hi = n_jobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (starts[mid] <= b) lo = mid; else hi = mid - 1;
    }
    const RefreshJob& j = jobs[lo];
    const int local = b - starts[lo];
    const int gx = j.gx[STAGE];
    refresh_stage<STAGE, WAVES>(j, local % gx, local / gx);
}

template <int STAGE, int WAVES = 4>
hipError_t launch_stage(const RefreshJob& j, hipStream_t st) {
    hipLaunchKernelGGL((refresh_kernel<STAGE, WAVES>), dim3(j.gx[STAGE], j.gy[STAGE]),
                       dim3(64 * WAVES), 0, st, j);
    return hipGetLastError();
}

template <int STAGE, int WAVES = 4>
hipError_t launch_batched_stage(const RefreshJob* d_jobs, const int* d_starts, int n_jobs,
                                int blocks, hipStream_t st) {
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL((refresh_batched_kernel<STAGE, WAVES>), dim3(blocks), dim3(64 * WAVES), 0, st,
                       d_jobs, d_starts, n_jobs);
    return hipGetLastError();
}

}  // namespace

int64_t product_pairs(const RefreshJob& j) { return (int64_t)j.gx[2] * ((j.v.S + 15) / 16); }

void set_product_tiles(RefreshJob* j, int64_t pairs) {
    j->lt_tiles = product_tiles(pairs);
    j->gy[2] = ((j->v.S + 15) / 16 + j->lt_tiles - 1) / j->lt_tiles;
}

void make_refresh_job(const dust_plan* p, RefreshJob* j) {
    const PlanView& v = p->view;
    *j = RefreshJob{};
    j->v = v;
    j->lam = p->d_lam; j->dlam = p->d_dlam; j->cabs = p->d_cabs; j->w = p->d_w;
    j->es = p->d_es; j->ge = p->ge;
    j->nu = p->d_nu; j->kf = p->d_kf; j->kb = p->d_kb; j->ku = p->d_ku; j->em = p->d_em;
    j->khi = p->d_khi; j->klo = p->d_klo; j->kdb = p->d_kdb; j->c2l = p->d_c2l;
    j->fwd = p->d_fwd; j->ylo = p->d_ylo; j->yhi = p->d_yhi;
    j->dyinv = p->d_dyinv; j->kidx = p->d_kidx; j->invd = p->d_invd;
    j->invf = reinterpret_cast<float2*>(p->d_invf);
    j->ylof = p->d_ylof; j->dyinvf = p->d_dyinvf;
    const bool tab = table_mode(v.mode);
    if (mixed_mode(v.mode)) {
        j->Nc = COLD_P;
        j->fwd_c = p->d_fwd_c; j->ylo_c = p->d_ylo_c; j->dyinv_c = p->d_dyinv_c;
        j->inv_c = p->d_inv_c;
        j->lnTmin_c = v.lnTmin - log(COLD_RATIO);
        j->hstep_c = log(COLD_RATIO) / (COLD_P - 1);
    }
    j->gx[0] = (v.NLp + 255) / 256;  j->gy[0] = v.Sp;
    j->gx[1] = 1;                    j->gy[1] = 0;
    const int pb = product_blocks(v.NL);
    j->gx[2] = ((v.N + j->Nc + 15) / 16 + pb - 1) / pb;
    set_product_tiles(j, product_pairs(*j));
    // (mixed: one more column for the table below the range)
    j->gx[3] = (v.M + 255) / 256 + (j->Nc > 0); j->gy[3] = tab ? v.S : 0;
}

hipError_t launch_prepare(const dust_plan* p, hipStream_t st) {
    RefreshJob j;
    make_refresh_job(p, &j);
    hipError_t e = launch_stage<0>(j, st);
    if (e != hipSuccess) return e;
    e = product_shares(j.v.NL) == LT_WAVES ? launch_stage<2, LT_WAVES>(j, st) : launch_stage<2>(j, st);
    if (e != hipSuccess || !table_mode(j.v.mode)) return e;
    return launch_stage<3>(j, st);
}

// Eight waves where the plans' wavelengths are many, and where a launch that is
// over soon waits for one long plan (six of 120 x 20 and one of 1000 x 80: 133 us
// with the batch, 145 with four waves).
bool long_product(const RefreshJob* jobs, int n_jobs) {
    double pairs = 0.0, steps = 0.0, workgroups = 0.0;
    int longest = 0;
    for (int k = 0; k < n_jobs; ++k) {
        const double p = (double)product_pairs(jobs[k]) * product_blocks(jobs[k].v.NL);
        pairs += p;
        steps += p * jobs[k].v.NL;
        workgroups += (double)jobs[k].gx[2] * jobs[k].gy[2];
        longest = longest > jobs[k].v.NL ? longest : jobs[k].v.NL;
    }
    return steps >= 700.0 * pairs || (longest >= 600 && workgroups <= 1024.0);
}

hipError_t launch_prepare_batched(const RefreshJob* d_jobs, const int* const d_starts[4],
                                  int n_jobs, const int blocks[4], bool long_prod,
                                  hipStream_t st) {
    hipError_t e;
    if ((e = launch_batched_stage<0>(d_jobs, d_starts[0], n_jobs, blocks[0], st)) != hipSuccess) return e;
    e = long_prod ? launch_batched_stage<2, LT_WAVES>(d_jobs, d_starts[2], n_jobs, blocks[2], st)
                  : launch_batched_stage<2>(d_jobs, d_starts[2], n_jobs, blocks[2], st);
    if (e != hipSuccess) return e;
    return launch_batched_stage<3>(d_jobs, d_starts[3], n_jobs, blocks[3], st);
}

}  // namespace dust
