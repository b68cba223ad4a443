// Meta-solver on the payoff table and meta-strategy sampling from device
// weights: the meta-update Comb_{t+1} ~ G(...) of Sec. 3.1 with the
// fictitious-play solver of the PSRO experiments (Sec. 4.2), closed on the GPU
// (table -> game -> fictitious play -> sigma -> meta-sample -> next rollout).
#include "device.hpp"
#include "internal.hpp"

namespace malib {

// M[i][j] = the mean of cell (i, j), sum * 2^-32 / count as the table read-back
// computes it; 0 where the cell has no simulations.
__global__ void payoff_matrix_kernel(const unsigned long long* __restrict__ sum,
                                     const unsigned long long* __restrict__ cnt, int PP,
                                     double* __restrict__ M)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= PP)
        return;
    const long long c = (long long)cnt[i];
    M[i] = c > 0 ? ldexp((double)(long long)sum[i], -32) / (double)c : 0.0;
}

hipError_t launch_payoff_matrix(const unsigned long long* sum, const unsigned long long* cnt,
                                int P, double* M, hipStream_t s)
{
    const int PP = P * P;
    payoff_matrix_kernel<<<(PP + 255) / 256, 256, 0, s>>>(sum, cnt, PP, M);
    return hipGetLastError();
}

constexpr int kSolveLdsP = 128;   // up to this P the game sits in LDS
static_assert(kMaxP <= 4 * 64, "the solver keeps at most 4 policies per lane");

// DPP controls: swap neighbours, swap pairs in a quad, mirror each 8-lane
// half row, mirror each 16-lane row.  After the four steps every lane holds
// its row's result.
constexpr int kDppQuadSwap1 = 0xB1;   // quad_perm [1, 0, 3, 2]
constexpr int kDppQuadSwap2 = 0x4E;   // quad_perm [2, 3, 0, 1]
constexpr int kDppHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;
constexpr int kDppRowBcast15 = 0x142;   // lane 15 of each row to the next row
constexpr int kDppRowBcast31 = 0x143;   // lane 31 to the rows above it

// A reduction step's other value (every lane has a source in these patterns, so
// the move folds into the instruction that uses it).
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int x)
{
    return __builtin_amdgcn_mov_dpp(x, CTRL, 0xF, 0xF, false);
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = dpp_i32<CTRL>((int)b), hi = dpp_i32<CTRL>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ double readlane_f64(double x, int l)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The wavefront's largest x and smallest y (signed integers), in every lane: four
// DPP steps inside the 16-lane rows, one instruction each, the two sides
// interleaved; then rows and halves exchanged (v_permlane16/32_swap of a value
// with itself leaves its even rows in one result and its odd rows in the other).
__device__ __forceinline__ void wave_max_min_i32(int& x, int& y)
{
    auto step = [&](int dx, int dy) {
        x = max(x, dx);
        y = min(y, dy);
    };
    step(dpp_i32<kDppQuadSwap1>(x), dpp_i32<kDppQuadSwap1>(y));
    step(dpp_i32<kDppQuadSwap2>(x), dpp_i32<kDppQuadSwap2>(y));
    step(dpp_i32<kDppHalfMirror>(x), dpp_i32<kDppHalfMirror>(y));
    step(dpp_i32<kDppRowMirror>(x), dpp_i32<kDppRowMirror>(y));
    const auto x1 = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    const auto y1 = __builtin_amdgcn_permlane16_swap(y, y, false, false);
    x = max((int)x1[0], (int)x1[1]);
    y = min((int)y1[0], (int)y1[1]);
    const auto x2 = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const auto y2 = __builtin_amdgcn_permlane32_swap(y, y, false, false);
    x = max((int)x2[0], (int)x2[1]);
    y = min((int)y2[0], (int)y2[1]);
}

// Exchanges between a wavefront's 16-lane rows and its halves: the even and the
// odd rows' (the lower and the upper half's) values of x, one after the other in
// every row.
template <int W>
__device__ __forceinline__ void swap_rows(int x, int& even, int& odd)
{
    if constexpr (W == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        even = (int)r[0];
        odd = (int)r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        even = (int)r[0];
        odd = (int)r[1];
    }
}

template <int W>
__device__ __forceinline__ void swap_rows(double x, double& even, double& odd)
{
    const long long b = __double_as_longlong(x);
    int l0, l1, h0, h1;
    swap_rows<W>((int)b, l0, l1);
    swap_rows<W>((int)(b >> 32), h0, h1);
    even = __longlong_as_double(((long long)h0 << 32) | (unsigned int)l0);
    odd = __longlong_as_double(((long long)h1 << 32) | (unsigned int)l1);
}

// op over the wavefront (op associative and commutative), in every lane.
template <class V, class Op>
__device__ __forceinline__ V wave_reduce(V x, Op op)
{
    auto dpp = [](V y, auto ctrl) {
        if constexpr (sizeof(V) == 8)
            return dpp_f64<decltype(ctrl)::value>(y);
        else
            return dpp_i32<decltype(ctrl)::value>(y);
    };
    x = op(x, dpp(x, std::integral_constant<int, kDppQuadSwap1>{}));
    x = op(x, dpp(x, std::integral_constant<int, kDppQuadSwap2>{}));
    x = op(x, dpp(x, std::integral_constant<int, kDppHalfMirror>{}));
    x = op(x, dpp(x, std::integral_constant<int, kDppRowMirror>{}));
    V e, o;
    swap_rows<16>(x, e, o);
    x = op(e, o);
    swap_rows<32>(x, e, o);
    return op(e, o);
}

__device__ __forceinline__ double wave_min_f64(double x)
{
    return wave_reduce(x, [](double a, double b) { return __builtin_fmin(a, b); });
}

__device__ __forceinline__ double wave_sum_f64(double x)
{
    return wave_reduce(x, [](double a, double b) { return a + b; });
}

__device__ __forceinline__ int wave_min_i32(int x)
{
    return wave_reduce(x, [](int a, int b) { return min(a, b); });
}

// Order-preserving halves of a double: comparing (hi, lo) as (signed, unsigned)
// integers compares the values (-0 below +0, NaN outside the infinities).
__device__ __forceinline__ void sort_key(double v, int& hi, unsigned int& lo)
{
    const long long b = __double_as_longlong(v);
    const int s = (int)(b >> 63);            // all ones for negative values
    hi = (int)(b >> 32) ^ (s & 0x7FFFFFFF);
    lo = (unsigned int)b ^ (unsigned int)s;
}

// The same across rows: lanes of the rows in ROWS take the pattern's source,
// the others keep their own value.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64_rows(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, CTRL, ROWS, 0xF, false);
    const int hi =
        __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), CTRL, ROWS, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The largest of x and the smallest of y over the wavefront, the same in
// every lane; the two reductions interleave.  IEEE maxNum / minNum (one
// v_max_f64 / v_min_f64 each): a NaN never replaces a number, and which of
// +0 and -0 survives does not matter (the callers compare with ==, and take
// the winning policy's own sum afterwards).
__device__ __forceinline__ void wave_max_min(double& x, double& y)
{
    auto hi = [](double a, double b) { return __builtin_fmax(a, b); };
    auto lo = [](double a, double b) { return __builtin_fmin(a, b); };
    double dx = dpp_f64<kDppQuadSwap1>(x), dy = dpp_f64<kDppQuadSwap1>(y);
    x = hi(x, dx);
    y = lo(y, dy);
    dx = dpp_f64<kDppQuadSwap2>(x);
    dy = dpp_f64<kDppQuadSwap2>(y);
    x = hi(x, dx);
    y = lo(y, dy);
    dx = dpp_f64<kDppHalfMirror>(x);
    dy = dpp_f64<kDppHalfMirror>(y);
    x = hi(x, dx);
    y = lo(y, dy);
    dx = dpp_f64<kDppRowMirror>(x);
    dy = dpp_f64<kDppRowMirror>(y);
    x = hi(x, dx);
    y = lo(y, dy);
    // rows: lane 15 of rows 0 and 2 into rows 1 and 3, then lane 31 into
    // rows 2 and 3; lane 63 then holds the wavefront's result
    dx = dpp_f64_rows<kDppRowBcast15, 0xA>(x);
    dy = dpp_f64_rows<kDppRowBcast15, 0xA>(y);
    x = hi(x, dx);
    y = lo(y, dy);
    dx = dpp_f64_rows<kDppRowBcast31, 0xC>(x);
    dy = dpp_f64_rows<kDppRowBcast31, 0xC>(y);
    x = hi(x, dx);
    y = lo(y, dy);
    x = readlane_f64(x, 63);
    y = readlane_f64(y, 63);
}

// Simultaneous fictitious play on the zero-sum game with row payoff M
// (P x P, fp64; meant for finite entries, a NaN anywhere in v or w leaves the
// counts unspecified and sets gap to NaN): at iteration t, i_t = first argmax
// of v = sum over s < t of M[:, j_s] and j_t = first argmin of w = sum over
// s < t of M[i_s, :]; then both play counts are incremented and v, w gain
// column j_t and row i_t (one fp64 add per element per iteration, in
// iteration order).  One wavefront: lane l keeps policies k = l + 64 q,
// q < K, so an iteration needs no barrier.  The first argmax is the lowest k
// whose v equals the wavefront's maximum: the lowest q with a match, then the
// lowest lane (a ballot).  Bound by that chain's latency: the reduction runs on
// the order-preserving high words, whose DPP steps are one instruction each, and
// on the low words only where several policies share the extreme (1000
// iterations at P = 128: 302 us with fp64 reductions throughout, 269 us; P = 64:
// 208 and 199 us).  Writes sigma[0][k], sigma[1][k] = the play counts (weights for
// meta-sampling) and gap = (v[i] - w[j]) / T at the best responses i, j to the
// final sums.
template <int K, bool IN_LDS>
__global__ __launch_bounds__(64) void solve_fp_kernel(const double* __restrict__ M, int P, int T,
                                                      float* __restrict__ sigma,
                                                      double* __restrict__ gap)
{
    // the game with a padded row stride (column reads hit different banks)
    constexpr int LDS_DOUBLES = IN_LDS ? kSolveLdsP * (kSolveLdsP + 1) : 1;
    __shared__ double Ms[LDS_DOUBLES];
    const int lane = threadIdx.x;
    const int stride = IN_LDS ? P + 1 : P;
    const double* G = M;
    if constexpr (IN_LDS) {
        for (int e = lane; e < P * P; e += 64)
            Ms[(e / P) * stride + e % P] = M[e];
        __syncthreads();
        G = Ms;
    }
    double v[K], w[K];
    int cx[K], cy[K];
    bool mine[K];
    // slots past P start at -inf (v) and +inf (w) and keep adding finite
    // entries, so they never win a reduction and need no masking
#pragma unroll
    for (int q = 0; q < K; ++q) {
        mine[q] = lane + 64 * q < P;
        v[q] = mine[q] ? 0.0 : -INFINITY;
        w[q] = mine[q] ? 0.0 : INFINITY;
        cx[q] = 0;
        cy[q] = 0;
    }
    // The policies whose value has the extreme high word (row side: largest v;
    // column side: smallest w), as lane masks per q; true when more than one
    // policy of a side has it, so that the low words decide.
    int vh[K], wh[K];
    unsigned int vl[K], wl[K];
    unsigned long long bi[K], bj[K];
    auto extremes = [&]() {
#pragma unroll
        for (int q = 0; q < K; ++q) {
            sort_key(v[q], vh[q], vl[q]);
            sort_key(w[q], wh[q], wl[q]);
        }
        int mv = vh[0], mw = wh[0];
#pragma unroll
        for (int q = 1; q < K; ++q) {
            mv = max(mv, vh[q]);
            mw = min(mw, wh[q]);
        }
        wave_max_min_i32(mv, mw);
#pragma unroll
        for (int q = 0; q < K; ++q) {
            bi[q] = __ballot(vh[q] == mv);
            bj[q] = __ballot(wh[q] == mw);
        }
    };
    auto tied = [&]() {
        int n = 0;
#pragma unroll
        for (int q = 0; q < K; ++q)
            n += __popcll(bi[q]) + __popcll(bj[q]);
        return n > 2;
    };
    auto low_words = [&]() {
        int lv = INT_MIN, lw = INT_MAX;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            lv = (bi[q] >> lane) & 1 ? max(lv, (int)(vl[q] ^ 0x80000000u)) : lv;
            lw = (bj[q] >> lane) & 1 ? min(lw, (int)(wl[q] ^ 0x80000000u)) : lw;
        }
        wave_max_min_i32(lv, lw);
#pragma unroll
        for (int q = 0; q < K; ++q) {
            bi[q] &= __ballot((int)(vl[q] ^ 0x80000000u) == lv);
            bj[q] &= __ballot((int)(wl[q] ^ 0x80000000u) == lw);
        }
    };
    // The first of them: the lowest q, then the lowest lane (with only NaN sums
    // any policy, below P).
    auto first = [&](const unsigned long long (&m)[K]) {
        int i = 64 * (K - 1) + ((__ffsll(m[K - 1]) - 1) & 63);
#pragma unroll
        for (int q = K - 2; q >= 0; --q)
            i = m[q] ? 64 * q + __ffsll(m[q]) - 1 : i;
        return min(i, P - 1);
    };
    // The same masks by fp64 maxima: no second pass, whatever is tied.
    auto extremes_f64 = [&]() {
        double lv = v[0], lw = w[0];
#pragma unroll
        for (int q = 1; q < K; ++q) {
            lv = __builtin_fmax(lv, v[q]);
            lw = __builtin_fmin(lw, w[q]);
        }
        wave_max_min(lv, lw);
#pragma unroll
        for (int q = 0; q < K; ++q) {
            bi[q] = __ballot(v[q] == lv);
            bj[q] = __ballot(w[q] == lw);
        }
    };
    auto play = [&](int i, int j) {
        // every slot reads (a slot past P reads policy P - 1 and is never
        // looked at), so all loads issue before the first add waits
        double gv[K], gw[K];
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const int kc = mine[q] ? lane + 64 * q : P - 1;
            gv[q] = G[kc * stride + j];
            gw[q] = G[i * stride + kc];
        }
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const int k = lane + 64 * q;
            cx[q] += k == i;
            cy[q] += k == j;
            v[q] = v[q] + gv[q];
            w[q] = w[q] + gw[q];
        }
    };
    // A game whose extremes tie in more than an eighth of the iterations (equal
    // rows of policies without a played cell, duplicates) goes on with fp64 maxima,
    // from the third tied iteration at the earliest (all sums tie in the first).
    // us per 1000 iterations, tied throughout: 428 at P = 128 with the high words,
    // 295 like this, 303 with fp64 maxima from the start; P = 64 292, 208 and 209.
    // With four policies per lane fp64 maxima are faster anyway (P = 256, no ties:
    // 535 us against 574).
    int t = 0, ties = 0;
    for (; K < 4 && t < T; ++t) {
        extremes();
        if (__builtin_expect(tied(), 0)) {
            if (8 * ++ties > t + 16)
                break;   // this iteration is played below
            low_words();
        }
        play(first(bi), first(bj));
    }
    for (; t < T; ++t) {
        if constexpr (K == 1) {
            // one policy per lane: from the two values, without the masks (which
            // took 214 instead of 209 us per 1000 iterations at P = 64)
            double vi = v[0], wj = w[0];
            wave_max_min(vi, wj);
            const unsigned long long mi = __ballot(v[0] == vi), mj = __ballot(w[0] == wj);
            const int i = mi ? __ffsll(mi) - 1 : P - 1, j = mj ? __ffsll(mj) - 1 : P - 1;
            play(min(i, P - 1), min(j, P - 1));
        } else {
            extremes_f64();
            play(first(bi), first(bj));
        }
    }
#pragma unroll
    for (int q = 0; q < K; ++q) {
        if (mine[q]) {
            sigma[lane + 64 * q] = (float)cx[q];
            sigma[P + lane + 64 * q] = (float)cy[q];
        }
    }
    if (gap) {
        bool nan = false;
#pragma unroll
        for (int q = 0; q < K; ++q)
            nan = nan || (mine[q] && (__builtin_isnan(v[q]) || __builtin_isnan(w[q])));
        const bool any_nan = __ballot(nan) != 0ull;
        extremes();
        if (tied())
            low_words();
        const int i = first(bi), j = first(bj);
        double vs = v[0], ws = w[0];
#pragma unroll
        for (int q = 1; q < K; ++q) {
            vs = q == (i >> 6) ? v[q] : vs;
            ws = q == (j >> 6) ? w[q] : ws;
        }
        const double vi = __shfl(vs, i & 63), wj = __shfl(ws, j & 63);
        if (lane == 0)
            *gap = any_nan ? (double)NAN : (vi - wj) / (double)T;
    }
}

hipError_t launch_solve_fp(const double* M, int P, int T, float* sigma, double* gap,
                           hipStream_t s)
{
    if (P < 1 || P > kMaxP || T < 1)
        return hipErrorInvalidValue;
    if (P <= 64)
        solve_fp_kernel<1, true><<<1, 64, 0, s>>>(M, P, T, sigma, gap);
    else if (P <= kSolveLdsP)
        solve_fp_kernel<2, true><<<1, 64, 0, s>>>(M, P, T, sigma, gap);
    else
        solve_fp_kernel<4, false><<<1, 64, 0, s>>>(M, P, T, sigma, gap);
    return hipGetLastError();
}

// Aggregate payoffs of a meta-strategy pair (the PSRO convergence judgement):
// x, y = the weight rows sigma[0], sigma[1] normalized in fp64 (sequential
// sums); u = M y and v = x^T M, each entry a sequential fp64 sum of rounded
// products (thread k forms u[k] over row k and v[k] over column k); nash =
// x^T u (sequential).  out = {nash, -nash, u[br_row], -v[br_col],
// improvement}, where improvement is the larger best-response gain of the
// sides whose br is >= 0 (a side with br = -1 gives NaN).
__global__ __launch_bounds__(kMaxP) void aggregate_kernel(const double* __restrict__ M, int P,
                                                          const float* __restrict__ sigma,
                                                          int br_row, int br_col,
                                                          double* __restrict__ out)
{
    __shared__ double x[kMaxP], y[kMaxP], u[kMaxP];
    __shared__ double S[2], vbr;
    const int k = threadIdx.x;
    if (k == 0) {
        double a = 0.0, b = 0.0;
#pragma unroll 16
        for (int m = 0; m < P; ++m)
            a += (double)sigma[m];
#pragma unroll 16
        for (int m = 0; m < P; ++m)
            b += (double)sigma[P + m];
        S[0] = a;
        S[1] = b;
    }
    __syncthreads();
    if (k < P) {
        x[k] = (double)sigma[k] / S[0];
        y[k] = (double)sigma[P + k] / S[1];
    }
    __syncthreads();
    if (k < P) {
        // (unrolled so that the loads run ahead of the dependent adds)
        double acc = 0.0;
#pragma unroll 16
        for (int j = 0; j < P; ++j)
            acc = acc + M[(size_t)k * P + j] * y[j];
        u[k] = acc;
        double accv = 0.0;
#pragma unroll 16
        for (int i = 0; i < P; ++i)
            accv = accv + x[i] * M[(size_t)i * P + k];
        if (k == br_col)
            vbr = accv;
    }
    __syncthreads();
    if (k == 0) {
        double nash = 0.0;
#pragma unroll 16
        for (int i = 0; i < P; ++i)
            nash = nash + x[i] * u[i];
        const double wr = br_row >= 0 ? u[br_row] : (double)NAN;
        const double wc = br_col >= 0 ? -vbr : (double)NAN;
        double imp = (double)NAN;
        if (br_row >= 0)
            imp = wr - nash;
        if (br_col >= 0) {
            const double g = wc - (-nash);
            imp = (br_row < 0 || g > imp) ? g : imp;
        }
        out[0] = nash;
        out[1] = -nash;
        out[2] = wr;
        out[3] = wc;
        out[4] = imp;
    }
}

hipError_t launch_aggregate(const double* M, int P, const float* sigma, int br_row, int br_col,
                            double* out, hipStream_t s)
{
    aggregate_kernel<<<1, kMaxP, 0, s>>>(M, P, sigma, br_row, br_col, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ alpha-rank
//
// Single-population alpha-rank (Omidshafiei et al., 2019; the meta-solver the
// paper lists beside fictitious play for PSRO, Sec. 4.2, Table 3) on the
// table's game made symmetric by a meeting on each side: a mutant s in a
// population of r has fitness advantage u = alpha (M[s][r] - M[r][s]); its
// fixation probability in a population of m is rho(u) = (1 - e^-u) /
// (1 - e^-mu) (1/m at u = 0), and the chain moves r -> s with probability
// rho / (P - 1).  The stationary distribution comes from the
// Grassmann-Taksar-Heyman elimination, which uses only the off-diagonal
// transition probabilities and never subtracts, so small probabilities keep
// their relative accuracy: for n = P-1 .. 1, S = sum_{j<n} A[n][j],
// A[i][n] /= S and A[i][j] += A[i][n] A[n][j] for i, j < n; then pi_0 = 1,
// pi_j = sum_{i<j} pi_i A[i][j], normalized.  One workgroup; the matrix in
// registers for P <= kArRegMax, else in the caller's workspace.

constexpr int kArThreads = 1024;
constexpr int kArLdsMax = 128;

__device__ __forceinline__ double ar_fixation(double u, int m)
{
    if (u == 0.0)
        return 1.0 / m;
    if (u > 0.0)
        return expm1(-u) / expm1(-m * u);
    // u < 0: e^((m-1) u) taken out, so that the ratio underflows gracefully
    const double v = -u;
    return exp(-(m - 1) * v) * (expm1(-v) / expm1(-m * v));
}

// Sum of one value per thread over the workgroup (fixed shuffle/LDS order).
__device__ __forceinline__ double ar_block_sum(double v, double* red)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_xor(v, off, 64);
    __syncthreads();        // red is reused
    if (lane == 0)
        red[wave] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kArThreads / 64; ++w)
        t += red[w];
    return t;
}

// P > kArRegMax: the matrix in the caller's workspace
__global__ __launch_bounds__(kArThreads) void alpharank_kernel(const double* __restrict__ M,
                                                               int P, double alpha, int m,
                                                               double* __restrict__ work,
                                                               double* __restrict__ pi,
                                                               float* __restrict__ sigma)
{
    __shared__ double red[kArThreads / 64];
    __shared__ double s_pi[kMaxP];
    double* A = work;
    const int ld = P;
    const int tid = threadIdx.x;
    // ---- the chain's off-diagonal transition probabilities
    const double mut = P > 1 ? 1.0 / (P - 1) : 0.0;
    for (int idx = tid; idx < P * P; idx += kArThreads) {
        const int r = idx / P, c = idx - r * P;
        double v = 0.0;
        if (r != c)
            v = ar_fixation(alpha * (M[(size_t)c * P + r] - M[(size_t)r * P + c]), m) * mut;
        A[(size_t)r * ld + c] = v;
    }
    __syncthreads();
    // ---- elimination, states P-1 .. 1; thread (ti, tj) of a 32 x 32 grid
    // updates A[i][j] for i = ti mod 32, j = tj mod 32
    const int ti = tid >> 5, tj = tid & 31;
    for (int n = P - 1; n >= 1; --n) {
        const double S = ar_block_sum(tid < n ? A[(size_t)n * ld + tid] : 0.0, red);
        for (int i = tid; i < n; i += kArThreads)
            A[(size_t)i * ld + n] /= S;
        __syncthreads();
        for (int i = ti; i < n; i += 32) {
            const double ain = A[(size_t)i * ld + n];
            for (int j = tj; j < n; j += 32)
                A[(size_t)i * ld + j] += ain * A[(size_t)n * ld + j];
        }
        __syncthreads();
    }
    // ---- back substitution, then normalization
    if (tid == 0)
        s_pi[0] = 1.0;
    __syncthreads();
    for (int j = 1; j < P; ++j) {
        const double v = ar_block_sum(tid < j ? s_pi[tid] * A[(size_t)tid * ld + j] : 0.0, red);
        if (tid == 0)
            s_pi[j] = v;
        __syncthreads();
    }
    const double total = ar_block_sum(tid < P ? s_pi[tid] : 0.0, red);
    if (tid < P) {
        const double x = s_pi[tid] / total;
        pi[tid] = x;
        if (sigma) {
            sigma[tid] = (float)x;
            sigma[P + tid] = (float)x;
        }
    }
}

// The same elimination for P <= kArRegMax with the matrix in registers: a TI x TJ
// grid of threads, element (ti + TI a, tj + TJ b) in register (a, b).  At step n
// the lanes that hold row n and column n write them to LDS; after one barrier
// each wavefront forms S by itself and scales the column's entries of its own
// rows (one division per lane).  The scaled columns are kept (U, in LDS up to
// P = 128, else the workspace) for the back substitution, in which one wavefront
// adds pi_i times row i to the later states' sums.  The fixation probabilities of
// both directions of a pair come from one evaluation: rho(-u) = e^(-(m-1)u)
// rho(u) is how the negative side is computed.  Bound by a step's chain (P = 100:
// 248 us with two block reductions and their barriers per state, 128 us).
constexpr int kArRegMax = 224;

template <int TI, int TJ, int KI, int KJ>
__global__ __launch_bounds__(TI * TJ) void alpharank_reg_kernel(
    const double* __restrict__ M, int P, double alpha, int m, double* __restrict__ work,
    double* __restrict__ pi, float* __restrict__ sigma)
{
    constexpr int THREADS = TI * TJ, NI = TI * KI, NJ = TJ * KJ;
    constexpr int NM = NI > NJ ? NI : NJ, L = (NM + 63) / 64;
    constexpr bool LDS_U = NM <= kArLdsMax;
    constexpr int WR = 64 / TJ;                       // grid rows of a wavefront
    static_assert(WR * KI <= 64, "one division per lane");
    __shared__ double u_s[LDS_U ? NM * (NM + 1) : 1];
    __shared__ double row_s[2][64 * L], col_s[2][64 * L], scaled_s[THREADS / 64][64];
    double* U = LDS_U ? u_s : work;
    const int ld = LDS_U ? P + 1 : P;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ti = tid / TJ, tj = tid % TJ;
    // ---- the chain's off-diagonal transition probabilities, by pairs r < c
    const double mut = P > 1 ? 1.0 / (P - 1) : 0.0;
    const int odd = P & 1, wide = P - 1 + odd, pairs = P * (P - 1) / 2;
    for (int k = tid; k < pairs; k += THREADS) {
        // row i of the folded triangle: pairs of row i, then of a row from the end
        const int i = k / wide, j = k - i * wide;
        const bool top = odd ? j > i : j >= i;
        const int r = top ? i : P - 1 - odd - i;
        const int c = top ? j + 1 - odd : P - 1 - j;
        const double u = alpha * (M[(size_t)c * P + r] - M[(size_t)r * P + c]);
        const double v = __builtin_fabs(u);
        double up = 1.0 / m, down = 1.0 / m;
        if (u != 0.0) {
            up = expm1(-v) / expm1(-m * v);
            // e^((m-1) u) taken out, so that the ratio underflows gracefully
            down = exp(-(m - 1) * v) * up;
        }
        U[(size_t)r * ld + c] = (u > 0.0 ? up : down) * mut;
        U[(size_t)c * ld + r] = (u > 0.0 ? down : up) * mut;
    }
    __syncthreads();
    double A[KI][KJ];
#pragma unroll
    for (int a = 0; a < KI; ++a)
#pragma unroll
        for (int b = 0; b < KJ; ++b) {
            const int i = ti + TI * a, j = tj + TJ * b;
            A[a][b] = i < P && j < P && i != j ? U[(size_t)i * ld + j] : 0.0;
        }
    __syncthreads();                                  // U now takes the scaled columns
    // ---- elimination, states P-1 .. 1
    for (int n = P - 1; n >= 1; --n) {
        double* row = row_s[n & 1];
        double* col = col_s[n & 1];
        const int na = n / TI, nb = n / TJ;
#pragma unroll
        for (int a = 0; a < KI; ++a)
            if (a == na && ti == n % TI)
#pragma unroll
                for (int b = 0; b < KJ; ++b)
                    row[tj + TJ * b] = A[a][b];
#pragma unroll
        for (int b = 0; b < KJ; ++b)
            if (b == nb && tj == n % TJ)
#pragma unroll
                for (int a = 0; a < KI; ++a)
                    col[ti + TI * a] = A[a][b];
        __syncthreads();
        double S = 0.0;
#pragma unroll
        for (int q = 0; q < L; ++q)
            S += lane + 64 * q < n ? row[lane + 64 * q] : 0.0;
        S = wave_sum_f64(S);
        if (lane < WR * KI) {
            const int i = wave * WR + lane % WR + TI * (lane / WR);
            const double v = col[i] / S;
            scaled_s[wave][lane] = v;
            if (i < n)
                U[(size_t)i * ld + n] = v;
        }
        wave_lds_sync();
        double rv[KJ];
#pragma unroll
        for (int b = 0; b < KJ; ++b)
            rv[b] = row[tj + TJ * b];
        // (entries at or past n are not looked at again)
#pragma unroll
        for (int a = 0; a < KI; ++a)
            if (TI * a < n) {
                const double ain = scaled_s[wave][ti % WR + WR * a];
#pragma unroll
                for (int b = 0; b < KJ; ++b)
                    A[a][b] += ain * rv[b];
            }
        wave_lds_sync();
    }
    __syncthreads();
    if (wave != 0)
        return;
    // ---- back substitution, then normalization
    double sum[L];
#pragma unroll
    for (int q = 0; q < L; ++q)
        sum[q] = lane + 64 * q == 0 ? 1.0 : 0.0;
    auto fetch = [&](int i, double (&u)[L]) {
#pragma unroll
        for (int q = 0; q < L; ++q) {
            const int j = lane + 64 * q;
            u[q] = j > i && j < P ? U[(size_t)i * ld + j] : 0.0;
        }
    };
    double u[L], un[L];
    fetch(0, u);
    for (int i = 0; i + 1 < P; ++i) {
        fetch(i + 1, un);
        double pv = sum[0];
#pragma unroll
        for (int q = 1; q < L; ++q)
            pv = (i >> 6) == q ? sum[q] : pv;
        pv = readlane_f64(pv, i & 63);
#pragma unroll
        for (int q = 0; q < L; ++q) {
            sum[q] += pv * u[q];
            u[q] = un[q];
        }
    }
    double total = 0.0;
#pragma unroll
    for (int q = 0; q < L; ++q)
        total += lane + 64 * q < P ? sum[q] : 0.0;
    total = wave_sum_f64(total);
#pragma unroll
    for (int q = 0; q < L; ++q) {
        const int j = lane + 64 * q;
        if (j < P) {
            const double x = sum[q] / total;
            pi[j] = x;
            if (sigma) {
                sigma[j] = (float)x;
                sigma[P + j] = (float)x;
            }
        }
    }
}

bool alpharank_needs_work(int P)
{
    return P > kArLdsMax;
}

hipError_t launch_alpharank(const double* M, int P, double alpha, int m, double* work,
                            double* pi, float* sigma, hipStream_t s)
{
    if (P > kMaxP || P > kArThreads || (P > kArLdsMax && !work))
        return hipErrorInvalidValue;
    auto go = [&](auto kernel, int threads) {
        kernel<<<1, threads, 0, s>>>(M, P, alpha, m, work, pi, sigma);
    };
    if (P <= 32)
        go(alpharank_reg_kernel<16, 16, 2, 2>, 256);
    else if (P <= 64)
        go(alpharank_reg_kernel<16, 16, 4, 4>, 256);
    else if (P <= 96)
        go(alpharank_reg_kernel<16, 32, 6, 3>, 512);
    else if (P <= 128)
        go(alpharank_reg_kernel<16, 32, 8, 4>, 512);
    else if (P <= 160)
        go(alpharank_reg_kernel<16, 32, 10, 5>, 512);
    else if (P <= kArRegMax)
        go(alpharank_reg_kernel<16, 32, 14, 7>, 512);
    else
        alpharank_kernel<<<1, kArThreads, 0, s>>>(M, P, alpha, m, work, pi, sigma);
    return hipGetLastError();
}

// ------------------------------------------------------------------ LP solver
//
// The zero-sum meta-game's exact equilibrium (the LP solver of the PSRO
// experiments, Sec. 4.2) by the primal simplex method on the column side's
// problem after a shift that makes every payoff positive: with
// M' = M - min(M) + 1, maximize sum_j w_j subject to M' w <= 1, w >= 0.  The
// origin is feasible (slack basis).  At the optimum the column side's
// strategy is y = w / sum w, the row side's x = u / sum u with u the slack
// columns' reduced costs (the dual solution), and the value is
// 1 / sum w + min(M) - 1.  The entering column is the most negative reduced
// cost (Dantzig); after kLpDegenerate consecutive degenerate pivots (zero
// ratio) the solver switches to Bland's rule (the lowest entering column, the
// lowest basic variable among tied ratios), which cannot cycle, until a pivot
// makes progress again.  One workgroup: the
// tableau in registers for P <= kLpRegMax (lp_reg_kernel), else [P+1][2P+1]
// (fp64) in the caller's workspace; there each pivot finds the entering column
// and the pivot row with block reductions, stages the column and the scaled pivot
// row in LDS and updates the other rows.

constexpr int kLpThreads = 1024;
constexpr int kLpWorkAbove = 96;   // callers give a workspace above this (used above kLpRegMax)
constexpr double kLpEps = 1e-11;
constexpr int kLpDegenerate = 8;

__device__ __forceinline__ double lp_block_min(double v, double* red)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v = fmin(v, __shfl_xor(v, off, 64));
    __syncthreads();
    if (lane == 0)
        red[wave] = v;
    __syncthreads();
    double t = red[0];
#pragma unroll
    for (int w = 1; w < kLpThreads / 64; ++w)
        t = fmin(t, red[w]);
    return t;
}

__device__ __forceinline__ int lp_block_min_int(int v, int* red)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v = min(v, __shfl_xor(v, off, 64));
    __syncthreads();
    if (lane == 0)
        red[wave] = v;
    __syncthreads();
    int t = red[0];
#pragma unroll
    for (int w = 1; w < kLpThreads / 64; ++w)
        t = min(t, red[w]);
    return t;
}

// P > kLpRegMax: the whole tableau in the caller's workspace
__global__ __launch_bounds__(kLpThreads) void lp_kernel(const double* __restrict__ M, int P,
                                                        int max_pivots,
                                                        double* __restrict__ work,
                                                        double* __restrict__ value,
                                                        double* __restrict__ x,
                                                        double* __restrict__ y,
                                                        float* __restrict__ sigma,
                                                        int* __restrict__ pivots)
{
    __shared__ double col[kMaxP + 1];
    __shared__ double prow[2 * kMaxP + 1];
    __shared__ int basis[kMaxP];
    __shared__ double redd[kLpThreads / 64];
    __shared__ int redi[kLpThreads / 64];
    const int tid = threadIdx.x;
    const int W = 2 * P + 1;                 // columns: w (P), slacks (P), right-hand side
    double* T = work;
    // ---- the shift: min(M); a NaN or infinite entry leaves no game to solve
    // (fmin would skip a NaN): every output is then NaN, pivots -1
    double mn = INFINITY, finite = 1.0;
    for (int i = tid; i < P * P; i += kLpThreads) {
        const double v = M[i];
        mn = fmin(mn, v);
        if (!isfinite(v))
            finite = 0.0;
    }
    mn = lp_block_min(mn, redd);
    if (lp_block_min(finite, redd) == 0.0) {
        for (int j = tid; j < P; j += kLpThreads) {
            x[j] = (double)NAN;
            y[j] = (double)NAN;
            if (sigma) {
                sigma[j] = NAN;
                sigma[P + j] = NAN;
            }
        }
        if (tid == 0) {
            *value = (double)NAN;
            if (pivots)
                *pivots = -1;
        }
        return;
    }
    // ---- the initial tableau (slack basis)
    for (int idx = tid; idx < (P + 1) * W; idx += kLpThreads) {
        const int i = idx / W, j = idx - i * W;
        double v;
        if (i < P)
            v = j < P ? M[(size_t)i * P + j] - mn + 1.0 : (j < 2 * P ? (j - P == i ? 1.0 : 0.0)
                                                                   : 1.0);
        else
            v = j < P ? -1.0 : 0.0;
        T[idx] = v;
    }
    if (tid < P)
        basis[tid] = P + tid;
    __syncthreads();
    int it = 0, degenerate = 0;
    bool done = false;
    for (; it < max_pivots; ++it) {
        // entering column: the most negative reduced cost (the lowest column
        // among equal ones), or under Bland's rule the lowest negative one
        const bool bland = degenerate >= kLpDegenerate;
        double best = INFINITY;
        if (!bland)
            for (int j = tid; j < 2 * P; j += kLpThreads)
                best = fmin(best, T[(size_t)P * W + j]);
        const double dmin = bland ? -INFINITY : lp_block_min(best, redd);
        int cand = INT_MAX;
        for (int j = tid; j < 2 * P; j += kLpThreads) {
            const double c = T[(size_t)P * W + j];
            if (c < -kLpEps && (bland || c == dmin))
                cand = min(cand, j);
        }
        const int e = lp_block_min_int(cand, redi);
        if (e == INT_MAX) {
            done = true;
            break;
        }
        for (int i = tid; i <= P; i += kLpThreads)
            col[i] = T[(size_t)i * W + e];
        __syncthreads();
        // ratio test: the smallest rhs / col over rows with col > 0, then the
        // lowest basic variable among the rows within rounding of it
        double ratio = INFINITY;
        for (int i = tid; i < P; i += kLpThreads)
            if (col[i] > kLpEps)
                ratio = T[(size_t)i * W + 2 * P] / col[i];
        const double rmin = lp_block_min(ratio, redd);
        if (!(rmin < INFINITY))
            break;                           // unbounded: not reachable for M' > 0
        int bcand = INT_MAX;
        for (int i = tid; i < P; i += kLpThreads)
            if (col[i] > kLpEps &&
                T[(size_t)i * W + 2 * P] / col[i] <= rmin + 1e-12 * fmax(1.0, rmin))
                bcand = min(bcand, basis[i] * 1024 + i);   // P <= 256 < 1024
        const int rb = lp_block_min_int(bcand, redi);
        const int r = rb & 1023;
        degenerate = rmin <= 0.0 ? degenerate + 1 : 0;
        // scaled pivot row, then every other row
        const double piv = col[r];
        for (int j = tid; j < W; j += kLpThreads) {
            const double v = T[(size_t)r * W + j] / piv;
            prow[j] = v;
            T[(size_t)r * W + j] = v;
        }
        __syncthreads();
        for (int idx = tid; idx < (P + 1) * W; idx += kLpThreads) {
            const int i = idx / W, j = idx - i * W;
            if (i != r)
                T[idx] -= col[i] * prow[j];
        }
        if (tid == 0)
            basis[r] = e;
        __syncthreads();
    }
    // ---- read the solution
    const double total = T[(size_t)P * W + 2 * P];      // sum of w = sum of u
    const bool ok = done && total > 0.0;
    for (int j = tid; j < P; j += kLpThreads) {
        y[j] = 0.0;
        x[j] = ok ? T[(size_t)P * W + P + j] / total : (double)NAN;
    }
    __syncthreads();
    for (int i = tid; i < P; i += kLpThreads) {
        if (basis[i] < P)
            y[basis[i]] = ok ? T[(size_t)i * W + 2 * P] / total : (double)NAN;
    }
    __syncthreads();
    if (!ok)
        for (int j = tid; j < P; j += kLpThreads)
            y[j] = (double)NAN;
    if (sigma) {
        __syncthreads();
        for (int j = tid; j < P; j += kLpThreads) {
            sigma[j] = (float)x[j];
            sigma[P + j] = (float)y[j];
        }
    }
    if (tid == 0) {
        *value = ok ? 1.0 / total + mn - 1.0 : (double)NAN;
        if (pivots)
            *pivots = done ? it : -1;
    }
}

// The same method for P <= kLpRegMax, with the same arithmetic and choices,
// bit for bit, and the tableau in registers.  Basic columns are unit columns, so
// only the P nonbasic ones are kept: a pivot puts the leaving variable into the
// entering one's place (its column there is the unit vector of the pivot row).
// TI x TJ threads hold the body, element (ti + TI a, tj + TJ b) in register (a,
// b); each wavefront keeps the reduced costs, the right-hand side and both
// variable lists spread over its lanes, and so finds the pivot by itself (few
// wavefronts, while the body fits their registers, repeat that work less): a pivot has two barriers, after the entering column and after
// the scaled pivot row reach LDS.  Bound by a pivot's chain of reductions, two
// divisions and barriers (P = 100: 1.9 us per pivot; the whole tableau in memory
// with 1024 threads and eight barriers took 8.6 us).
constexpr int kLpRegMax = 224;

// A TI x TJ grid of threads, KI x KJ elements each (P <= TI KI and TJ KJ).
template <int TI, int TJ, int KI, int KJ>
__global__ __launch_bounds__(TI * TJ) void lp_reg_kernel(
    const double* __restrict__ M, int P, int max_pivots, double* __restrict__ value,
    double* __restrict__ x, double* __restrict__ y, float* __restrict__ sigma,
    int* __restrict__ pivots)
{
    constexpr int THREADS = TI * TJ, NI = TI * KI, NJ = TJ * KJ;
    constexpr int L = ((NI > NJ ? NI : NJ) + 63) / 64;      // entries of a row or column per lane
    __shared__ double col_s[2][64 * L], prow_s[64 * L], raw_s[64 * L];
    __shared__ double redd[THREADS / 64], xs[64 * L], ys[64 * L];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ti = tid / TJ, tj = tid % TJ;
    // ---- the shift: min(M); a NaN or infinite entry leaves no game to solve
    double mn = INFINITY;
    bool finite = true;
    for (int i = tid; i < P * P; i += THREADS) {
        const double v = M[i];
        mn = fmin(mn, v);
        finite = finite && isfinite(v);
    }
    mn = wave_min_f64(mn);
    if (lane == 0)
        redd[wave] = mn;
    if (__syncthreads_or(!finite)) {
        for (int j = tid; j < P; j += THREADS) {
            x[j] = (double)NAN;
            y[j] = (double)NAN;
            if (sigma) {
                sigma[j] = NAN;
                sigma[P + j] = NAN;
            }
        }
        if (tid == 0) {
            *value = (double)NAN;
            if (pivots)
                *pivots = -1;
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < THREADS / 64; ++k)
        mn = fmin(mn, redd[k]);
    // ---- the initial body: row i slack P + i, column j variable j
    double T[KI][KJ];
#pragma unroll
    for (int a = 0; a < KI; ++a)
#pragma unroll
        for (int b = 0; b < KJ; ++b) {
            const int i = ti + TI * a, j = tj + TJ * b;
            T[a][b] = i < P && j < P ? M[(size_t)i * P + j] - mn + 1.0 : 0.0;
        }
    double rc[L], rhs[L];
    int var[L], bas[L];                        // variable of column / of row lane + 64 q
#pragma unroll
    for (int q = 0; q < L; ++q) {
        const bool in = lane + 64 * q < P;
        rc[q] = in ? -1.0 : 0.0;               // (columns past P never enter)
        rhs[q] = 1.0;
        var[q] = lane + 64 * q;
        bas[q] = P + lane + 64 * q;
    }
    double total = 0.0;                        // sum of w = sum of u
    int it = 0, degenerate = 0;
    bool done = false;
    for (; it < max_pivots; ++it) {
        double* col = col_s[it & 1];
        // entering column: the most negative reduced cost (the lowest variable
        // among equal ones), or under Bland's rule the lowest negative one
        const bool bland = degenerate >= kLpDegenerate;
        double best = rc[0];
#pragma unroll
        for (int q = 1; q < L; ++q)
            best = fmin(best, rc[q]);
        const double dmin = wave_min_f64(best);
        if (!(dmin < -kLpEps)) {
            done = true;
            break;
        }
        int cand = INT_MAX;
#pragma unroll
        for (int q = 0; q < L; ++q)
            if (rc[q] < -kLpEps && (bland || rc[q] == dmin))
                cand = min(cand, var[q] * 256 + lane + 64 * q);
        const int ev = wave_min_i32(cand), e = ev & 255, evar = ev >> 8;
        // its reduced cost, uniform
        double rce = rc[0];
#pragma unroll
        for (int q = 1; q < L; ++q)
            rce = (e >> 6) == q ? rc[q] : rce;
        rce = readlane_f64(rce, __builtin_amdgcn_readfirstlane(e & 63));
        const int eb = __builtin_amdgcn_readfirstlane(e / TJ);
#pragma unroll
        for (int b = 0; b < KJ; ++b)
            if (b == eb && tj == e % TJ)
#pragma unroll
                for (int a = 0; a < KI; ++a) {
                    col[ti + TI * a] = T[a][b];
                    T[a][b] = 0.0;             // the leaving variable's, but for row r
                }
        __syncthreads();
        // ratio test: the smallest rhs / col over rows with col > 0, then the
        // lowest basic variable among the rows within rounding of it
        double ratio[L], cl[L], rbest = INFINITY;
#pragma unroll
        for (int q = 0; q < L; ++q) {
            const int i = lane + 64 * q;
            cl[q] = i < NI ? col[i] : 0.0;
            ratio[q] = i < P && cl[q] > kLpEps ? rhs[q] / cl[q] : INFINITY;
            rbest = fmin(rbest, ratio[q]);
        }
        const double rmin = wave_min_f64(rbest);
        if (!(rmin < INFINITY))
            break;                             // unbounded: not reachable for M' > 0
        int bcand = INT_MAX;
#pragma unroll
        for (int q = 0; q < L; ++q)
            if (ratio[q] <= rmin + 1e-12 * fmax(1.0, rmin))
                bcand = min(bcand, bas[q] * 256 + lane + 64 * q);
        const int rv = wave_min_i32(bcand), r = rv & 255, rvar = rv >> 8;
        degenerate = rmin <= 0.0 ? degenerate + 1 : 0;
        const int rl = __builtin_amdgcn_readfirstlane(r & 63);
        double piv = cl[0], pr = ratio[0];     // pivot element, scaled right-hand side
#pragma unroll
        for (int q = 1; q < L; ++q) {
            piv = (r >> 6) == q ? cl[q] : piv;
            pr = (r >> 6) == q ? ratio[q] : pr;
        }
        piv = readlane_f64(piv, rl);
        pr = readlane_f64(pr, rl);
        // scaled pivot row: raw entries from the lanes that hold row r (all in
        // one wavefront), divided by that wavefront
        const int ra = __builtin_amdgcn_readfirstlane(r / TI);
        if (wave == __builtin_amdgcn_readfirstlane(r % TI / (64 / TJ))) {
#pragma unroll
            for (int a = 0; a < KI; ++a)
                if (a == ra && ti == r % TI)
#pragma unroll
                    for (int b = 0; b < KJ; ++b)
                        raw_s[tj + TJ * b] = T[a][b];
            wave_lds_sync();
#pragma unroll
            for (int q = 0; q < L; ++q) {
                const int j = lane + 64 * q;
                if (j < NJ)
                    prow_s[j] = (j == e ? 1.0 : raw_s[j]) / piv;
            }
        }
        __syncthreads();
        double pc[KJ];
#pragma unroll
        for (int b = 0; b < KJ; ++b)
            pc[b] = prow_s[tj + TJ * b];
#pragma unroll
        for (int a = 0; a < KI; ++a) {
            const double ca = col[ti + TI * a];
#pragma unroll
            for (int b = 0; b < KJ; ++b)
                T[a][b] -= ca * pc[b];
        }
#pragma unroll
        for (int a = 0; a < KI; ++a)
            if (a == ra && ti == r % TI)
#pragma unroll
                for (int b = 0; b < KJ; ++b)
                    T[a][b] = pc[b];
#pragma unroll
        for (int q = 0; q < L; ++q) {
            const int k = lane + 64 * q;
            const double pj = k < NJ ? prow_s[k] : 0.0;
            rc[q] = (k == e ? 0.0 : rc[q]) - rce * pj;
            rhs[q] = k == r ? pr : rhs[q] - cl[q] * pr;
            var[q] = k == e ? rvar : var[q];
            bas[q] = k == r ? evar : bas[q];
        }
        total -= rce * pr;
    }
    // ---- read the solution (every wavefront holds it; the first writes)
    const bool ok = done && total > 0.0;
    if (wave != 0)
        return;
#pragma unroll
    for (int q = 0; q < L; ++q) {
        xs[lane + 64 * q] = 0.0;
        ys[lane + 64 * q] = 0.0;
    }
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < L; ++q)
        if (lane + 64 * q < P) {
            if (var[q] >= P)
                xs[var[q] - P] = rc[q] / total;
            if (bas[q] < P)
                ys[bas[q]] = rhs[q] / total;
        }
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < L; ++q) {
        const int j = lane + 64 * q;
        if (j < P) {
            const double xv = ok ? xs[j] : (double)NAN, yv = ok ? ys[j] : (double)NAN;
            x[j] = xv;
            y[j] = yv;
            if (sigma) {
                sigma[j] = (float)xv;
                sigma[P + j] = (float)yv;
            }
        }
    }
    if (lane == 0) {
        *value = ok ? 1.0 / total + mn - 1.0 : (double)NAN;
        if (pivots)
            *pivots = done ? it : -1;
    }
}

bool lp_needs_work(int P)
{
    return P > kLpWorkAbove;
}

hipError_t launch_lp(const double* M, int P, int max_pivots, double* work, double* value,
                     double* x, double* y, float* sigma, int* pivots, hipStream_t s)
{
    if (P > kMaxP || (P > kLpRegMax && !work))
        return hipErrorInvalidValue;
    auto go = [&](auto kernel, int threads) {
        kernel<<<1, threads, 0, s>>>(M, P, max_pivots, value, x, y, sigma, pivots);
    };
    if (P <= 16)
        go(lp_reg_kernel<16, 16, 1, 1>, 256);
    else if (P <= 32)
        go(lp_reg_kernel<16, 16, 2, 2>, 256);
    else if (P <= 48)
        go(lp_reg_kernel<16, 16, 3, 3>, 256);
    else if (P <= 64)
        go(lp_reg_kernel<16, 16, 4, 4>, 256);
    else if (P <= 80)
        go(lp_reg_kernel<16, 16, 5, 5>, 256);
    else if (P <= 96)
        go(lp_reg_kernel<16, 16, 6, 6>, 256);
    else if (P <= 112)
        go(lp_reg_kernel<16, 16, 7, 7>, 256);
    else if (P <= 128)
        go(lp_reg_kernel<16, 16, 8, 8>, 256);
    else if (P <= 160)
        go(lp_reg_kernel<16, 32, 10, 5>, 512);
    else if (P <= 192)
        go(lp_reg_kernel<16, 32, 12, 6>, 512);
    else if (P <= kLpRegMax)
        go(lp_reg_kernel<16, 32, 14, 7>, 512);
    else
        lp_kernel<<<1, kLpThreads, 0, s>>>(M, P, max_pivots, work, value, x, y, sigma, pivots);
    return hipGetLastError();
}

// Thresholds of meta-sampling from device weights, the same fp64 arithmetic as
// the host path: T_m = floor(C_m / C_{P-1} * 2^32) from the sequential fp64
// cumulative sum C of row r, T_{P-1} = 2^32.  A row with a negative or
// non-finite weight or no positive mass gets T = 0 everywhere, which the
// sampling kernel turns into policy id -1 (flagged by the next rollout).
__global__ __launch_bounds__(64) void thresholds_kernel(const float* __restrict__ sigma, int P,
                                                        unsigned long long* __restrict__ thr)
{
    // one wavefront per row: lane 0 forms the sequential fp64 cumulative sum
    // (the order of the host path), every lane then converts its share
    __shared__ double run[kMaxP];
    const int r = blockIdx.x, lane = threadIdx.x;
    const float* s = sigma + (size_t)r * P;
    unsigned long long* T = thr + (size_t)r * P;
    bool ok = true;
    for (int m = lane; m < P; m += 64) {
        const float x = s[m];
        ok = ok && __builtin_isfinite(x) && x >= 0.0f;
    }
    if (lane == 0) {
        double c = 0.0;
        for (int m = 0; m < P; ++m) {
            c += (double)s[m];
            run[m] = c;
        }
    }
    __syncthreads();
    const double total = run[P - 1];
    ok = !__syncthreads_or(!ok) && total > 0.0;
    for (int m = lane; m < P; m += 64) {
        double c = floor(run[m] / total * 4294967296.0);
        if (c > 4294967296.0)
            c = 4294967296.0;
        T[m] = !ok ? 0ull : m == P - 1 ? 4294967296ull : (unsigned long long)c;
    }
}

hipError_t launch_thresholds(const float* sigma, int n_sigma, int P, unsigned long long* thr,
                             hipStream_t s)
{
    thresholds_kernel<<<n_sigma, 64, 0, s>>>(sigma, P, thr);
    return hipGetLastError();
}

}  // namespace malib
