// Environment kernels: reset, one step of each family with return
// accumulation, and the payoff-table reduction.
//
// State layouts (struct of arrays, coalesced per env index):
//   ITER_MATRIX  uint16 [n_envs]         joint action per lag in 4-bit fields,
//                                        lag 1 in the low nibble, 15 = none
//   PURSUIT      uint8  [2][n_envs]      pursuer cell, evader cell; done [n_envs]
//   FEATURE      fp32   [n_envs][d]      double-buffered between steps
// Returns: fp32 [n_agents][n_envs].
#include "device.hpp"
#include "feat_ring.hpp"
#include "internal.hpp"

namespace malib {

__device__ __forceinline__ int64_t traj_rec(const TrajArgs& tr, int t, int64_t n, int64_t e)
{
    return (tr.base + (int64_t)t * n + e) % tr.cap;
}


// ---------------------------------------------------------------- reset

// x[0..n) = 0 with a kernel rather than a memset node, so that a caller may
// capture the launch sequence in a HIP graph.
__global__ void zero_f32_kernel(float* __restrict__ x, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        x[i] = 0.0f;
}

hipError_t launch_zero_f32(float* x, int64_t n, hipStream_t s)
{
    if (n > 0)
        zero_f32_kernel<<<(int)((n + 255) / 256), 256, 0, s>>>(x, n);
    return hipGetLastError();
}

__global__ void reset_iter_kernel(uint16_t* __restrict__ hist, int64_t n)
{
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n)
        hist[e] = 0xFFFF;
}

// G x G torus: pursuer cell = floor(lane0 * G^2 / 2^32) (the top 6 bits of
// lane 0 when G = 8); evader = pursuer + 1 + floor(lane1 * (G^2 - 1) / 2^32)
// mod G^2, so the two never start on the same cell.
__global__ void reset_pursuit_kernel(uint8_t* __restrict__ pos, uint8_t* __restrict__ done,
                                     int64_t n, int grid, uint64_t seed, int64_t env_offset,
                                     int shared)
{
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n)
        return;
    uint64_t g = shared ? 0 : (uint64_t)(env_offset + e);
    u64x4 b = stream_block(seed, g, 0, kPurposeReset, 0, 0);
    uint32_t x0 = (uint32_t)b.x, x1 = (uint32_t)(b.x >> 32);
    uint32_t cells = (uint32_t)(grid * grid);
    uint32_t pc = (uint32_t)(((uint64_t)x0 * (uint64_t)cells) >> 32);
    uint32_t shift = (uint32_t)(((uint64_t)x1 * (uint64_t)(cells - 1)) >> 32);
    uint32_t ec = (pc + 1 + shift) % cells;
    pos[e] = (uint8_t)pc;
    pos[n + e] = (uint8_t)ec;
    done[e] = 0;
}

// s0[k] = (2*(x_k>>9)+1 - 2^23) * 2^-23 with x_k lane k%8 of block k/8.
// One thread per (env, block of 8 coordinates).
__global__ void reset_feature_kernel(float* __restrict__ s, uint16_t* __restrict__ obs, int64_t n,
                                     int d, uint64_t seed, int64_t env_offset, int shared)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int nb = d / 8;
    if (i >= n * nb)
        return;
    int64_t e = i / nb;
    int blk = (int)(i - e * nb);
    uint64_t g = shared ? 0 : (uint64_t)(env_offset + e);
    u64x4 b = stream_block(seed, g, 0, kPurposeReset, 0, (uint64_t)blk);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        int32_t odd = (int32_t)(2u * (block_lane(b, j) >> 9) + 1u);
        v[j] = (float)(odd - (1 << 23)) * 0x1p-23f;
    }
    float4* dst = reinterpret_cast<float4*>(s + e * d + blk * 8);
    dst[0] = make_float4(v[0], v[1], v[2], v[3]);
    dst[1] = make_float4(v[4], v[5], v[6], v[7]);
    if (obs)
        *reinterpret_cast<uint4*>(obs + e * d + blk * 8) =
            make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                       pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
}

hipError_t launch_reset(const EnvArgs& e, int64_t n_envs, uint64_t seed, int64_t env_offset,
                        void* state, uint8_t* done, hipStream_t s)
{
    int shared = e.init_mode == MALIB_INIT_SHARED;
    if (e.kind == MALIB_ENV_ITER_MATRIX) {
        reset_iter_kernel<<<(int)((n_envs + 255) / 256), 256, 0, s>>>((uint16_t*)state, n_envs);
    } else if (e.kind == MALIB_ENV_PURSUIT) {
        reset_pursuit_kernel<<<(int)((n_envs + 255) / 256), 256, 0, s>>>(
            (uint8_t*)state, done, n_envs, e.grid, seed, env_offset, shared);
    } else if (e.kind == MALIB_ENV_FEATURE) {
        int64_t total = n_envs * (e.d / 8);
        reset_feature_kernel<<<(int)((total + 255) / 256), 256, 0, s>>>(
            (float*)state, e.obs, n_envs, e.d, seed, env_offset, shared);
    }
    return hipGetLastError();
}

// W [d][d] -> the A operands of v_mfma_f32_16x16x4_f32, lane by lane:
// WP[nt][g][lane][j] = W[16 nt + lane % 16][16 g + 4 j + lane / 16], so a lane
// loads its operands of four consecutive k-steps (16 inputs) as 16 bytes and a
// wavefront 1 KiB contiguous.
__global__ void pack_dynamics_kernel(const float* __restrict__ W, float* __restrict__ WP, int d)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= d * d)
        return;
    const int j = i & 3, lane = (i >> 2) & 63, r = i >> 8, gs = d / 16;
    const int nt = r / gs, g = r - nt * gs;
    WP[i] = W[(16 * nt + (lane & 15)) * d + 16 * g + 4 * j + (lane >> 4)];
}

hipError_t launch_pack_dynamics(const float* W, float* WP, int d, hipStream_t s)
{
    pack_dynamics_kernel<<<(d * d + 255) / 256, 256, 0, s>>>(W, WP, d);
    return hipGetLastError();
}

// ------------------------------- iterated game and pursuit, step by step

// The two seats' actions of env e (Gumbel-max over their logits, logged when
// asked); a NaN logit raises kErrNaN.
template <int AMAX>
__device__ __forceinline__ void sample_pair(const SampleArgs& sa, int A, int64_t e, int& a0,
                                            int& a1)
{
    bool n0, n1;
    const uint64_t g = (uint64_t)(sa.env_offset + e);
    a0 = gumbel_action<AMAX>(sa.logits + (2 * e) * A, A, sa.seed, g, sa.t, 0, n0);
    a1 = gumbel_action<AMAX>(sa.logits + (2 * e + 1) * A, A, sa.seed, g, sa.t, 1, n1);
    if (n0 || n1)
        atomicOr(sa.flags, kErrNaN);
    if (sa.log) {
        sa.log[2 * e] = (uint8_t)a0;
        sa.log[2 * e + 1] = (uint8_t)a1;
    }
}

// Iterated game, one thread per env: both seats' actions (at most 3), r0 =
// A[a0][a1], r1 = -r0, the joint action shifted into the history.
__global__ void step_iter_kernel(const float* __restrict__ Amat, int A, int64_t n, SampleArgs sa,
                                 TrajArgs tr, uint16_t* __restrict__ hist,
                                 float* __restrict__ ret)
{
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n)
        return;
    int a0, a1;
    sample_pair<8>(sa, A, e, a0, a1);
    float v = Amat[a0 * A + a1];
    ret[e] = ret[e] + v;
    ret[n + e] = ret[n + e] + (-v);
    const uint32_t h = hist[e];
    hist[e] = (uint16_t)(((h << 4) | (uint32_t)(a0 * 3 + a1)) & 0xFFFFu);
    if (tr.act) {
        const int64_t r = traj_rec(tr, sa.t, n, e);
        tr.act[2 * r] = (uint8_t)a0;
        tr.act[2 * r + 1] = (uint8_t)a1;
        tr.rew[r] = v;
        tr.flags[r] = sa.t == tr.horizon - 1 ? 2 : 0;
        if (tr.obs)
            ((uint16_t*)tr.obs)[r] = (uint16_t)h;
    }
}

__device__ __forceinline__ uint32_t torus_move(uint32_t cell, int a, int grid)
{
    int x = (int)cell % grid, y = (int)cell / grid;
    if (a == 1)
        y = (y + grid - 1) % grid;
    else if (a == 2)
        y = (y + 1) % grid;
    else if (a == 3)
        x = (x + grid - 1) % grid;
    else if (a == 4)
        x = (x + 1) % grid;
    return (uint32_t)(y * grid + x);
}

// One thread per slot (lanes 2e and 2e+1: pursuer and evader of env e), all
// loads issued first: each lane samples its seat's action (5 actions), the
// pair exchange them, and the pursuer's lane makes the simultaneous moves;
// capture if the two land on the same cell or swap cells: pursuer +1, evader
// -1, env done.  Finished envs take no action (logged as 255).  Counts live
// agent-frames (two per live env) with one atomic per workgroup.
__global__ __launch_bounds__(256) void step_pursuit_kernel(
    int grid, int64_t n, SampleArgs sa, TrajArgs tr, uint8_t* __restrict__ pos,
    uint8_t* __restrict__ done, float* __restrict__ ret, unsigned long long* frames)
{
    __shared__ int live_s;
    if (threadIdx.x == 0)
        live_s = 0;
    __syncthreads();
    const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t e = slot >> 1;
    const int seat = (int)(slot & 1);
    const bool valid = e < n;                 // both lanes of a pair agree
    const int64_t ec = valid ? e : 0;
    const bool dn = done[ec] != 0;
    const uint32_t p0 = pos[ec], q0 = pos[n + ec];
    bool nan = false;
    const int a = gumbel_action<8>(sa.logits + (valid ? slot : 0) * 5, 5, sa.seed,
                                   (uint64_t)(sa.env_offset + ec), sa.t, seat, nan);
    const int a_other = __shfl_xor(a, 1);
    const bool live = valid && !dn;
    if (live && nan)
        atomicOr(sa.flags, kErrNaN);
    if (valid && sa.log)
        sa.log[slot] = live ? (uint8_t)a : (uint8_t)255;
    bool caught = false;
    if (live && seat == 0) {
        const uint32_t p1 = torus_move(p0, a, grid);
        const uint32_t q1 = torus_move(q0, a_other, grid);
        pos[e] = (uint8_t)p1;
        pos[n + e] = (uint8_t)q1;
        if (p1 == q1 || (p1 == q0 && q1 == p0)) {
            caught = true;
            done[e] = 1;
            ret[e] = ret[e] + 1.0f;
            ret[n + e] = ret[n + e] + (-1.0f);
        }
    }
    if (valid && tr.act) {
        const int64_t r = traj_rec(tr, sa.t, n, e);
        tr.act[2 * r + seat] = live ? (uint8_t)a : (uint8_t)255;
        if (seat == 0) {
            tr.rew[r] = caught ? 1.0f : 0.0f;
            tr.flags[r] = (uint8_t)((caught ? 1 : 0) | (sa.t == tr.horizon - 1 ? 2 : 0) |
                                    (dn ? 4 : 0));
            if (tr.obs) {
                uint8_t* o = (uint8_t*)tr.obs + 2 * r;
                o[0] = (uint8_t)p0;
                o[1] = (uint8_t)q0;
            }
        }
    }
    const unsigned long long b = __ballot(live && seat == 0);
    if ((threadIdx.x & 63) == 0 && b)
        atomicAdd(&live_s, __popcll(b));
    __syncthreads();
    if (threadIdx.x == 0 && live_s)
        atomicAdd(frames, (unsigned long long)live_s * 2ull);
}

// ------------------------------------------------------------ feature dynamics

// GW consecutive floats (GW = 1, 2 or 4) as one load or store: outputs are
// mapped to threads in groups of GW consecutive indices, so the accumulator rows
// in LDS, the embedding loads and the state stores are single wide accesses.
template <int GW>
struct FVec;
template <>
struct FVec<1> {
    float v[1];
    __device__ __forceinline__ void load(const float* p) { v[0] = *p; }
    __device__ __forceinline__ void store(float* p) const { *p = v[0]; }
};
template <>
struct FVec<2> {
    float v[2];
    __device__ __forceinline__ void load(const float* p)
    {
        typedef float v2f __attribute__((ext_vector_type(2)));
        const v2f t = *reinterpret_cast<const v2f*>(p);
        v[0] = t.x;
        v[1] = t.y;
    }
    __device__ __forceinline__ void store(float* p) const
    {
        typedef float v2f __attribute__((ext_vector_type(2)));
        *reinterpret_cast<v2f*>(p) = v2f{v[0], v[1]};
    }
};
template <>
struct FVec<4> {
    float v[4];
    __device__ __forceinline__ void load(const float* p)
    {
        typedef float v4f __attribute__((ext_vector_type(4)));
        const v4f t = *reinterpret_cast<const v4f*>(p);
        v[0] = t.x;
        v[1] = t.y;
        v[2] = t.z;
        v[3] = t.w;
    }
    __device__ __forceinline__ void store(float* p) const
    {
        typedef float v4f __attribute__((ext_vector_type(4)));
        *reinterpret_cast<v4f*>(p) = v4f{v[0], v[1], v[2], v[3]};
    }
};

// bf16_rne of GW consecutive floats as one 2-, 4- or 8-byte store.
template <int GW>
__device__ __forceinline__ void store_bf16(uint16_t* p, const FVec<GW>& t)
{
    if constexpr (GW == 1) {
        *p = bf16_bits(t.v[0]);
    } else if constexpr (GW == 2) {
        *reinterpret_cast<uint32_t*>(p) = pack_bf16x2(t.v[0], t.v[1]);
    } else {
        *reinterpret_cast<uint2*>(p) =
            make_uint2(pack_bf16x2(t.v[0], t.v[1]), pack_bf16x2(t.v[2], t.v[3]));
    }
}

// Feature dynamics, for every env e and output k:
//   s'[e][k] = tanh_ref( fma-chain_{c=0..D-1}(W[k][c], s[e][c]) + emb[0][a_0][k]
//                        + emb[1][a_1][k] + ... )
// then the reward r = u . s', a sequential fused chain per env.
//
// The chains run on the matrix cores: v_mfma_f32_16x16x4_f32 adds its four
// products to the accumulator one after the other in ascending k, each as a
// fused multiply-add with one rounding (compared bit for bit with a VALU chain,
// subnormals, infinities and NaN included), so an accumulator that starts at 0
// and takes the inputs in ascending order holds exactly the sequential fused
// chain.  A = W (16 outputs x 4 inputs, packed by pack_dynamics_kernel and read
// from the L2, 1 KiB per wavefront for 16 inputs), B = the state (4 inputs x 16
// envs) from LDS, where the 16 inputs of a group sit in the operand order (input
// 4 j + m at 4 m + j), so a lane reads its operands of four k-steps as 16 bytes.
//
// A tile is E = 16 RT envs.  Its accumulators go through LDS to one wavefront
// per env, lane tx taking groups of GW consecutive outputs, so that the
// embedding rows are read and the state rows written as whole lines.
//
// Bound: fp32 MFMA and VALU instructions share a SIMD's cycles (wavefronts doing
// the one and the other take the sum of their times: 126 + 215 -> 334 us
// measured), so the time is the chains at 157 TFLOP/s plus the VALU work, about
// 50 instructions per output, mostly tanh_ref.  A fused-multiply-add chain on
// the VALU takes twice the chains' time: d = 512, 65536 envs, 2 seats 486 ->
// 311 us (110 TFLOP/s; MFMA 65% and VALU 20% of the cycles); d = 256, 16384
// envs, 8 seats 44 -> 35 us (half of it the state's 42 MB and latencies).
// Splitting the wavefronts into MFMA and epilogue ones with the next tile's
// loads in flight gains nothing for that reason (389 and 44 us).
template <int D, int RT, int WAVES>
struct FeatTile {
    static constexpr int E = 16 * RT;
    static constexpr int KG = D / 16;               // groups of 16 inputs
    static constexpr int NTW = D / 16 / WAVES;      // output tiles per wavefront
    static constexpr int EPW = E / WAVES;           // envs per wavefront in the epilogue
    static constexpr int NJ = D / 64;               // outputs per lane and env in the epilogue
    static constexpr int GW = NJ < 4 ? NJ : 4;      // ... in groups of GW consecutive ones
    static constexpr int NG = NJ / GW;              // output k of (g, j) = g*64*GW + GW*tx + j
    static constexpr int SLD = D + 4;               // env row stride in LDS (rows 4 banks apart)
    static constexpr int Q4 = D / 4;
    static constexpr int SQ = E * Q4 / (64 * WAVES);   // state float4s per thread
    static_assert(NTW * WAVES * 16 == D && EPW * WAVES == E && SQ * 64 * WAVES == E * Q4, "split");
    static_assert(EPW * kMaxAgents <= 64, "an epilogue wavefront takes its envs' given actions "
                                          "with one lane per slot");
};

typedef float v4f_t __attribute__((ext_vector_type(4)));

struct FeatArgs {
    const float* WP;
    const float* emb;
    const float* u;
    EnvArgs ea;
    SampleArgs sa;
    int64_t n;
    const float* s_in;
    float* s_out;
    float* ret;
};

// The tile's state rows -> registers (envs past the end: zeros, never stored).
template <class T>
__device__ __forceinline__ void feat_load_state(const FeatArgs& f, int64_t e0, int st,
                                                int threads, v4f_t (&sreg)[T::SQ])
{
#pragma unroll
    for (int q = 0; q < T::SQ; ++q) {
        const int i = q * threads + st, el = i / T::Q4, c4 = i - el * T::Q4;
        sreg[q] = v4f_t{0.f, 0.f, 0.f, 0.f};
        if (e0 + el < f.n)
            sreg[q] = *reinterpret_cast<const v4f_t*>(f.s_in + (e0 + el) * (4 * T::Q4) + 4 * c4);
    }
}

// Trajectory observation of the step: bf16(s) of the staged rows.
template <class T>
__device__ __forceinline__ void feat_record_obs(const FeatArgs& f, int64_t e0, int st,
                                                int threads, const v4f_t (&sreg)[T::SQ])
{
    const TrajArgs& tr = f.ea.tr;
    if (!tr.obs)
        return;
    const int64_t rec0 = traj_rec(tr, f.sa.t, f.n, e0);
#pragma unroll
    for (int q = 0; q < T::SQ; ++q) {
        const int i = q * threads + st, el = i / T::Q4, c4 = i - el * T::Q4;
        int64_t rec = rec0 + el;
        if (rec >= tr.cap)
            rec %= tr.cap;
        if (e0 + el < f.n)
            *reinterpret_cast<uint2*>((uint16_t*)tr.obs + rec * (4 * T::Q4) + 4 * c4) =
                make_uint2(pack_bf16x2(sreg[q].x, sreg[q].y), pack_bf16x2(sreg[q].z, sreg[q].w));
    }
}

// The staged rows -> LDS in operand order.
template <class T>
__device__ __forceinline__ void feat_stage_state(float* Ss, int st, int threads,
                                                 const v4f_t (&sreg)[T::SQ])
{
#pragma unroll
    for (int q = 0; q < T::SQ; ++q) {
        const int i = q * threads + st, el = i / T::Q4, c4 = i - el * T::Q4;
        float* dst = Ss + el * T::SLD + (c4 >> 2) * 16 + (c4 & 3);
        dst[0] = sreg[q].x;
        dst[4] = sreg[q].y;
        dst[8] = sreg[q].z;
        dst[12] = sreg[q].w;
    }
}

// W operands through a buffer resource: base and size in scalar registers, one
// lane offset for all loads, the (wave-uniform) operand block's offset in a
// scalar register, so the main loop spends no VALU on addresses (VALU and fp32
// MFMA share a SIMD's cycles).
using WSrc = __amdgpu_buffer_rsrc_t;

__device__ __forceinline__ v4f_t load_w4(WSrc src, int blk, int loff)
{
    return __builtin_bit_cast(v4f_t,
                              __builtin_amdgcn_raw_buffer_load_b128(src, loff, blk * 1024, 0));
}

// The chains of wavefront mw's output tiles over the staged state; the ring
// holds groups 0 .. DEPTH-1 on entry.  The last round of the ring stands by itself,
// without refills: those would lie past the tile's blocks, and for the last tile
// past W (a buffer resource's range check does not cover the scalar offset).
// Against a refill clamped to the tile's last block: d = 256, 5003 envs of 8 seats
// 24.6 -> 23.7 us a step, 16384 envs 39.5 -> 38.3; d = 512, 8192 envs 55 -> 53.
template <class T, int RT, int DEPTH>
__device__ __forceinline__ void feat_mfma(WSrc W, const float* Ss, int mw, int tx,
                                          v4f_t (&a)[DEPTH][T::NTW], v4f_t (&acc)[T::NTW][RT])
{
    static_assert(T::KG % DEPTH == 0, "whole rounds of the ring");
#pragma unroll
    for (int i = 0; i < T::NTW; ++i)
#pragma unroll
        for (int r = 0; r < RT; ++r)
            acc[i][r] = v4f_t{0.f, 0.f, 0.f, 0.f};
    const float* bp = Ss + (tx & 15) * T::SLD + 4 * (tx >> 4);
    auto round = [&](int g0, auto refill) {
#pragma unroll
        for (int h = 0; h < DEPTH; ++h) {
            const int g = g0 + h;
            v4f_t b[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r)
                b[r] = *reinterpret_cast<const v4f_t*>(bp + 16 * r * T::SLD + 16 * g);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < T::NTW; ++i)
#pragma unroll
                    for (int r = 0; r < RT; ++r)
                        acc[i][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h][i][j], b[r][j],
                                                                         acc[i][r], 0, 0, 0);
            if constexpr (decltype(refill)::value)
#pragma unroll
                for (int i = 0; i < T::NTW; ++i)
                    a[h][i] = load_w4(W, feat_block(mw * T::NTW + i, g + DEPTH, T::KG), tx * 16);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int g0 = 0;
#pragma unroll 1
    for (; feat_refills(g0, DEPTH, T::KG); g0 += DEPTH)
        round(g0, std::true_type{});
    round(g0, std::false_type{});
}

// Accumulators -> Ss[env][k] (lane: env tx % 16 of its row tile, 4 outputs).
template <class T, int RT>
__device__ __forceinline__ void feat_store_acc(float* Ss, int mw, int tx,
                                               const v4f_t (&acc)[T::NTW][RT])
{
#pragma unroll
    for (int i = 0; i < T::NTW; ++i)
#pragma unroll
        for (int r = 0; r < RT; ++r)
            *reinterpret_cast<v4f_t*>(Ss + (16 * r + (tx & 15)) * T::SLD +
                                      16 * (mw * T::NTW + i) + 4 * (tx >> 4)) = acc[i][r];
}

// The actions of epilogue wavefront ew's envs -> act (bytes [EPW][kMaxAgents]):
// read where the policy kernel sampled them, else Gumbel-max over the slot's
// logits, four lanes per slot, lane b taking Philox block b (actions 8b .. 8b+7);
// the slot's best is combined by two shuffles (larger z, the lower action on
// equal z).  Envs past the end take action 0.
// (given: this lane's byte of the former, loaded by the caller).
template <class T>
__device__ __forceinline__ void feat_actions(const FeatArgs& f, int64_t e0, int ew, int tx,
                                             int given, uint8_t* act)
{
    const EnvArgs& ea = f.ea;
    const SampleArgs& sa = f.sa;
    const int slots = T::EPW * ea.n_agents;
    auto put = [&](int i, int el, int64_t e, int a) {
        const int seat = i - (el - ew * T::EPW) * ea.n_agents;
        if (e < f.n) {
            if (sa.log)
                sa.log[e * ea.n_agents + seat] = (uint8_t)a;
            if (ea.tr.act)
                ea.tr.act[traj_rec(ea.tr, sa.t, f.n, e) * ea.n_agents + seat] = (uint8_t)a;
        }
        act[(el - ew * T::EPW) * kMaxAgents + seat] = (uint8_t)a;
    };
    if (sa.actions) {
        if (tx < slots) {   // one lane per slot
            const int el = ew * T::EPW + tx / ea.n_agents;
            put(tx, el, e0 + el, given);
        }
    } else {
        for (int i0 = 0; i0 < slots; i0 += 16) {
            const int i = i0 + (tx >> 2), b = tx & 3;
            const int el = ew * T::EPW + i / ea.n_agents;
            const int64_t e = e0 + el;
            const bool live = i < slots && e < f.n;
            float zbest = -__builtin_inff();
            int best = -1;
            bool bad = false;
            if (live && 8 * b < ea.A) {
                const int seat = i - (el - ew * T::EPW) * ea.n_agents;
                const float* l = sa.logits + (e * ea.n_agents + seat) * ea.A;
                float lv[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    lv[j] = l[8 * b + j < ea.A ? 8 * b + j : ea.A - 1];
                const u64x4 blk = stream_block(sa.seed, (uint64_t)(sa.env_offset + e),
                                               (uint64_t)sa.t, kPurposeAction, (uint32_t)seat,
                                               (uint64_t)b);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float z = lv[j] + gumbel01(uniform01(block_lane(blk, j)));
                    bad |= __builtin_isnan(lv[j]);
                    if (8 * b + j < ea.A && (best < 0 || z > zbest)) {
                        zbest = z;
                        best = 8 * b + j;
                    }
                }
            }
#pragma unroll
            for (int m = 1; m <= 2; m <<= 1) {
                const float zo = __shfl_xor(zbest, m, 64);
                const int bo = __shfl_xor(best, m, 64);
                if (bo >= 0 && (best < 0 || zo > zbest || (zo == zbest && bo < best))) {
                    zbest = zo;
                    best = bo;
                }
                bad |= __shfl_xor((int)bad, m, 64) != 0;
            }
            if (b == 0 && i < slots) {
                if (live && bad)
                    atomicOr(sa.flags, kErrNaN);
                put(i, el, e, live && !bad ? best : 0);
            }
        }
    }
    wave_lds_sync();
}

// Epilogue of wavefront ew's envs (rows of Ss, all outputs of an env in one
// wavefront): embeddings in seat order, tanh_ref, s' out and back into Ss.
template <class T>
__device__ __forceinline__ void feat_epilogue(const FeatArgs& f, int64_t e0, float* Ss,
                                              const uint8_t* act, int ew, int tx)
{
    constexpr int EPW = T::EPW, GW = T::GW, NG = T::NG, D = 4 * T::Q4;
    const EnvArgs& ea = f.ea;
    // all embedding loads of an env are issued together.  The env is the same
    // for all lanes: its action bytes, and with them the embedding rows'
    // addresses, are kept in scalar registers.
#pragma unroll
    for (int i = 0; i < EPW; ++i) {
        const int el = ew * EPW + i;
        const int64_t e = e0 + el;
        const uint64_t pk = *reinterpret_cast<const uint64_t*>(act + i * kMaxAgents);
        const uint64_t acts =
            (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)pk) |
            ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(pk >> 32)) << 32);
        FVec<GW> t[kMaxAgents][NG];
#pragma unroll
        for (int q = 0; q < kMaxAgents; ++q)
            if (q < ea.n_agents) {
                const int a_q = (int)((acts >> (8 * q)) & 0xFFu);
                const float* row = f.emb + (q * ea.A + a_q) * D + GW * tx;
#pragma unroll
                for (int g = 0; g < NG; ++g)
                    t[q][g].load(row + g * 64 * GW);
            }
        FVec<GW> pre[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g)
            pre[g].load(Ss + el * T::SLD + g * 64 * GW + GW * tx);
#pragma unroll
        for (int q = 0; q < kMaxAgents; ++q)
            if (q < ea.n_agents)
#pragma unroll
                for (int g = 0; g < NG; ++g)
#pragma unroll
                    for (int j = 0; j < GW; ++j)
                        pre[g].v[j] = pre[g].v[j] + t[q][g].v[j];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int k0 = g * 64 * GW + GW * tx;
#pragma unroll
            for (int j = 0; j < GW; ++j)
                pre[g].v[j] = tanh_ref(pre[g].v[j]);
            if (e < f.n) {
                pre[g].store(f.s_out + e * D + k0);
                if (ea.obs)
                    store_bf16<GW>(ea.obs + e * D + k0, pre[g]);
            }
            pre[g].store(Ss + el * T::SLD + k0);
        }
    }
}

// One tile per workgroup.  Two 32-env workgroups share a CU; a batch of at most
// one 16-env tile per CU takes 16 wavefronts per tile, being bound by one tile's
// latency.
template <int D, int RT, int WAVES, int DEPTH>
__global__ __launch_bounds__(64 * WAVES, 4) void step_feature_kernel(FeatArgs f)
{
    using T = FeatTile<D, RT, WAVES>;
    constexpr int THREADS = 64 * WAVES;
    __shared__ __attribute__((aligned(16))) float Ss[T::E * T::SLD];
    // the reward weights u, staged once: the chain reads both operands from LDS
    __shared__ __attribute__((aligned(16))) float Us[D];
    __shared__ __attribute__((aligned(8))) uint8_t act_s[T::E * kMaxAgents];
    const int tid = threadIdx.x, tx = tid & 63;
    const int ty = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t e0 = (int64_t)blockIdx.x * T::E;
    const EnvArgs& ea = f.ea;
    v4f_t sreg[T::SQ], a[DEPTH][T::NTW], acc[T::NTW][RT];
    feat_load_state<T>(f, e0, tid, THREADS, sreg);
    // u and the given actions before W: loads complete in order
    constexpr int UQ = (D + THREADS - 1) / THREADS;
    float ureg[UQ];
#pragma unroll
    for (int k = 0; k < UQ; ++k)
        ureg[k] = k * THREADS + tid < D ? f.u[k * THREADS + tid] : 0.f;
    const int64_t slot0 = (e0 + ty * T::EPW) * ea.n_agents + tx;
    int given = 0;
    if (f.sa.actions && tx < T::EPW * ea.n_agents && slot0 < f.n * ea.n_agents)
        given = f.sa.actions[slot0];
    const WSrc W = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(f.WP), (short)0,
                                                     D * D * 4, 0x00020000);
    auto fill = [&] {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s)
#pragma unroll
            for (int i = 0; i < T::NTW; ++i)
                a[s][i] = load_w4(W, feat_block(ty * T::NTW + i, s, T::KG), tx * 16);
    };
    // the first W operands at once where registers allow, else after the actions
    constexpr bool kEarly = DEPTH * T::NTW + T::SQ <= 12;
    if constexpr (kEarly)
        fill();
#pragma unroll
    for (int k = 0; k < UQ; ++k)
        if (k * THREADS + tid < D)
            Us[k * THREADS + tid] = ureg[k];
    uint8_t* act = act_s + ty * T::EPW * kMaxAgents;
    feat_actions<T>(f, e0, ty, tx, given, act);
    if constexpr (!kEarly)
        fill();
    feat_stage_state<T>(Ss, tid, THREADS, sreg);
    feat_record_obs<T>(f, e0, tid, THREADS, sreg);
    __syncthreads();
    feat_mfma<T, RT, DEPTH>(W, Ss, ty, tx, a, acc);
    __syncthreads();   // every wavefront is done with the state rows
    feat_store_acc<T, RT>(Ss, ty, tx, acc);
    __syncthreads();
    feat_epilogue<T>(f, e0, Ss, act, ty, tx);
    // reward chain of the workgroup's envs (one lane each); the seats' running
    // returns are fetched before the chain so their latency overlaps it, and
    // the chain is unrolled so that its LDS loads run ahead of the dependent
    // FMAs
    const int64_t er = e0 + tid;
    const bool rlane = tid < T::E && er < f.n;
    float rv[kMaxAgents];
#pragma unroll
    for (int q = 0; q < kMaxAgents; ++q)
        if (rlane && q < ea.n_agents)
            rv[q] = f.ret[(int64_t)q * f.n + er];
    __syncthreads();
    if (rlane) {
        float r = 0.0f;
        const float* row = Ss + tid * T::SLD;
#pragma unroll 64
        for (int k = 0; k < D; ++k)
            r = __builtin_fmaf(Us[k], row[k], r);
#pragma unroll
        for (int q = 0; q < kMaxAgents; ++q)
            if (q < ea.n_agents)
                f.ret[(int64_t)q * f.n + er] = rv[q] + (((ea.team_row >> q) & 1u) ? r : -r);
        if (ea.tr.rew) {
            const int64_t rec = traj_rec(ea.tr, f.sa.t, f.n, er);
            ea.tr.rew[rec] = r;
            ea.tr.flags[rec] = f.sa.t == ea.tr.horizon - 1 ? 2 : 0;
        }
    }
}

template <int D, int RT, int WAVES, int DEPTH>
static void launch_feature(const FeatArgs& f, hipStream_t s)
{
    const int blocks = (int)((f.n + 16 * RT - 1) / (16 * RT));
    step_feature_kernel<D, RT, WAVES, DEPTH><<<blocks, 64 * WAVES, 0, s>>>(f);
}

hipError_t launch_env_step(const EnvArgs& e, const SampleArgs& sa, int64_t n_envs,
                           const void* state_in, void* state_out, uint8_t* done, float* ret,
                           unsigned long long* frames, hipStream_t s)
{
    int blocks = (int)((n_envs + 255) / 256);
    switch (e.kind) {
    case MALIB_ENV_ITER_MATRIX:
        if (e.A > 3)
            return hipErrorInvalidValue;
        step_iter_kernel<<<blocks, 256, 0, s>>>(e.Amat, e.A, n_envs, sa, e.tr,
                                                (uint16_t*)state_out, ret);
        break;
    case MALIB_ENV_PURSUIT:
        if (e.A != 5)
            return hipErrorInvalidValue;
        // one thread per slot
        step_pursuit_kernel<<<(int)((2 * n_envs + 255) / 256), 256, 0, s>>>(
            e.grid, n_envs, sa, e.tr, (uint8_t*)state_out, done, ret, frames);
        break;
    case MALIB_ENV_FEATURE: {
        if (e.A > kMaxActions)
            return hipErrorInvalidValue;
        const FeatArgs f{e.WP, e.emb, e.u, e, sa, n_envs, (const float*)state_in,
                         (float*)state_out, ret};
        // 32-env tiles read half as much of W per env, 16-env ones spread a
        // batch better: up to one per CU (n <= 16 cus), and again where some CUs
        // would get two 32-env tiles and others one (32 cus < n <= 48 cus).  us
        // a step with 32- and with 16-env tiles, 256 CUs: d = 64 7.2 / 5.8 (5003
        // envs), 8.7 / 7.7 (16384), 10.3 / 10.6 (20480); d = 128 9.2 / 9.0
        // (5003), 13.1 / 12.3 (10000), 13.8 / 14.6 (13000); d = 256 19.9 / 19.0
        // (5003), 30.8 / 27.5 (10000), 32.0 / 34.6 (13000); d = 512 45.9 / 45.3
        // (5003), 49.7 / 51.3 (8192), 79.0 / 70.6 (10000), 81 / 88 (13000).
        // One 16-env tile per CU takes more wavefronts (257 envs of 8 seats at
        // d = 256: 12.8 us with 8, 12.2 with 16).
        const int64_t cus = e.n_cus > 0 ? e.n_cus : 256;
        const bool one = n_envs <= 16 * cus, two = n_envs <= 32 * cus;
        const bool three = n_envs <= 48 * cus, four = n_envs <= 64 * cus;
        if (e.d == 64 && four)
            launch_feature<64, 1, 4, 4>(f, s);
        else if (e.d == 64)
            launch_feature<64, 2, 4, 4>(f, s);
        else if (e.d == 128 && two)
            launch_feature<128, 1, 8, 8>(f, s);
        else if (e.d == 128 && three)
            launch_feature<128, 1, 4, 4>(f, s);
        else if (e.d == 128)
            launch_feature<128, 2, 8, 4>(f, s);
        else if (e.d == 256 && one)
            launch_feature<256, 1, 16, 8>(f, s);
        else if (e.d == 256 && three)
            launch_feature<256, 1, 8, 4>(f, s);
        else if (e.d == 256)
            launch_feature<256, 2, 8, 2>(f, s);
        else if (e.d == 512 && one)
            launch_feature<512, 1, 16, 4>(f, s);
        else if (e.d == 512 && three && !two)
            launch_feature<512, 1, 8, 4>(f, s);
        else if (e.d == 512)
            launch_feature<512, 2, 8, 2>(f, s);
        else
            return hipErrorInvalidValue;
        break;
    }
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// PURSUIT snapshot in the trace format [n_envs][3] = (pursuer, evader, done).
__global__ void snapshot_pursuit_kernel(const uint8_t* __restrict__ pos,
                                        const uint8_t* __restrict__ done, int64_t n,
                                        uint8_t* __restrict__ out)
{
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n)
        return;
    out[3 * e] = pos[e];
    out[3 * e + 1] = pos[n + e];
    out[3 * e + 2] = done[e];
}

hipError_t launch_snapshot_pursuit(const void* state, const uint8_t* done, int64_t n_envs,
                                   uint8_t* out, hipStream_t s)
{
    snapshot_pursuit_kernel<<<(int)((n_envs + 255) / 256), 256, 0, s>>>(
        (const uint8_t*)state, done, n_envs, out);
    return hipGetLastError();
}

// ------------------------------------------------------------ payoff reduction

// One thread per env.  Every (row-side seat a, column-side seat b) pair adds
// the fixed-point return of seat a (2^-32 units; squares in 2^-20 units) and a
// count to cell (pid[a], pid[b]).  When a whole wavefront targets one cell
// (blocked assignments), it reduces with shuffles and issues one set of
// atomics; otherwise each lane adds its own.
__device__ __forceinline__ long long wave_sum_i64(long long v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v += __shfl_xor(v, off, 64);
    return v;
}

__global__ __launch_bounds__(256) void payoff_kernel(
    const float* __restrict__ ret, const int32_t* __restrict__ pids, int64_t n, int n_agents,
    EnvArgs ea, int P, unsigned long long* __restrict__ sum,
    unsigned long long* __restrict__ sumsq, unsigned long long* __restrict__ cnt)
{
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool valid = e < n;
    for (int a = 0; a < n_agents; ++a) {
        if (!((ea.team_row >> a) & 1u))
            continue;
        long long fx = 0, fsq = 0;
        if (valid) {
            double g = (double)ret[(int64_t)a * n + e];
            fx = __double2ll_rn(g * 4294967296.0);
            fsq = __double2ll_rn(g * g * 1048576.0);
        }
        for (int b = 0; b < n_agents; ++b) {
            if (!((ea.team_col >> b) & 1u))
                continue;
            int cell = -1;
            if (valid) {
                int pa = pids[e * n_agents + a], pb = pids[e * n_agents + b];
                if (pa >= 0 && pa < P && pb >= 0 && pb < P)
                    cell = pa * P + pb;
            }
            int c0 = __shfl(cell, 0, 64);
            bool uniform = __ballot(cell != c0) == 0ull;
            if (uniform) {
                if (c0 >= 0) {
                    long long s1 = wave_sum_i64(fx), s2 = wave_sum_i64(fsq);
                    long long c = wave_sum_i64(cell >= 0 ? 1 : 0);
                    if ((threadIdx.x & 63) == 0) {
                        atomicAdd(&sum[c0], (unsigned long long)s1);
                        atomicAdd(&sumsq[c0], (unsigned long long)s2);
                        atomicAdd(&cnt[c0], (unsigned long long)c);
                    }
                }
            } else if (cell >= 0) {
                atomicAdd(&sum[cell], (unsigned long long)fx);
                atomicAdd(&sumsq[cell], (unsigned long long)fsq);
                atomicAdd(&cnt[cell], 1ull);
            }
        }
    }
}

// Small populations (P*P cells fit one workgroup's LDS): each workgroup walks
// a contiguous range of envs in env order (coalesced reads of the returns and
// ids) and reduces every incidence into a private copy of the whole table in
// LDS: one LDS atomic per incidence, or, where a whole wavefront targets one
// cell (blocked assignments), a shuffle reduction and one LDS atomic per
// wavefront.  The workgroup then adds each touched cell to the table with one
// set of global atomics.  64-bit integer atomics keep the sums exact and
// independent of the order.
__device__ __forceinline__ void lds_incidence(unsigned long long* s_sum,
                                              unsigned long long* s_sq, unsigned int* s_cnt,
                                              int cell, long long fx, long long fsq)
{
    const int c0 = __shfl(cell, 0, 64);
    if (__ballot(cell != c0) == 0ull) {
        if (c0 >= 0) {
            const long long s1 = wave_sum_i64(fx), s2 = wave_sum_i64(fsq);
            if ((threadIdx.x & 63) == 0) {
                atomicAdd(&s_sum[c0], (unsigned long long)s1);
                atomicAdd(&s_sq[c0], (unsigned long long)s2);
                atomicAdd(&s_cnt[c0], 64u);
            }
        }
    } else if (cell >= 0) {
        atomicAdd(&s_sum[cell], (unsigned long long)fx);
        atomicAdd(&s_sq[cell], (unsigned long long)fsq);
        atomicAdd(&s_cnt[cell], 1u);
    }
}

constexpr int kPayoffStreamThreads = 512;
constexpr int kPayoffStreamBatch = 2;     // envs per thread per iteration (loads in flight)

// The incidences of one env whose seats' returns and ids are in registers.
template <int NA>
__device__ __forceinline__ void stream_env(unsigned long long* s_sum, unsigned long long* s_sq,
                                           unsigned int* s_cnt, const float (&g)[NA],
                                           const int (&pid)[NA], uint32_t team_row,
                                           uint32_t team_col, int P)
{
#pragma unroll
    for (int a = 0; a < NA; ++a) {
        if (!((team_row >> a) & 1u))
            continue;
        const double gd = (double)g[a];
        const long long fx = __double2ll_rn(gd * 4294967296.0);
        const long long fsq = __double2ll_rn(gd * gd * 1048576.0);
#pragma unroll
        for (int b = 0; b < NA; ++b) {
            if (!((team_col >> b) & 1u))
                continue;
            // lanes past the range carry id -1, hence cell -1: a partial
            // wavefront never takes the shuffle path with them
            const int cell = (pid[a] >= 0 && pid[a] < P && pid[b] >= 0 && pid[b] < P)
                                 ? pid[a] * P + pid[b]
                                 : -1;
            lds_incidence(s_sum, s_sq, s_cnt, cell, fx, fsq);
        }
    }
}

// NA: seats per env known at compile time (2), or 0 (any count, one env per
// thread per iteration)
template <int CELLS, int NA>
__global__ __launch_bounds__(kPayoffStreamThreads) void payoff_stream_kernel(
    const float* __restrict__ ret, const int32_t* __restrict__ pids, int64_t n, int n_agents,
    uint32_t team_row, uint32_t team_col, int P, unsigned long long* __restrict__ sum,
    unsigned long long* __restrict__ sumsq, unsigned long long* __restrict__ cnt)
{
    __shared__ unsigned long long s_sum[CELLS], s_sq[CELLS];
    __shared__ unsigned int s_cnt[CELLS];
    const int cells = P * P;
    for (int c = threadIdx.x; c < cells; c += kPayoffStreamThreads) {
        s_sum[c] = 0;
        s_sq[c] = 0;
        s_cnt[c] = 0;
    }
    __syncthreads();
    const int64_t e0 = n * blockIdx.x / gridDim.x, e1 = n * (blockIdx.x + 1) / gridDim.x;
    if constexpr (NA > 0) {
        constexpr int kStep = kPayoffStreamThreads * kPayoffStreamBatch;
        // the loop bound is uniform over the workgroup (shuffles inside)
        for (int64_t base = e0; base < e1; base += kStep) {
            // every seat's return and id of this thread's envs first (all
            // loads in flight together), then the incidences
            float g[kPayoffStreamBatch][NA];
            int pid[kPayoffStreamBatch][NA];
#pragma unroll
            for (int k = 0; k < kPayoffStreamBatch; ++k) {
                const int64_t e = base + k * kPayoffStreamThreads + threadIdx.x;
                const bool valid = e < e1;
#pragma unroll
                for (int a = 0; a < NA; ++a) {
                    pid[k][a] = valid ? pids[e * NA + a] : -1;
                    g[k][a] = valid && ((team_row >> a) & 1u) ? ret[(int64_t)a * n + e] : 0.f;
                }
            }
#pragma unroll
            for (int k = 0; k < kPayoffStreamBatch; ++k)
                stream_env<NA>(s_sum, s_sq, s_cnt, g[k], pid[k], team_row, team_col, P);
        }
    } else {
        for (int64_t base = e0; base < e1; base += kPayoffStreamThreads) {
            const int64_t e = base + threadIdx.x;
            const bool valid = e < e1;
            for (int a = 0; a < n_agents; ++a) {
                if (!((team_row >> a) & 1u))
                    continue;
                long long fx = 0, fsq = 0;
                int pa = -1;
                if (valid) {
                    const double gd = (double)ret[(int64_t)a * n + e];
                    fx = __double2ll_rn(gd * 4294967296.0);
                    fsq = __double2ll_rn(gd * gd * 1048576.0);
                    pa = pids[e * n_agents + a];
                }
                for (int b = 0; b < n_agents; ++b) {
                    if (!((team_col >> b) & 1u))
                        continue;
                    const int pb = valid ? pids[e * n_agents + b] : -1;
                    const int cell =
                        (pa >= 0 && pa < P && pb >= 0 && pb < P) ? pa * P + pb : -1;
                    lds_incidence(s_sum, s_sq, s_cnt, cell, fx, fsq);
                }
            }
        }
    }
    __syncthreads();
    for (int c = threadIdx.x; c < cells; c += kPayoffStreamThreads) {
        const unsigned int k = s_cnt[c];
        if (k) {
            atomicAdd(&sum[c], s_sum[c]);
            atomicAdd(&sumsq[c], s_sq[c]);
            atomicAdd(&cnt[c], (unsigned long long)k);
        }
    }
}

// Larger populations: from the slots sorted by policy id (the bucketing of
// the policy forward).  The sorted slot list is cut into equal ranges, one
// per workgroup, so that a heavily played policy spreads over many
// workgroups; a range holds one or a few policy segments.  For each segment
// (row policy p) the row-side slots add their env's incidences (p, id of each
// column-side seat) into one row of P cells in LDS, which is then added to the
// table with one set of global atomics per touched cell.  Each thread keeps
// kPayoffBatch slots' loads in flight.  Slots whose id is out of range (the
// bucketing files them under policy 0) are skipped.
constexpr int kPayoffThreads = 256;
constexpr int kPayoffBatch = 4;

__global__ __launch_bounds__(kPayoffThreads) void payoff_bucketed_kernel(
    const float* __restrict__ ret, const int32_t* __restrict__ pids,
    const int32_t* __restrict__ perm, const int32_t* __restrict__ offsets, int64_t n,
    int n_agents, uint32_t team_row, uint32_t team_col, int P, int64_t rows_per_wg,
    unsigned long long* __restrict__ sum, unsigned long long* __restrict__ sumsq,
    unsigned long long* __restrict__ cnt)
{
    __shared__ unsigned long long s_sum[kMaxP], s_sq[kMaxP];
    __shared__ unsigned int s_cnt[kMaxP];
    __shared__ int s_off[kMaxP + 1];
    const int64_t ns = n * n_agents;
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_wg;
    const int64_t r1 = r0 + rows_per_wg < ns ? r0 + rows_per_wg : ns;
    for (int c = threadIdx.x; c <= P; c += kPayoffThreads)
        s_off[c] = offsets[c];
    __syncthreads();
    // first policy whose segment reaches past r0 (offsets is non-decreasing,
    // offsets[0] = 0, offsets[P] = ns)
    int p = 0;
    {
        int lo = 0, hi = P - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_off[mid] <= r0)
                lo = mid;
            else
                hi = mid - 1;
        }
        p = lo;
    }
    for (; p < P && s_off[p] < r1; ++p) {
        const int64_t s0 = s_off[p] > r0 ? s_off[p] : r0;
        const int64_t s1 = s_off[p + 1] < r1 ? s_off[p + 1] : r1;
        if (s0 >= s1)
            continue;          // uniform over the workgroup
        for (int c = threadIdx.x; c < P; c += kPayoffThreads) {
            s_sum[c] = 0;
            s_sq[c] = 0;
            s_cnt[c] = 0;
        }
        __syncthreads();
        for (int64_t r = s0 + threadIdx.x; r < s1; r += (int64_t)kPayoffThreads * kPayoffBatch) {
            int slot[kPayoffBatch], pid[kPayoffBatch];
            float g[kPayoffBatch];
#pragma unroll
            for (int k = 0; k < kPayoffBatch; ++k) {
                const int64_t rk = r + (int64_t)k * kPayoffThreads;
                slot[k] = rk < s1 ? perm[rk] : -1;
            }
#pragma unroll
            for (int k = 0; k < kPayoffBatch; ++k) {
                pid[k] = -1;
                g[k] = 0.f;
                if (slot[k] >= 0) {
                    const int64_t e = slot[k] / n_agents, a = slot[k] - e * n_agents;
                    if ((team_row >> a) & 1u) {
                        pid[k] = pids[slot[k]];
                        g[k] = ret[a * n + e];
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < kPayoffBatch; ++k) {
                if (pid[k] != p)
                    continue;
                const int64_t e = slot[k] / n_agents;
                const double gd = (double)g[k];
                const long long fx = __double2ll_rn(gd * 4294967296.0);
                const long long fsq = __double2ll_rn(gd * gd * 1048576.0);
                for (int b = 0; b < n_agents; ++b) {
                    if (!((team_col >> b) & 1u))
                        continue;
                    const int pb = pids[e * n_agents + b];
                    if (pb < 0 || pb >= P)
                        continue;
                    atomicAdd(&s_sum[pb], (unsigned long long)fx);
                    atomicAdd(&s_sq[pb], (unsigned long long)fsq);
                    atomicAdd(&s_cnt[pb], 1u);
                }
            }
        }
        __syncthreads();
        for (int c = threadIdx.x; c < P; c += kPayoffThreads) {
            const unsigned int k = s_cnt[c];
            if (k) {
                const int64_t cell = (int64_t)p * P + c;
                atomicAdd(&sum[cell], s_sum[c]);
                atomicAdd(&sumsq[cell], s_sq[c]);
                atomicAdd(&cnt[cell], (unsigned long long)k);
            }
        }
        __syncthreads();       // the row is cleared for the next segment
    }
}

hipError_t launch_payoff_bucketed(const float* ret, const int32_t* pids, const int32_t* perm,
                                  const int32_t* offsets, int64_t n_envs, int n_agents,
                                  uint32_t team_row, uint32_t team_col, int P, int n_cus,
                                  unsigned long long* sum, unsigned long long* sumsq,
                                  unsigned long long* cnt, hipStream_t s)
{
    const int64_t ns = n_envs * n_agents;
    // about four workgroups per CU, at least 256 slots each
    const int64_t want = std::max<int64_t>(1, std::min<int64_t>(4 * (int64_t)n_cus,
                                                                (ns + 255) / 256));
    const int64_t rows = (ns + want - 1) / want;
    const int grid = (int)((ns + rows - 1) / rows);
    payoff_bucketed_kernel<<<grid, kPayoffThreads, 0, s>>>(ret, pids, perm, offsets, n_envs,
                                                           n_agents, team_row, team_col, P,
                                                           rows, sum, sumsq, cnt);
    return hipGetLastError();
}

bool payoff_stream_fits(int P)
{
    return P * P <= kPayoffStreamMaxCells;
}

hipError_t launch_payoff_stream(const float* ret, const int32_t* pids, int64_t n_envs,
                                int n_agents, uint32_t team_row, uint32_t team_col, int P,
                                int n_cus, unsigned long long* sum, unsigned long long* sumsq,
                                unsigned long long* cnt, hipStream_t s)
{
    const int cells = P * P;
    // up to four workgroups per CU (two for the 80 KB table), at least 1024
    // envs each
    const int per_cu = cells <= 1024 ? 4 : 2;
    const int grid = (int)std::max<int64_t>(
        1, std::min<int64_t>((int64_t)per_cu * n_cus, (n_envs + 1023) / 1024));
    auto go = [&](auto cells_c) {
        constexpr int C = decltype(cells_c)::value;
        if (n_agents == 2)
            payoff_stream_kernel<C, 2><<<grid, kPayoffStreamThreads, 0, s>>>(
                ret, pids, n_envs, n_agents, team_row, team_col, P, sum, sumsq, cnt);
        else
            payoff_stream_kernel<C, 0><<<grid, kPayoffStreamThreads, 0, s>>>(
                ret, pids, n_envs, n_agents, team_row, team_col, P, sum, sumsq, cnt);
    };
    if (cells <= 256)
        go(std::integral_constant<int, 256>{});
    else if (cells <= 1024)
        go(std::integral_constant<int, 1024>{});
    else if (cells <= kPayoffStreamMaxCells)
        go(std::integral_constant<int, kPayoffStreamMaxCells>{});
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_payoff(const float* ret, const int32_t* pids, int64_t n_envs, int n_agents,
                         const int8_t* team, int P, unsigned long long* sum,
                         unsigned long long* sumsq, unsigned long long* cnt, hipStream_t s)
{
    EnvArgs ea{};
    for (int k = 0; k < n_agents; ++k) {
        if (team[k] > 0)
            ea.team_row |= 1u << k;
        else if (team[k] < 0)
            ea.team_col |= 1u << k;
    }
    payoff_kernel<<<(int)((n_envs + 255) / 256), 256, 0, s>>>(ret, pids, n_envs, n_agents, ea,
                                                              P, sum, sumsq, cnt);
    return hipGetLastError();
}

// ------------------------------------------------------------ table read-back

// One thread per cell: mean = sum 2^-32 / n (NaN for an empty cell), standard
// error sqrt(variance / n) with the variance from the sums (NaN below two
// simulations).  Writes the finalized table to host memory and clears what the
// caller asked for in the same launch, so a read-back is one launch and one
// synchronization.
__global__ void read_table_kernel(unsigned long long* __restrict__ acc, int64_t PP, int reset,
                                  unsigned long long* __restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < PP) {
        const long long cnt = (long long)acc[2 * PP + i];
        double mean = (double)NAN, err = (double)NAN;
        if (cnt > 0) {
            const double n = (double)cnt;
            mean = (double)(long long)acc[i] * 0x1p-32 / n;
            if (cnt >= 2) {
                const double s2 = (double)(long long)acc[PP + i] * 0x1p-20;
                const double var = (s2 - n * mean * mean) / (n - 1.0);
                err = sqrt(var > 0.0 ? var / n : 0.0);
            }
        }
        out[i] = (unsigned long long)__double_as_longlong(mean);
        out[PP + i] = (unsigned long long)cnt;
        out[2 * PP + i] = (unsigned long long)__double_as_longlong(err);
        if (reset) {
            acc[i] = 0;
            acc[PP + i] = 0;
            acc[2 * PP + i] = 0;
        }
    } else if (i == PP) {
        out[3 * PP] = acc[3 * PP];
        if (reset)
            acc[3 * PP] = 0;
    } else if (i == PP + 1) {
        out[3 * PP + 1] = acc[3 * PP + 1];
        acc[3 * PP + 1] = 0;
    }
}

hipError_t launch_read_table(unsigned long long* acc, int64_t PP, int reset,
                             unsigned long long* out, hipStream_t s)
{
    read_table_kernel<<<(int)((PP + 2 + 255) / 256), 256, 0, s>>>(acc, PP, reset, out);
    return hipGetLastError();
}

}  // namespace malib
