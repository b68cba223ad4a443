// Games with few distinct observations: the matrix games (tabular policies see
// nothing, the iterated game's observation is the last four joint actions) and
// pursuit (the opponent's place in a 5x5 window, or out of sight).
//
// A policy's logits depend on the observation alone, so a batch evaluates every
// policy once on every observation that can occur (a table of logits, by the
// same forward kernels, hence the same bits) and then plays the whole horizon in
// one kernel: a step is one look-up, the Gumbel noise and the game's rule, with
// the state in registers.  Per step and slot this replaces a policy evaluation
// and the state's, the logits' and two launches' round trips.
//
// Bound: large batches by the random stream (56 64-bit multiply-adds, at 16
// cycles, per slot and step), small ones by the steps' latency.  2^20 envs of the
// iterated game, 32 steps: 32 x (265 + 17) us before, now 25 us for the table's
// 118096 rows and 400 us; pursuit, 16384 envs, 100 steps: 100 x (12 + 5) us
// before, now 8 + 68 us.
#include "device.hpp"
#include "internal.hpp"

namespace malib {

// ------------------------------------------------------------------ the table

// Observations of the table.  Iterated game, one seat (the other's view is the
// history with each joint action's two digits exchanged): histories of k < 5
// joint actions d = a_own * A + a_other, entry off_k + sum_i d_i q^i with d_0 the
// most recent, q = A^2 and off_k = 1 + q + .. + q^(k-1).  Pursuit, both seats:
// 26 states, the evader 5 (dy + 2) + (dx + 2) from the pursuer inside the window,
// or 25 where they do not see each other.
int finite_rows(int env_kind, int A, int horizon)
{
    if (env_kind == MALIB_ENV_PURSUIT)
        return 26;
    int rows = 0, pw = 1;
    for (int k = 0; k < 5 && k < horizon; ++k, pw *= A * A)
        rows += pw;
    return rows;
}

// One thread per (policy, entry): the state of the entry's virtual env, the rows
// (sorted by policy as they are) and the tile table of the forward.
__global__ void finite_table_kernel(int env_kind, int A, int grid, int P, int rows, int seats,
                                    int tile_rows, int n_entries, int striped,
                                    void* __restrict__ state, int32_t* __restrict__ perm,
                                    int32_t* __restrict__ perm_env, int4* __restrict__ info)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t envs = (int64_t)P * rows;
    if (i < envs) {
        const int row = (int)(i % rows);
        if (env_kind == MALIB_ENV_PURSUIT) {
            // pursuer at (2, 2); out of sight: evader at (5, 2) (on a 5x5 torus,
            // where everything is in sight, the entry is not used)
            const int x = row < 25 ? row % 5 : (grid > 5 ? 5 : 0), y = row < 25 ? row / 5 : 2;
            ((uint8_t*)state)[i] = (uint8_t)(2 * grid + 2);
            ((uint8_t*)state)[envs + i] = (uint8_t)(y * grid + x);
        } else {
            const int q = A * A;
            int k = 0, e = row, pw = 1;
            while (e >= pw) {
                e -= pw;
                pw *= q;
                ++k;
            }
            uint32_t h = 0xFFFFu;
            for (int l = 0; l < k; ++l, e /= q) {
                const int d = e % q;
                h = (h & ~(15u << (4 * l))) | (uint32_t)((d / A) * 3 + d % A) << (4 * l);
            }
            ((uint16_t*)state)[i] = (uint16_t)h;
        }
        for (int s = 0; s < seats; ++s) {
            perm[i * seats + s] = (int32_t)(i * seats + s);
            perm_env[i * seats + s] = (int32_t)i;
        }
    }
    if (i < n_entries) {
        const int per_p = rows * seats, tiles_p = (per_p + tile_rows - 1) / tile_rows;
        const int T = P * tiles_p;
        int t = (int)i;
        if (striped) {   // the layout of tile_table_kernel
            const int per = n_entries / 8, x = t / per, j = t - x * per;
            const int lo = (int)((int64_t)x * T / 8), hi = (int)((int64_t)(x + 1) * T / 8);
            t = j < hi - lo ? lo + j : T;
        }
        int4 v = make_int4(-1, 0, 0, 0);
        if (t < T) {
            const int p = t / tiles_p, r = (t - p * tiles_p) * tile_rows;
            v = make_int4(p, p * per_p + r, min(tile_rows, per_p - r), 0);
        }
        info[i] = v;
    }
}

hipError_t launch_finite_table(int env_kind, int A, int grid, int P, int rows, int seats,
                               int tile_rows, int n_entries, bool striped, void* state,
                               int32_t* perm, int32_t* perm_env, int4* info, hipStream_t s)
{
    const int64_t n = std::max<int64_t>((int64_t)P * rows, n_entries);
    finite_table_kernel<<<(int)((n + 255) / 256), 256, 0, s>>>(
        env_kind, A, grid, P, rows, seats, tile_rows, n_entries, striped ? 1 : 0, state, perm,
        perm_env, info);
    return hipGetLastError();
}

// ------------------------------------------------------------------ the horizon

// Block 0 of the action stream of one (env, seat < 2) at successive steps: the
// counter words (g, t, seat, 0) enter rounds 1 to 3 so that six of the twenty
// 64-bit products do not depend on t, or only on t (a scalar).
struct ActionStream {
    uint64_t seed, w1, y2, lo3, hi3;

    __device__ __forceinline__ void init(uint64_t key, uint64_t g, uint32_t seat)
    {
        seed = key;
        uint64_t lo, hi;
        mul_hilo64(kPhiloxM0, g, w1, hi);                  // round 1: z1 = hi, w1
        const uint64_t y1 = seat ? kPhiloxM1 : 0ull;       // lo(m1 seat), its hi is 0
        mul_hilo64(kPhiloxM1, hi, y2, lo);                 // round 2: hi half in lo
        const uint64_t x2 = lo ^ y1 ^ (seed + kPhiloxW0);
        mul_hilo64(kPhiloxM0, x2, lo3, hi3);               // round 3's first product
    }

    __device__ __forceinline__ u64x4 block(uint64_t t) const
    {
        uint64_t lo, hi, l1, h1;
        mul_hilo64(kPhiloxM0, t ^ seed, lo, hi);           // round 2, t alone
        const uint64_t z2 = hi ^ w1 ^ kPhiloxW1, w2 = lo;
        mul_hilo64(kPhiloxM1, z2, l1, h1);                 // round 3
        u64x4 c;
        c.x = h1 ^ y2 ^ (seed + 2 * kPhiloxW0);
        c.y = l1;
        c.z = hi3 ^ w2 ^ (2 * kPhiloxW1);
        c.w = lo3;
        return philox_rounds<7>(c, seed + 3 * kPhiloxW0, 3 * kPhiloxW1);
    }
};

struct FiniteArgs {
    const float* table;      // logits [policy][row][seat][A] (see launch_finite)
    const int32_t* pids;     // [n][2]
    const float* Amat;
    int P, A, grid, rows, shared, iter, per_seat;
    int64_t n, env_offset;
    uint64_t seed;
    int t0, t1;              // steps played by this launch
    int resume, keep;        // state and returns read at t0 (else reset) / written back after t1
    uint8_t* log;            // action log of step 0, or null
    TrajArgs tr;
    void* state;             // iterated game: uint16 [n]; pursuit: uint8 [2][n]
    uint8_t* done;
    float* ret;              // [2][n]
    unsigned long long* frames;
    int* flags;
    // payoff table accumulators [P][P] (null: reduced by another kernel): the
    // row side is seat row_seat
    unsigned long long* sum;
    unsigned long long* sumsq;
    unsigned long long* cnt;
    int row_seat;
};

// The two seats' actions exchanged between neighbouring lanes.
__device__ __forceinline__ int swap_pair(int x)
{
    return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, false);   // quad_perm [1, 0, 3, 2]
}

// x + d on a ring of G cells, x in [0, G), |d| < G (a negative value is a large
// unsigned one, so each wrap is one minimum).
__device__ __forceinline__ int ring_add(int x, int d, int G)
{
    const uint32_t v = (uint32_t)(x + d), w = min(v, v + (uint32_t)G);
    return (int)min(w, w - (uint32_t)G);
}

// Moves: 0 stay, 1 up, 2 down, 3 left, 4 right (two bits per action, plus one).
__device__ __forceinline__ int move_x(int a) { return ((0x215 >> (2 * a)) & 3) - 1; }
__device__ __forceinline__ int move_y(int a) { return ((0x161 >> (2 * a)) & 3) - 1; }

// First index of the largest z (the lower index on equal values): the maximum,
// then the first element equal to it.
template <int N>
__device__ __forceinline__ int first_max(const float (&z)[N])
{
    float m = z[0];
#pragma unroll
    for (int a = 1; a < N; ++a)
        m = __builtin_fmaxf(m, z[a]);
    int ix = N - 1;
#pragma unroll
    for (int a = N - 2; a >= 0; --a)
        ix = z[a] == m ? a : ix;
    return ix;
}

// NL lanes per env (2, 8 or 32), lane parity = seat.  With NL = 2 a lane draws
// its own noise at each step.  With more, a small batch's latency is cut: lane i
// of an env draws the noise of step t + i / 2 for its seat, NL / 2 steps at once,
// into LDS (one wavefront's own part), and all lanes then play those steps alike,
// lanes 0 and 1 writing; pursuit's rows of the two policies are copied to LDS.
// A step is then a chain of about 50 dependent instructions and one LDS read.
// CA: the number of actions where it is known (pursuit's 5, the 3x3 games), else
// 0 (AMAX >= A; 8 unless NL = 2).  REC: something besides the returns is kept (an
// action log, records, the state).
template <bool PURSUIT, int AMAX, int NL, int CA, bool REC>
__global__ __launch_bounds__(256) void finite_kernel(FiniteArgs f)
{
    static_assert(NL == 2 || AMAX == 8, "one block of noise per lane");
    constexpr int AZ = CA ? CA : AMAX;                 // logits held per slot
    constexpr int SN = NL / 2;                         // steps per round of noise
    constexpr int NZ = 12;                             // noise of a (step, seat), 16-byte rows
    constexpr bool kLdsTab = PURSUIT && NL > 2;
    constexpr int TS = 26 * 5 + 1;                     // odd: the slots' rows spread over banks
    // the noise, after the last step the workgroup's entries of the payoff table
    constexpr int NOISE = NL > 2 ? (256 + 2) * NZ * 4 : 0, SLOT = 2 * 8 + 2 * 4;
    constexpr int LDS = NOISE > 512 / NL * SLOT ? NOISE : 512 / NL * SLOT;
    __shared__ __attribute__((aligned(16))) char lds[LDS];
    float* noise = (float*)lds;
    __shared__ float tab_s[kLdsTab ? 256 / NL * 2 * TS : 1];
    __shared__ int live_s;
    if (PURSUIT && threadIdx.x == 0)
        live_s = 0;
    __syncthreads();
    const int A = CA ? CA : f.A;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t e = i / NL;
    const int li = (int)(i % NL), seat = li & 1;
    const bool valid = e < f.n, writer = valid && li < 2;
    const int64_t ec = valid ? e : 0;
    const uint64_t g = (uint64_t)(f.env_offset + ec);
    const int pid = f.pids[2 * ec + seat];
    const bool known = pid >= 0 && pid < f.P;
    if (!known && writer)
        atomicOr(f.flags, kErrPid);
    const int p = known ? pid : 0;
    // this lane's rows of the table
    int stride = f.per_seat ? 2 * A : A;
    const float* tab = f.table + (int64_t)p * f.rows * stride + (f.per_seat ? seat * A : 0);
    if constexpr (kLdsTab) {
        float* dst = tab_s + ((int)(threadIdx.x / NL) * 2 + seat) * TS;
        for (int j = li >> 1; j < f.rows * 5; j += SN)
            dst[j] = tab[j / 5 * stride + j % 5];
        wave_lds_sync();
        tab = dst;
        stride = 5;
    }
    ActionStream rs;
    rs.init(f.seed, g, (uint32_t)seat);

    // ---- state
    const int G = f.grid;
    int px = 0, py = 0, ex = 0, ey = 0;                // pursuit: cells
    int ux = 0, uy = 0;                                // evader - pursuer + 2 on the torus
    bool dn = !valid;
    uint32_t hist = 0xFFFFu;                           // iterated game
    const int q = A * A;
    int lags = 0, row = 0, off = 0, pw = 1;            // k, table entry - off_k, off_k, q^k
    float ret = 0.0f;
    const bool resume = REC && f.resume;
    if (resume)
        ret = f.ret[seat * f.n + ec];
    if constexpr (PURSUIT) {
        uint32_t pc, qc;
        if (resume) {
            pc = ((const uint8_t*)f.state)[ec];
            qc = ((const uint8_t*)f.state)[f.n + ec];
            dn = dn || f.done[ec] != 0;
        } else {
            const u64x4 b = stream_block(f.seed, f.shared ? 0 : g, 0, kPurposeReset, 0, 0);
            const uint32_t cells = (uint32_t)(G * G);
            pc = (uint32_t)(((b.x & 0xFFFFFFFFull) * cells) >> 32);
            qc = (pc + 1 + (uint32_t)(((b.x >> 32) * (uint64_t)(cells - 1)) >> 32)) % cells;
        }
        px = (int)pc % G;
        py = (int)pc / G;
        ex = (int)qc % G;
        ey = (int)qc / G;
        ux = ring_add(ring_add(ex, -px, G), 2, G);
        uy = ring_add(ring_add(ey, -py, G), 2, G);
    } else if (f.iter && resume) {
        hist = ((const uint16_t*)f.state)[ec];
        for (int l = 3; l >= 0; --l) {
            const uint32_t j = (hist >> (4 * l)) & 15u;
            if (j == 15u)
                continue;
            const int a0 = (int)j / 3, a1 = (int)j % 3;
            row = row * q + (seat == 0 ? a0 * A + a1 : a1 * A + a0);
            off += pw;
            pw *= q;
            ++lags;
        }
    }
    int lives = 0;
    bool got = false;                                  // captured in this launch

    for (int tb = f.t0; tb < f.t1; tb += SN) {
        // ---- noise of the next SN steps
        float nz[AZ];
        const float* nrow = noise + ((int)threadIdx.x - li + seat) * NZ;
        auto read_noise = [&]() {
#pragma unroll
            for (int a = 0; a < AZ; ++a)
                nz[a] = nrow[a];
            nrow += 2 * NZ;
        };
        if constexpr (NL > 2) {
            const u64x4 b = rs.block((uint64_t)(tb + (li >> 1)));
#pragma unroll
            for (int j = 0; j < AZ; ++j)
                noise[threadIdx.x * NZ + j] = gumbel01(uniform01(block_lane(b, j)));
            wave_lds_sync();
            read_noise();
        } else {
            u64x4 blk[AMAX / 8];
            blk[0] = rs.block((uint64_t)tb);
#pragma unroll
            for (int b = 1; b < AMAX / 8; ++b)
                if (8 * b < A)
                    blk[b] = stream_block(f.seed, g, (uint64_t)tb, kPurposeAction,
                                          (uint32_t)seat, (uint64_t)b);
#pragma unroll
            for (int a = 0; a < AZ; ++a)
                if (a < A)
                    nz[a] = gumbel01(uniform01(block_lane(blk[a >> 3], a & 7)));
        }
        const int te = min(tb + SN, f.t1);
        for (int t = tb; t < te; ++t) {
            // ---- the logits of this seat's observation, the action
            int entry = 0;
            if (f.rows > 1) {
                if constexpr (PURSUIT)
                    entry = max(ux, uy) < 5 ? 5 * uy + ux : 25;
                else
                    entry = off + row;
            }
            const float* l = tab + entry * stride;
            float z[AZ];
#pragma unroll
            for (int a = 0; a < AZ; ++a)
                z[a] = a < A ? l[a] + nz[a] : -__builtin_inff();
            if constexpr (NL > 2)   // the next step's noise, ahead of its use (past
                read_noise();       // the round's last step: the next row, unused)
            // (the noise is finite: a NaN here is a NaN logit)
            bool bad = false;
#pragma unroll
            for (int a = 0; a < AZ; a += 2)
                bad |= __builtin_isunordered(z[a], z[a + 1 < AZ ? a + 1 : a]);
            int act = first_max<AZ>(z);
            const bool live = !dn;
            if (__ballot(bad) != 0ull) {
                act = bad ? 0 : act;
                if (bad && live && writer)
                    atomicOr(f.flags, kErrNaN);
            }
            const int other = swap_pair(act);
            const int a0 = seat == 0 ? act : other, a1 = seat == 0 ? other : act;
            // ---- the step
            float rew = 0.0f;
            bool caught = false;
            const uint32_t h0 = hist, p0 = (uint32_t)(py * G + px), q0 = (uint32_t)(ey * G + ex);
            if constexpr (PURSUIT) {
                const int wx = move_x(a1) - move_x(a0), wy = move_y(a1) - move_y(a0);
                const int vx = ring_add(ux, wx, G), vy = ring_add(uy, wy, G);
                // the same cell afterwards, or the two swap neighbouring cells (the
                // evader, at r = u - 2 from the pursuer, then moves by -2 r against it)
                caught = ((vx == 2) & (vy == 2)) | ((wx == 4 - 2 * ux) & (wy == 4 - 2 * uy));
                caught = caught & live;
                lives += live;
                if constexpr (REC) {
                    if (live) {
                        ux = vx;
                        uy = vy;
                        px = ring_add(px, move_x(a0), G);
                        py = ring_add(py, move_y(a0), G);
                        ex = ring_add(ex, move_x(a1), G);
                        ey = ring_add(ey, move_y(a1), G);
                    }
                    rew = caught ? 1.0f : 0.0f;
                } else {   // a finished env's place is not looked at
                    ux = vx;
                    uy = vy;
                }
                dn = dn | caught;
                got = got | caught;
            } else {
                rew = f.Amat[a0 * A + a1];
                ret = ret + (seat == 0 ? rew : -rew);
                if (REC && f.iter)
                    hist = ((hist << 4) | (uint32_t)(a0 * 3 + a1)) & 0xFFFFu;
                if (f.rows > 1) {
                    const int d = act * A + other;
                    if (lags == 4) {               // the oldest drops out
                        row = row % (q * q * q) * q + d;
                    } else {
                        row = row * q + d;
                        off += pw;
                        pw *= q;
                        ++lags;
                    }
                }
            }
            if constexpr (REC) {
                if (f.log && writer)
                    f.log[(int64_t)t * 2 * f.n + 2 * e + seat] =
                        live ? (uint8_t)act : (uint8_t)255;
                // record t n + e of the batch; of those that share a place in the
                // ring only the newest is written: the envs are not in step here
                if (f.tr.act && writer && (f.tr.horizon - t) * f.n - e <= f.tr.cap) {
                    const int64_t rec = (f.tr.base + (int64_t)t * f.n + e) % f.tr.cap;
                    f.tr.act[2 * rec + seat] = live ? (uint8_t)act : (uint8_t)255;
                    if (seat == 0) {
                        f.tr.rew[rec] = rew;
                        const int last = t == f.tr.horizon - 1 ? 2 : 0;
                        f.tr.flags[rec] =
                            (uint8_t)(PURSUIT ? (caught ? 1 : 0) | last | (live ? 0 : 4) : last);
                        if (f.tr.obs) {
                            if constexpr (PURSUIT) {
                                ((uint8_t*)f.tr.obs)[2 * rec] = (uint8_t)p0;
                                ((uint8_t*)f.tr.obs)[2 * rec + 1] = (uint8_t)q0;
                            } else if (f.iter) {
                                ((uint16_t*)f.tr.obs)[rec] = (uint16_t)h0;
                            }
                        }
                    }
                }
            }
        }
        if constexpr (NL > 2)
            wave_lds_sync();   // the noise was read: the next round may replace it
        // nothing is left to play or to write down
        if (PURSUIT && !(REC && (f.log || f.tr.act)) && __all(dn))
            break;
    }

    if (PURSUIT && got)
        ret += seat == 0 ? 1.0f : -1.0f;
    if (writer) {
        f.ret[seat * f.n + e] = ret;
        if (REC && f.keep && seat == 0) {
            if constexpr (PURSUIT) {
                ((uint8_t*)f.state)[e] = (uint8_t)(py * G + px);
                ((uint8_t*)f.state)[f.n + e] = (uint8_t)(ey * G + ex);
                f.done[e] = dn ? 1 : 0;
            } else if (f.iter) {
                ((uint16_t*)f.state)[e] = (uint16_t)hist;
            }
        }
    }
    if (f.sum) {
        // the envs' entries of the table, by their row seats' lanes (neither seat's
        // id out of range): those of one cell are combined in the workgroup first,
        // in an LDS hash table of twice as many slots as it has envs.  An atomic on
        // one line of the table takes 12 ns, whoever sends it, so envs that share
        // few cells (a meta-strategy on few policies) must not each send theirs:
        // ids of two policies only, one-step games of P = 64, 16384 envs 72 -> 12 us
        // a fill, iterated games of P = 100, 2^20 envs 3236 -> 166 us (ids of all
        // policies: 12 -> 13 and 228 -> 227 us).
        constexpr int SLOTS = 2 * (256 / NL);
        unsigned long long* h_sum = (unsigned long long*)lds;
        unsigned long long* h_sq = h_sum + SLOTS;
        int* h_cell = (int*)(h_sq + SLOTS);
        unsigned int* h_cnt = (unsigned int*)(h_cell + SLOTS);
        __syncthreads();   // the noise has been read
        if (threadIdx.x < SLOTS) {
            h_sum[threadIdx.x] = 0;
            h_sq[threadIdx.x] = 0;
            h_cell[threadIdx.x] = -1;
            h_cnt[threadIdx.x] = 0;
        }
        __syncthreads();
        const int other = swap_pair(known ? pid : -1);
        if (writer && seat == f.row_seat && known && other >= 0) {
            const int cell = pid * f.P + other;
            const double gd = (double)ret;
            // (at most half of the slots are ever taken: the search ends)
            uint32_t k = ((uint32_t)cell * 0x9E3779B1u) >> 16 & (SLOTS - 1);
            for (;; k = (k + 1) & (SLOTS - 1)) {
                const int had = atomicCAS(&h_cell[k], -1, cell);
                if (had == -1 || had == cell)
                    break;
            }
            atomicAdd(&h_sum[k], (unsigned long long)__double2ll_rn(gd * 4294967296.0));
            atomicAdd(&h_sq[k], (unsigned long long)__double2ll_rn(gd * gd * 1048576.0));
            atomicAdd(&h_cnt[k], 1u);
        }
        __syncthreads();
        if (threadIdx.x < SLOTS && h_cell[threadIdx.x] >= 0) {
            const int cell = h_cell[threadIdx.x];
            atomicAdd(&f.sum[cell], h_sum[threadIdx.x]);
            atomicAdd(&f.sumsq[cell], h_sq[threadIdx.x]);
            atomicAdd(&f.cnt[cell], (unsigned long long)h_cnt[threadIdx.x]);
        }
    }
    if constexpr (PURSUIT) {
        // live agent-frames, two per env and step
        int mine = writer ? lives : 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
            mine += __shfl_xor(mine, o, 64);
        if ((threadIdx.x & 63) == 0 && mine)
            atomicAdd(&live_s, mine);
        __syncthreads();
        if (threadIdx.x == 0 && live_s)
            atomicAdd(f.frames, (unsigned long long)live_s);
    }
}

hipError_t launch_finite(const FiniteLaunch& L, hipStream_t s)
{
    const EnvArgs& e = L.env;
    FiniteArgs f = {};
    f.table = L.table;
    f.pids = L.pids;
    f.Amat = e.Amat;
    f.P = L.P;
    f.A = e.A;
    f.grid = e.grid;
    f.rows = L.rows;
    f.per_seat = L.per_seat;
    f.shared = e.init_mode == MALIB_INIT_SHARED;
    f.iter = e.kind == MALIB_ENV_ITER_MATRIX;
    f.n = L.n_envs;
    f.env_offset = L.env_offset;
    f.seed = L.seed;
    f.t0 = L.t0;
    f.t1 = L.t1;
    f.resume = L.t0 > 0;
    f.keep = L.keep;
    f.log = L.log;
    f.tr = e.tr;
    f.state = L.state;
    f.done = L.done;
    f.ret = L.ret;
    f.frames = L.frames;
    f.flags = L.flags;
    f.sum = L.sum;
    f.sumsq = L.sumsq;
    f.cnt = L.cnt;
    f.row_seat = (e.team_row & 1u) ? 0 : 1;
    const int64_t n = L.n_envs;
    const int H = L.t1 - L.t0;
    // lanes per env: the noise of more steps at once where the batch leaves the
    // chip idle, by envs per CU (256 CUs, pursuit, 100 steps: 1040 envs 37 / 51 / 82
    // us with 32 / 8 / 2, 16384 envs 109 / 68 / 83 us, 32768 envs 194 / 114 / 88 us)
    const int64_t cus = e.n_cus > 0 ? e.n_cus : 256;
    int nl = n <= 16 * cus ? 32 : n <= 96 * cus ? 8 : 2;
    if (e.A > 8)
        nl = 2;
    while (nl > 2 && nl / 2 > H)
        nl /= 4;
    const int blocks = (int)((n * nl + 255) / 256);
    const bool rec = L.log || e.tr.act || f.keep || f.resume;
    auto go = [&](auto pursuit, auto amax, auto lanes, auto ca) {
        constexpr bool PU = decltype(pursuit)::value;
        constexpr int AM = decltype(amax)::value, NL = decltype(lanes)::value;
        constexpr int CA = decltype(ca)::value;
        if (rec)
            finite_kernel<PU, AM, NL, CA, true><<<blocks, 256, 0, s>>>(f);
        else
            finite_kernel<PU, AM, NL, CA, false><<<blocks, 256, 0, s>>>(f);
    };
    std::integral_constant<int, 0> any;
    std::integral_constant<int, 2> two;
    std::integral_constant<int, 8> eight;
    auto by_lanes = [&](auto pursuit, auto ca) {
        if (nl == 32)
            go(pursuit, eight, std::integral_constant<int, 32>{}, ca);
        else if (nl == 8)
            go(pursuit, eight, eight, ca);
        else
            go(pursuit, eight, two, ca);
    };
    if (e.kind == MALIB_ENV_PURSUIT) {
        if (e.A != 5)
            return hipErrorInvalidValue;
        by_lanes(std::true_type{}, std::integral_constant<int, 5>{});
    } else if (e.A == 3) {
        by_lanes(std::false_type{}, std::integral_constant<int, 3>{});
    } else if (e.A <= 8) {
        by_lanes(std::false_type{}, any);
    } else if (e.A <= 16) {
        go(std::false_type{}, std::integral_constant<int, 16>{}, two, any);
    } else if (e.A <= 24) {
        go(std::false_type{}, std::integral_constant<int, 24>{}, two, any);
    } else if (e.A <= 32) {
        go(std::false_type{}, std::integral_constant<int, 32>{}, two, any);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Trace snapshot: the step's logits of every slot [n][2][A], from the table.
__global__ void finite_logits_kernel(const float* __restrict__ table,
                                     const int32_t* __restrict__ pids, int64_t n_slots, int kind,
                                     int A, int grid, int P, int rows, int per_seat,
                                     const void* __restrict__ state, float* __restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_slots)
        return;
    const int64_t e = i >> 1, n = n_slots / 2;
    const int seat = (int)(i & 1);
    int p = pids[i];
    p = p < 0 || p >= P ? 0 : p;
    int entry = 0;
    if (rows > 1 && kind == MALIB_ENV_PURSUIT) {
        const uint8_t* pos = (const uint8_t*)state;
        const int pc = pos[e], qc = pos[n + e];
        int dx = qc % grid - pc % grid, dy = qc / grid - pc / grid;
        dx += dx < 0 ? grid : 0;
        dy += dy < 0 ? grid : 0;
        dx -= 2 * dx > grid ? grid : 0;
        dy -= 2 * dy > grid ? grid : 0;
        entry = dx >= -2 && dx <= 2 && dy >= -2 && dy <= 2 ? 5 * (dy + 2) + dx + 2 : 25;
    } else if (rows > 1) {
        const uint32_t hist = ((const uint16_t*)state)[e];
        int row = 0, off = 0, pw = 1;
        for (int l = 3; l >= 0; --l) {
            const uint32_t j = (hist >> (4 * l)) & 15u;
            if (j == 15u)
                continue;
            const int a0 = (int)j / 3, a1 = (int)j % 3;
            row = row * A * A + (seat == 0 ? a0 * A + a1 : a1 * A + a0);
            off += pw;
            pw *= A * A;
        }
        entry = off + row;
    }
    const int stride = per_seat ? 2 * A : A;
    const float* l = table + ((int64_t)p * rows + entry) * stride + (per_seat ? seat * A : 0);
    for (int a = 0; a < A; ++a)
        out[i * A + a] = l[a];
}

hipError_t launch_finite_logits(const FiniteLaunch& L, float* out, hipStream_t s)
{
    const int64_t ns = 2 * L.n_envs;
    finite_logits_kernel<<<(int)((ns + 255) / 256), 256, 0, s>>>(
        L.table, L.pids, ns, L.env.kind, L.env.A, L.env.grid, L.P, L.rows, L.per_seat, L.state,
        out);
    return hipGetLastError();
}

}  // namespace malib
