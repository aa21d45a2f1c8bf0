// Two LSTM layers in one launch, or three (at the end of this file).  gfx950 only.
//
// Paper: the policy is a multi-layer LSTM (section 4 "Architecture") evaluated over packed minibatches
// (section 2.2).  The time loop of a layer is a chain of hundreds of dependent steps that leaves most of the
// chip idle, and the second layer's step t only needs the first layer's output of step t: so the two time
// loops run side by side, a few timesteps apart, instead of one after the other.
//
//   XCD 0..2   time loop of the producer layer (forward: layer 0; backward: layer 1), one group per XCD
//   XCD 3..5   time loop of the consumer layer, group g on XCD 3 + g
//   XCD 6..7   workers: for every finished chunk of a group's timesteps, the product that turns the producer's rows
//              into the consumer's input (forward: gates_1 = h_0 W_ih1^T + b; backward: dh_0 = dz_1 W_ih1)
//
// Which pieces a group runs.  A timestep of a time loop costs a fixed latency (one exchange between the group's
// workgroups, 1.1 to 1.7 us) plus a little per alive piece, and the launch lasts as long as its slowest group.  The
// pieces are sorted longest first, so they are cut into three blocks of consecutive pieces: group 0 gets the few
// longest ones (its chain of T_max dependent steps is what bounds the launch, so its steps should be the
// cheapest), the last group the many short ones (few steps, each with many pieces).  The plan
// picks the two cuts that minimise the largest predicted group time
//     sum over the group's timesteps of (step + low * min(b_t, 4) + over (b_t > 4) + piece * b_t + tile * (ceil(b_t / 16) - 1)),   b_t = alive pieces
// (a time loop works through the alive pieces 16 at a time: the MFMA's columns; up to four have a form of their own), which it
// evaluates per candidate from the pieces' lengths: sum_t b_t = sum of the block's lengths (a prefix sum), and the timesteps
// with more than k alive pieces are those of the block's piece number k.  Producer and
// consumer group g run the same block, and everything between them is per group: chunks of the group's own
// timesteps, tiles over the group's own rows (gathered: a group's rows of a timestep are consecutive, those of
// a chunk are not), completion counters of its own.  So a group never waits for another one: with
// the pieces dealt round-robin all groups had to march in step, and every step paid for a third of all alive pieces.
//
// Hand-over (lstm_rec.h, PipeLink): producer rows are written through to memory and their completion is
// published per group; every chunk belongs to a fixed set of workers that hold all of W_ih1 in their registers
// (work_deal); they write their columns of the result through, wait for the stores and count themselves in
// done[group][chunk]; the consumer group waits until that count has reached the number of the set's workers.  Waiting only ever points backwards along
// producer -> worker -> consumer and every worker takes a group's chunks in the order its consumer needs them,
// so the launch cannot deadlock; every wait is bounded and raises the shared error word on time-out.
#pragma once
#include "lstm_rec.h"

namespace ver {

constexpr int PIPE_GROUPS = 3;       // groups (XCDs) per layer
constexpr int TRIPLE_GROUPS = 2;     // the same with three layers in a launch
constexpr int PIPE_XCDS = 8;         // XCDs of the chip: those beyond the two layers' groups are workers
static_assert(PIPE_XCDS - 2 * PIPE_GROUPS == 2, "two worker XCDs");

// The plan of a launch (ints in global memory, written by plan_launches):
constexpr int PLAN_KB = 0;           // [PIPE_GROUPS + 1] first piece of every group's block, then the number of pieces
constexpr int PLAN_GROUPS = 4;       // [2] groups of a layer's time loop: the lower layers, the top one of three
constexpr int PLAN_ALONE = 6;        // not 0: too many alive pieces per timestep, the layers run alone (see plan_launches)
constexpr int PLAN_NO_PAIR = 7;      // three layers: 0 if the two lower ones share a launch
constexpr int PLAN_T = 8;            // [PIPE_GROUPS] timesteps of the group (those of its first piece; 0 if it has none)
constexpr int PLAN_NO_TRIPLE = 11;   // three layers: 0 if all share a launch
constexpr int PLAN_CT = 12;          // [PIPE_GROUPS] timesteps per chunk
constexpr int PLAN_TOP = 15;         // three layers: not 0 if the top one has a launch of its own
constexpr int PLAN_WORDS = 16;
inline __host__ __device__ size_t plan_scratch_floats(int M) { return 2 * ((size_t)M + 1); }
// The words a launch synchronises through (zero at launch): progress[g] at g, then done[g][chunk] from 16 with
// PIPE_GROUPS rows of pipe_done_stride(M) words.
constexpr int PIPE_CT_MIN = 2, PIPE_CT_MAX = 8;
inline __host__ __device__ int pipe_done_stride(int M) { return M / PIPE_CT_MIN + 2; }
inline __host__ __device__ int pipe_sync_words(int M) { return 16 + PIPE_GROUPS * pipe_done_stride(M); }

// Predicted microseconds of a timestep with b alive pieces of the group: step + low * min(b, 4) + over (more than four) + piece * b +
// tile * (ceil(b / 16) - 1): up to four pieces, up to 16 and more run in forms of their own.
struct PlanCost {
    float step, low, over, piece, tile;
    int chunk_rows, dense;   // rows per chunk that groups of more than 16 pieces aim at from `dense` alive pieces per timestep on
                             // (average over the launch), where the workers set the pace; 0: never
    int few;                 // timesteps per chunk of groups of up to 16 pieces
};
// Timesteps per chunk by the pieces of the group: a chunk is handed on when it is complete, so the consumer starts and
// ends that much later than the producer; it costs a worker about 4 us beside the product of its rows.
// Up to 16 pieces: 8, or 4 where the workers keep up with that: bf16 with three or more teams of workers (work_deal) or the long
// timesteps of the widths above 512.  us per forward and backward pass, 8 -> 4 timesteps, 200 rows in few pieces: 64 units 260 -> 250, 320
// 280 -> 271, 1024 389 -> 385; 800 rows in 12: 1024 449 -> 432; 3000 rows in 46: 192 421 -> 406; but 512 486 -> 500, and fp32 2 x 512 on
// 1024 rows 1062 -> 1099.
constexpr int PLAN_CT_FEW = 8, PLAN_CT_FEW_FAST = 4, PLAN_CT_MANY = 2;   // up to 16 pieces, more pieces
// fp32 forward from 384 units on, where only two teams of workers hold the weights and a tile costs them 1.8 to 2.5 us:
// with 48 alive pieces per timestep or more the workers are behind and long chunks pay, with fewer the delay costs more.  us per timestep with 32 equally long pieces per group (96 alive), chunks of 2
// timesteps -> of 256 rows: H = 384 9.0 -> 7.0, 512 10.7 -> 8.5; us per launch: 512 units, 32768 rows in 256 pieces (64
// alive) 3750 -> 3080, 8192 in 256 (64) 1075 -> 962, 4096 in 128 (39) 557 -> 611, 4096 in 64 (23) 604 -> 680.
// bf16 forward at 512 units: the same from 90 alive pieces on, with shorter chunks.  us per launch over equally long pieces,
// 2 timesteps -> 192 rows: 64 timesteps of 32 / 48 pieces per group 296 -> 256 / 359 -> 324, 128 timesteps 504 -> 529 / 702 -> 723, 24
// pieces (72 alive) 223 -> 253; 8192 rows in 192 pieces of about equal length 354 -> 318.  (Narrower layers have workers to spare: 448
// units, 32 timesteps of 48 pieces 222 -> 251.)
// us per timestep of launches over equally long pieces (time of a launch against its timesteps; up to 8 per group two layers, from 16 on one, since with
// as many in all three groups the workers set the pace, 1.7 us per 16 rows at H = 1024):
//   pieces               1     2     4     5     8    16    17    32    64
//   bf16 H=1024 fwd   1.25  1.24  1.42  1.89  1.93  2.08  3.59  4.59  8.6      bwd  1.58  1.61  2.01  2.36  2.38  2.94  5.29  6.48  12.3
//   bf16 H=512  fwd   0.90  0.88  0.94  1.27  1.27  1.29  2.53  2.86  6.0      bwd  1.16  1.16  1.34  1.48  1.51  1.95  3.03  4.35   8.5
//   fp32 H=512  fwd   1.12  1.42  2.05  3.02  3.00  2.98  5.88  6.08  12.4     bwd  1.28  1.82  2.74  3.59  3.53  4.18  7.32  7.92  15.9
// (backward beyond 16 pieces bf16 at 512 units is the form of lstm_rec.h, the others that of lstm_many.h.)  The constants
// are fitted by hand to it, and for the narrow bf16 layers to the other widths too (a tile backward 1.0 at 17 pieces, 1.4 at 64 and 512 units, 0.4 at
// 320; with 1.2 an update of 2 x 512 units and three layers of 320 take the same time).  Without the step from four to five pieces, two short groups of
// fp32 got five and more pieces each and ended 50 us after the long one: 2 x 512 on 1024 rows in 8; with 2.4 and 3.8 us per tile, what the wide layers
// took before, 8192 rows in about 100 pieces of 2 x 1024 units took 2.55 ms forward and backward, now 2.38.
inline PlanCost plan_cost(int mode, bool wide, bool fwd, int G, int workers) {
    const int teams = workers / G;
    if (mode == MODE_F32)
        return fwd ? PlanCost{0.85f, 0.25f, 0.7f, 0.06f, 2.2f, teams < 3 ? 256 : 0, 48, PLAN_CT_FEW} : PlanCost{0.85f, 0.42f, 0.45f, 0.06f, 3.f, 0, 0, PLAN_CT_FEW};
    if (wide) return fwd ? PlanCost{1.13f, 0.03f, 0.45f, 0.042f, 1.4f, 0, 0, PLAN_CT_FEW_FAST} : PlanCost{1.45f, 0.08f, 0.2f, 0.08f, 1.8f, 0, 0, PLAN_CT_FEW_FAST};
    const int few = teams < 3 ? PLAN_CT_FEW : PLAN_CT_FEW_FAST;
    return fwd ? PlanCost{0.84f, 0.f, 0.25f, 0.03f, 1.1f, G == REC_MAX_GROUP ? 192 : 0, 90, few} : PlanCost{1.09f, 0.01f, 0.05f, 0.05f, 1.f, 0, 0, few};
}

struct PipeWork {
    const void* A;      // producer rows [M, K], operand type (forward: h, backward: dz)
    const void* B;      // [N, K] operand type, K contiguous
    float* C;           // [M, N]
    const float* bias;  // [N] or NULL
    int K, N, M;
    const int32_t* t_off;
    const int* plan;
    int* sync;          // progress, done counters (see above)
    int* err;
    int G;              // workers of a team; each owns N / G columns
    int count;          // workers in all
    const int* alone;   // the planned kernels do nothing if it points to anything but a zero
};

constexpr int PLAN_THREADS = 1024;
// Exclusive prefix sums of N values per thread over the 1024 threads of the block (thread order); total: the sums.
// s_w: 16 * N words of LDS.
template <typename T, int N>
__device__ __forceinline__ void plan_scan(T (&v)[N], T* s_w, T (&total)[N]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    T inc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) inc[i] = v[i];
#pragma unroll
    for (int d = 1; d < 64; d <<= 1)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const T o = __shfl_up(inc[i], d, VER_WAVE);
            if (lane >= d) inc[i] += o;
        }
    if (lane == 63)
#pragma unroll
        for (int i = 0; i < N; ++i) s_w[wave * N + i] = inc[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        T off = 0, tot = 0;
        for (int w = 0; w < PLAN_THREADS / 64; ++w) {
            const T x = s_w[w * N + i];
            if (w < wave) off += x;
            tot += x;
        }
        total[i] = tot;
        v[i] = off + inc[i] - v[i];
    }
    __syncthreads();
}

// The plans of the forward and of the backward launch of one minibatch (the same packing, two cost models).
// IN_LDS: the batch sizes and the per-piece arrays (lengths and their prefix sums) live in LDS (up to PLAN_LDS_N
// pieces and timesteps: the search for the cuts is a chain of dependent reads of them), else in global memory.
constexpr int PLAN_LDS_N = 4096;
constexpr int PLAN_DIRS = 2;
template <bool IN_LDS>
__device__ __forceinline__ void plan_body(const int32_t* __restrict__ batch_sizes, int M, int n_seq, int T, int* __restrict__ plan_fwd,
                                          int* __restrict__ plan_bwd, float* __restrict__ scratch, int* s_bs, float* s_len, float* s_S1,
                                          const PlanCost& pc_fwd, const PlanCost& pc_bwd, int groups) {
    constexpr int WAVES = PLAN_THREADS / 64;
    __shared__ float s_wf[WAVES];
    __shared__ float s_obj[WAVES];
    __shared__ int s_k1[WAVES], s_k2[WAVES];
    __shared__ int s_kb[PLAN_DIRS][PIPE_GROUPS + 1];
    const int tid = threadIdx.x;
    const int32_t* bs = batch_sizes;
    if (IN_LDS) {
        for (int t = tid; t < T; t += PLAN_THREADS) s_bs[t] = batch_sizes[t];
        __syncthreads();
        bs = s_bs;
    }
    float* len = IN_LDS ? s_len : scratch;          // [n_seq] timesteps of piece n
    float* S1 = IN_LDS ? s_S1 : scratch + M + 1;    // [n_seq + 1] sum of len[j], j < n
    for (int t = tid; t < T; t += PLAN_THREADS) {
        const int hi = min(bs[t], n_seq), lo = t + 1 < T ? min(bs[t + 1], n_seq) : 0;
        for (int n = lo; n < hi; ++n) len[n] = (float)(t + 1);   // the pieces that end with timestep t
    }
    __syncthreads();
    float c1 = 0.f;
    for (int b0 = 0; b0 < n_seq; b0 += PLAN_THREADS) {
        const int n = b0 + tid;
        float l[1] = {n < n_seq ? len[n] : 0.f}, t1[1];
        plan_scan<float, 1>(l, s_wf, t1);
        if (n < n_seq) S1[n] = c1 + l[0];
        c1 += t1[0];
    }
    if (tid == 0) S1[n_seq] = c1;
    __syncthreads();
    // The first half of the block searches the cuts of the forward plan, the second half those of the backward plan.
    const int dir = tid / (PLAN_THREADS / PLAN_DIRS), rank = tid % (PLAN_THREADS / PLAN_DIRS);
    const PlanCost pc = dir == 0 ? pc_fwd : pc_bwd;
    // predicted time of a group that runs the pieces [lo, hi)
    auto cost = [&](int lo, int hi) -> float {
        if (hi <= lo) return 0.f;
        // timesteps with more than 16, 32, ... alive pieces; beyond 64 such terms the rest by the midpoint rule
        float P = 0.f;
        int k = lo + 16;
        for (int i = 0; i < 64 && k < hi; ++i, k += 16) P += len[k];
        if (k < hi) P += (S1[hi] - S1[k - 8]) * (1.f / 16.f);
        const float over = lo + QUAD_MAX < hi ? len[lo + QUAD_MAX] : 0.f;
        return pc.step * len[lo] + pc.low * (S1[min(lo + QUAD_MAX, hi)] - S1[lo]) + pc.over * over + pc.piece * (S1[hi] - S1[lo]) + pc.tile * P;
    };
    // every first cut k1 with the second cut that balances the two remaining groups; ties go to the smaller cuts
    float best = 3.0e38f;
    int bk1 = n_seq, bk2 = n_seq;
    for (int k1 = 1 + rank; k1 <= n_seq; k1 += PLAN_THREADS / PLAN_DIRS) {
        int lo = k1, hi = n_seq;
        while (lo < hi && groups != TRIPLE_GROUPS) {
            const int mid = (lo + hi) >> 1;
            if (cost(k1, mid) >= cost(mid, n_seq)) hi = mid; else lo = mid + 1;
        }
        const float c0 = cost(0, k1);
        if (groups == TRIPLE_GROUPS) lo = n_seq;   // (the third block stays empty)
        for (int k2 = groups == TRIPLE_GROUPS ? lo : max(lo - 1, k1); k2 <= lo; ++k2) {
            const float obj = fmaxf(c0, fmaxf(cost(k1, k2), cost(k2, n_seq)));
            if (obj < best) { best = obj; bk1 = k1; bk2 = k2; }
        }
    }
    // smallest (objective, k1, k2) of each half: inside the waves by shuffles, then over the half's waves
    auto better = [](float o, int o1, int o2, float m, int m1, int m2) { return o < m || (o == m && (o1 < m1 || (o1 == m1 && o2 < m2))); };
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const float o = __shfl_xor(best, d, VER_WAVE);
        const int o1 = __shfl_xor(bk1, d, VER_WAVE), o2 = __shfl_xor(bk2, d, VER_WAVE);
        if (better(o, o1, o2, best, bk1, bk2)) { best = o; bk1 = o1; bk2 = o2; }
    }
    if ((tid & 63) == 0) { s_obj[tid >> 6] = best; s_k1[tid >> 6] = bk1; s_k2[tid >> 6] = bk2; }
    __syncthreads();
    if (rank == 0) {
        for (int w = dir * (WAVES / PLAN_DIRS) + 1; w < (dir + 1) * (WAVES / PLAN_DIRS); ++w)
            if (better(s_obj[w], s_k1[w], s_k2[w], best, bk1, bk2)) { best = s_obj[w]; bk1 = s_k1[w]; bk2 = s_k2[w]; }
        s_kb[dir][0] = 0; s_kb[dir][1] = bk1; s_kb[dir][2] = bk2; s_kb[dir][3] = n_seq;
        int* plan = dir == 0 ? plan_fwd : plan_bwd;
        for (int g = 0; g <= PIPE_GROUPS; ++g) plan[PLAN_KB + g] = s_kb[dir][g];
    }
    __syncthreads();
    if (tid < PLAN_DIRS * PIPE_GROUPS) {   // per plan and group: its timesteps and its chunk length
        const int d = tid / PIPE_GROUPS, g = tid % PIPE_GROUPS;
        const int lo = s_kb[d][g], cap = s_kb[d][g + 1] - lo;
        int* plan = d == 0 ? plan_fwd : plan_bwd;
        plan[PLAN_T + g] = cap > 0 ? (int)len[lo] : 0;
        const PlanCost& p = d == 0 ? pc_fwd : pc_bwd;
        const int aim = M >= p.dense * T ? p.chunk_rows : 0;
        plan[PLAN_CT + g] = cap <= 16 ? p.few : min(max(aim / cap, PLAN_CT_MANY), PLAN_CT_FEW);
    }
}

// By one workgroup in front of the forward launch: clears that launch's synchronisation words and writes the plans of the
// forward and of the backward launch (see the top of this file).  scratch: plan_scratch_floats(M) floats.
struct PlanArgs {
    const int32_t* info; const int32_t* batch_sizes;
    int M;
    int* plan_fwd; int* plan_bwd; float* scratch;
    int* clear; int n_clear;
    PlanCost fwd, bwd;                // of the launches of two layers
    // Two layers share a launch up to min(most, base + T / per) alive pieces per timestep (average over the T timesteps) and up to `rows` rows;
    // most = 0: always.
    int base, per, most, rows;
    // Three layers do up to n1 alive pieces, up to n2 where 2 T >= t2 + s2 times their number, and up to n3 from t3 timesteps on; else
    // the two lower ones do by the rule above.
    PlanCost fwd_three, bwd_three;
    int three;                        // 0: not three layers, 1: by the rule, 2: always
    int n1, n2, t2, s2, n3, t3;
};
// Whether all of three layers share a launch (M rows over T timesteps).
inline __host__ __device__ bool plan_three(const PlanArgs& a, int M, int T) {
    const long long m = M, t = T;
    return a.three == 2 || m <= a.n1 * t || (m <= a.n2 * t && 2 * t * t >= a.t2 * t + a.s2 * m) || (m <= a.n3 * t && T >= a.t3);
}
struct PlanLds {
    int bs[PLAN_LDS_N];
    float len[PLAN_LDS_N], S1[PLAN_LDS_N + 1];
};
__device__ __forceinline__ void plan_launches(const PlanArgs& a, PlanLds& lds) {
    const int M = a.M, n_seq = min(max(a.info[0], 0), M), T = min(max(a.info[1], 0), M);
    for (int i = threadIdx.x; i < a.n_clear; i += PLAN_THREADS) a.clear[i] = 0;
    const bool triple = a.three != 0 && plan_three(a, M, T);
    const bool alone = !triple && a.most > 0 && M > a.rows && M > min(a.most, a.base + T / a.per) * T;
    if (threadIdx.x < PLAN_DIRS) {
        int* plan = threadIdx.x == 0 ? a.plan_fwd : a.plan_bwd;
        plan[PLAN_ALONE] = alone ? 1 : 0;
        plan[PLAN_NO_PAIR] = triple || alone ? 1 : 0;
        plan[PLAN_NO_TRIPLE] = triple ? 0 : 1;
        plan[PLAN_TOP] = triple ? 0 : 1;
        plan[PLAN_GROUPS] = triple ? TRIPLE_GROUPS : alone ? REC_GROUPS : PIPE_GROUPS;
        plan[PLAN_GROUPS + 1] = triple ? TRIPLE_GROUPS : REC_GROUPS;
    }
    if (alone) return;
    const PlanCost fwd = triple ? a.fwd_three : a.fwd, bwd = triple ? a.bwd_three : a.bwd;
    const int groups = triple ? TRIPLE_GROUPS : PIPE_GROUPS;
    if (n_seq <= PLAN_LDS_N && T <= PLAN_LDS_N)
        plan_body<true>(a.batch_sizes, M, n_seq, T, a.plan_fwd, a.plan_bwd, a.scratch, lds.bs, lds.len, lds.S1, fwd, bwd, groups);
    else
        plan_body<false>(a.batch_sizes, M, n_seq, T, a.plan_fwd, a.plan_bwd, a.scratch, lds.bs, lds.len, lds.S1, fwd, bwd, groups);
}

// One 128 x 256 tile of C[M, N] = A[M, K] B[N, K]^T + bias for bf16 operands, by 8 waves (2 x 4 of 64 x 64) of a workgroup
// that has the CU to itself: K-tiles of 64 go from global memory straight into LDS (three stages, two K-tiles in flight
// while one is multiplied, one barrier per K-tile, no registers or LDS stores in between).  An LDS row is the 128 bytes
// of a tile row, as 8 chunks of 16 bytes; chunk position p of row r holds chunk p ^ ((r >> 1) & 7), which makes the
// 16-byte MFMA operand reads of 16 consecutive rows hit all banks once.  A load instruction fills 8 rows (lane -> row
// lane / 8, position lane % 8), so the swizzle is applied on the global side.
constexpr int PIPE_BM = 128;         // rows per GEMM tile
constexpr int PIPE_BN = 256;         // columns per GEMM tile
constexpr int PIPE_STAGES = 3;
constexpr int PIPE_STAGE_BYTES = (PIPE_BM + PIPE_BN) * 128;
// K need not be a multiple of 64 (it is a multiple of 4): the last K-tile then also fetches what follows the rows'
// ends (the next row, or zeros past the end of the arrays), and the A operand is cleared beyond K in registers, so
// that whatever was fetched on the B side is multiplied by zero.
struct ProjWork {
    const void* A;      // [M, K]
    const void* B;      // [N, K]
    float* C;           // [M, N]
    const float* bias;  // [N] or NULL
    int K, N, M;
    const int* alone;   // (gemm_group.h)
};
__device__ __forceinline__ void proj_tile_dma(const ProjWork& w, int row0, int row_end, int col0, unsigned char* smem) {
    constexpr int BK = 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 2) * 64, wn = (wave & 3) * 64;
    const int lr = lane & 15, lk = lane >> 4;
    const int K = w.K, N = w.N, nk = (K + BK - 1) / BK, k_tail = K % BK;
    const int ncols = min(N - col0, PIPE_BN);
    __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(static_cast<const bf16_t*>(w.A)) + (size_t)row0 * K, 0, (row_end - row0) * K * 2, 0x00020000);
    __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(static_cast<const bf16_t*>(w.B)) + (size_t)col0 * K, 0, ncols * K * 2, 0x00020000);
    // source offsets of this lane in the 2 (A) + 4 (B) load instructions of this wave per K-tile
    int voffA[2], voffB[4];
    const int row_in = lane >> 3, pos = lane & 7;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = (wave * 2 + j) * 8 + row_in;
        voffA[j] = row * K * 2 + ((pos ^ ((row >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = (wave * 4 + j) * 8 + row_in;
        voffB[j] = row * K * 2 + ((pos ^ ((row >> 1) & 7)) << 4);
    }
    auto issue = [&](int kt) {
        unsigned char* st = smem + (kt % PIPE_STAGES) * PIPE_STAGE_BYTES;
#pragma unroll
        for (int j = 0; j < 2; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_ptr_t)(st + (wave * 2 + j) * 1024), 16, voffA[j], kt * BK * 2, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (lds_ptr_t)(st + PIPE_BM * 128 + (wave * 4 + j) * 1024), 16, voffB[j],
                                                     kt * BK * 2, 0, 0);
    };
    // operand read offsets: row byte offset and swizzle of this lane's row in each 16-row tile
    int arow[4], asw[4], brow[4], bsw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int ra_ = wm + i * 16 + lr, rb_ = wn + i * 16 + lr;
        arow[i] = ra_ * 128; asw[i] = (ra_ >> 1) & 7;
        brow[i] = PIPE_BM * 128 + rb_ * 128; bsw[i] = (rb_ >> 1) & 7;
    }
    f32x4_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    issue(0);
    if (nk > 1) issue(1);
    for (int kt = 0; kt < nk; ++kt) {
        // this wave's loads of stage kt have landed (the 6 of stage kt+1 may still be in flight) ...
        if (kt + 1 < nk) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        bar_lds();   // ... and so have everyone's; everyone has also finished reading stage kt-1
        if (kt + 2 < nk) issue(kt + 2);   // into the stage that was read in iteration kt-1
        const unsigned char* st = smem + (kt % PIPE_STAGES) * PIPE_STAGE_BYTES;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            u16x8_t a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                a[i] = *reinterpret_cast<const u16x8_t*>(st + arow[i] + (((ks * 4 + lk) ^ asw[i]) << 4));
            if (k_tail != 0 && kt == nk - 1) {
                // this lane's 8 elements start at ks * 32 + lk * 8 of the K-tile: clear the pairs beyond K
                const int e0 = ks * 32 + lk * 8;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    u32x4_t v = __builtin_bit_cast(u32x4_t, a[i]);
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = e0 + 2 * q < k_tail ? v[q] : 0u;
                    a[i] = __builtin_bit_cast(u16x8_t, v);
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                b[j] = *reinterpret_cast<const u16x8_t*>(st + brow[j] + (((ks * 4 + lk) ^ bsw[j]) << 4));
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = mfma_bf16_16x16x32(a[i], b[j], acc[i][j]);
        }
    }
    // C fragment: element e of lane l is row (l / 16) * 4 + e, column l % 16 of the 16x16 tile
    __amdgpu_buffer_rsrc_t rsC = __builtin_amdgcn_make_buffer_rsrc(w.C + (size_t)row0 * N, 0, (row_end - row0) * N * 4, 0x00020000);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int crow = (wm + i * 16 + lk * 4) * N * 4;   // rows the tile does not have are dropped (buffer bounds)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = col0 + wn + j * 16 + lr;
            if (n >= N) continue;
            const float bv = w.bias ? w.bias[n] : 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][e] + bv), rsC, crow + (e * N + n) * 4, 0, 0);
        }
    }
}

// C[M, N] = A[M, K] B[N, K]^T + bias (the input projection of the first layer).  One workgroup per tile; consecutive
// workgroups (dealt round-robin to the XCDs) take the column tiles of one row tile, so that a row tile of A is fetched
// from memory by one round of workgroups.
static __global__ __launch_bounds__(REC_THREADS) void lstm_proj_dma_kernel(ProjWork w, int tiles_n) {
    extern __shared__ __attribute__((aligned(16))) unsigned char proj_smem[];
    if (w.alone && *w.alone == 0) return;
    const int rt = blockIdx.x / tiles_n, ct = blockIdx.x % tiles_n;
    proj_tile_dma(w, rt * PIPE_BM, min(w.M, (rt + 1) * PIPE_BM), ct * PIPE_BN, proj_smem);
}

// How the chunks of a group of `cap` pieces are dealt to the workers.  G workers hold the weights once (a team); both XCDs
// together hold WORK_COUNT / G teams, which form sets: the chunks go to the sets in turn, and the teams of a set share the
// rows of a chunk.  Up to 16 pieces a chunk is a handful of tiles of 16 rows and every team is a set of its own; with
// more, 16, 8 and 4 teams are two sets, so that a chunk of hundreds of rows does not wait for a single team.
constexpr int WORK_COUNT = (PIPE_XCDS - 2 * PIPE_GROUPS) * REC_MAX_GROUP;
constexpr int TRIPLE_WORK_COUNT = REC_MAX_GROUP;   // (three layers: an XCD for each of the two products)
static_assert(PIPE_XCDS - 3 * TRIPLE_GROUPS == 2, "an XCD of workers per product");
struct WorkDeal {
    int sets, share;   // a set is 1 << share teams
};
inline __host__ __device__ WorkDeal work_deal(int G, int cap, int count = WORK_COUNT) {
    const int teams = count / G;
    const int share = cap > 16 && teams % 2 == 0 ? __builtin_ctz(teams) - 1 : 0;
    return WorkDeal{teams >> share, share};
}

// One group's view of the hand-over words, from the plan.
// out: the product that takes this layer's rows, in: the one that makes its input (with two layers the same for both).
__device__ __forceinline__ PipeLink pipe_link_of(const PipeWork& out, const PipeWork& in, int g) {
    const int* plan = in.plan;
    PipeLink pl;
    pl.progress = out.sync + g;
    pl.done = in.sync + 16 + g * pipe_done_stride(in.M);
    pl.need = in.G << work_deal(in.G, plan[PLAN_KB + g + 1] - plan[PLAN_KB + g], in.count).share;
    pl.ct = plan[PLAN_CT + g];
    pl.T = plan[PLAN_T + g];
    return pl;
}
__device__ __forceinline__ PieceSet pipe_pieces_of(const int* plan, int g) {
    const int lo = plan[PLAN_KB + g];
    return PieceSet{lo, 1, plan[PLAN_KB + g + 1] - lo, g};
}

// ---- workers -------------------------------------------------------------------------------------------------
// The 32 CUs of an XCD hold 8 MB of weights in their registers, which is all of W_ih1 (as it is all of a W_hh): a worker
// keeps the weights of its N / G columns resident, in the layout of the time loops of lstm_few.h (8 waves, each an
// eighth of the contraction), and turns 16 rows at a time into the consumer's input.  What bounds it: the 16 MFMA
// cycles per weight operand and 16 rows (0.43 us at H = 1024), the partial sums of 16 rows through LDS (64 KB forward),
// and per chunk the round trips of progress word, rows and stores (about 4 us).  (128 x 256 tiles that streamed the
// weights from L2 through LDS took 18 us forward and 54 us backward each, 14 and 38 us for a handful of rows: the
// consumer started and ended that much later, and 32768 rows kept the two XCDs busy for 2.9 ms.)
// Where a third of the 64 workers or fewer hold the weights (up to 320 units; 576 and 640), the others hold them again
// (work_deal).  One team per XCD left 28 of 32 CUs idle at H = 64 and made the workers the bound of launches over hundreds
// of pieces: fp32 forward on 32768 rows in 1024 pieces 2.40 ms, now 1.44 (H = 320 in 256 pieces 3.9 -> 2.6 ms).
constexpr int WORK_LDS_T = 2047;   // timesteps whose row offsets are kept in LDS
inline __host__ __device__ size_t work_lds_bytes(int cols, int nb, int bufs) {
    return (size_t)bufs * few_part_floats(cols) * sizeof(float) + (size_t)REC_WAVES * few_stage_bytes(nb) + (WORK_LDS_T + 1) * sizeof(int);
}

__device__ __forceinline__ void work_load_lds(__amdgpu_buffer_rsrc_t rs, unsigned char* lds, unsigned off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)lds, 16, off, 0, 0, 17);
}
// Requests this wave's slice of 16 rows (numbers in LDS) into its staging area; a lane's LDS address is the load's base + 16 * lane.
template <int NB>
__device__ __forceinline__ void work_request(__amdgpu_buffer_rsrc_t rs, unsigned char* stage, const int* rows, unsigned row_bytes, int b_lo, int n_blk) {
#pragma unroll
    for (int j = 0; j < FewStage<NB>::LOADS; ++j) {
        const int r = FewStage<NB>::row(j);
        work_load_lds(rs, stage + j * 1024, (unsigned)rows[r] * row_bytes + (unsigned)b_lo * 64u + FewStage<NB>::src(r, n_blk));
    }
}

// The fp32 forward workers add up the partial sums of a tile behind the MFMAs of the next one: two buffers of them.
template <int MODE, bool FWD> constexpr int work_bufs() { return FWD && MODE == MODE_F32 ? 2 : 1; }
// First block of slice s when the contraction is dealt evenly over the waves; slices s and s + 4 round to opposite sides.
inline __host__ __device__ int work_even(int blocks, int s) { return (s * blocks + (s > REC_WAVES / 2 ? REC_WAVES - 1 : 0)) / REC_WAVES; }

// FWD: 16 * MT columns per worker, four of them (a unit's gates) per thread; else one column per thread.
// EVEN: the contraction is dealt evenly over the waves (w and w + 4 share a SIMD) instead of NB blocks at a time.  For fp32 forward below H = 512, where the MFMAs set the pace: two layers of 384 on
// 32768 rows in 256 pieces 2.9 ms instead of 4.0.
template <int MODE, int MT, int NB, bool FWD, bool EVEN>
__device__ __forceinline__ void pipe_worker(const PipeWork& w, int id, unsigned char* smem) {
    typedef typename RecGeom<MODE>::E E;
    constexpr int es = (int)sizeof(E), KBLK = RecGeom<MODE>::KBLK, VEC = RecGeom<MODE>::VEC;
    constexpr int COLS = 16 * MT, ROW = few_row(COLS), PER = FWD ? 4 : 1, TPR = COLS / PER;   // threads per row
    static_assert(16 * TPR <= REC_THREADS, "a thread per row and column group");
    constexpr bool DESCEND = !FWD;   // the backward consumer needs the last chunk first
    const int team = id / w.G, rank = id % w.G;
    __shared__ int s_sel[2];
    __shared__ int s_row[REC_THREADS];
    float* part = reinterpret_cast<float*>(smem);
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int BUFS = work_bufs<MODE, FWD>();
    unsigned char* stages = smem + (size_t)BUFS * few_part_floats(COLS) * sizeof(float);
    unsigned char* stage = stages + wave * few_stage_bytes(NB);
    int* s_toff = reinterpret_cast<int*>(stages + REC_WAVES * few_stage_bytes(NB));
    const int K = w.K, N = w.N, blocks = K / KBLK, n_slices = EVEN ? REC_WAVES : (blocks + NB - 1) / NB;
    // (which slice a wave takes rotates with the rank: all workers read the same rows at the same moment)
    const int slice = n_slices == REC_WAVES ? (wave + rank) % REC_WAVES : wave;
    const int b_lo = EVEN ? work_even(blocks, slice) : slice * NB;
    const int n_blk = EVEN ? work_even(blocks, slice + 1) - b_lo : min(NB, blocks - b_lo);
    f32x4_t wreg[MT * NB];
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const E* wrow = static_cast<const E*>(w.B) + ((size_t)rank * COLS + j * 16 + lr) * K + (b_lo * 4 + lk * n_blk) * VEC;
#pragma unroll
        for (int b = 0; b < NB; ++b)
            wreg[j * NB + b] = b < n_blk ? *reinterpret_cast<const f32x4_t*>(wrow + b * VEC) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < MT * NB; ++i) asm volatile("" : "+v"(wreg[i]));
    const int m = tid / TPR, col = rank * COLS + (tid % TPR) * PER;
    f32x4_t bias = {0.f, 0.f, 0.f, 0.f};
    if (FWD && w.bias) bias = *reinterpret_cast<const f32x4_t*>(w.bias + rank * COLS + (tid % TPR) * 4);
    int lo[PIPE_GROUPS], cap[PIPE_GROUPS], T[PIPE_GROUPS], ct[PIPE_GROUPS], at[PIPE_GROUPS], step[PIPE_GROUPS], share[PIPE_GROUPS], t_max = 0;
    float part_of[PIPE_GROUPS];   // of the group's chunks, one chunk
#pragma unroll
    for (int g = 0; g < PIPE_GROUPS; ++g) {
        lo[g] = w.plan[PLAN_KB + g];
        cap[g] = w.plan[PLAN_KB + g + 1] - lo[g];
        T[g] = w.plan[PLAN_T + g];
        ct[g] = w.plan[PLAN_CT + g];
        const int n = (T[g] + ct[g] - 1) / ct[g];
        // this team's first chunk of the group in the consumer's order (none: behind the last)
        const WorkDeal d = work_deal(w.G, cap[g], w.count);
        const int first = team < d.sets << d.share ? ((team >> d.share) + g) % d.sets : n;
        at[g] = DESCEND ? n - 1 - first : first;
        step[g] = DESCEND ? -d.sets : d.sets;
        share[g] = d.share;
        part_of[g] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(1.f / (float)max(n, 1))));
        t_max = max(t_max, T[g]);
    }
    for (int t = tid; t <= min(t_max, WORK_LDS_T); t += REC_THREADS) s_toff[t] = w.t_off[t];
#pragma unroll
    for (int i = 0; i < BUFS; ++i) few_clear_part<COLS>(part + i * few_part_floats(COLS));
    bar_lds();
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(w.A), 0, w.M * K * es, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsC = __builtin_amdgcn_make_buffer_rsrc(w.C, 0, w.M * N * 4, 0x00020000);
    int have = lane < PIPE_GROUPS && wave == 0 ? ld_agent(w.sync + lane) : 0;   // the producers' progress
    for (;;) {
        // The next chunk: of the groups whose producer has completed their next one, the one with the largest part still to come (the
        // plan makes them end together).  Taken in the order of the groups, the last group's consumer waited until the workers were through
        // with the first, wherever the producers are ahead of the workers: us per launch over 128 timesteps of 32 / 64 equally long pieces per
        // group, 1024 units (bf16) forward 842 / 1298 -> 691 / 1212, backward 948 -> 867; 512 units, fp32, 1301 / 2552 -> 1086 / 2103; evaluation of
        // 32768 rows in about 400 pieces of 2 x 1024 units 2530 -> 2376.
        if (wave == 0) {
            int sel = -1;
            long long spins = 0;
            for (;;) {
                bool left = false;
                float most = -1.f;
#pragma unroll
                for (int g = 0; g < PIPE_GROUPS; ++g) {
                    const bool more = DESCEND ? at[g] >= 0 : at[g] * ct[g] < T[g];
                    const int need = DESCEND ? T[g] - at[g] * ct[g] : min((at[g] + 1) * ct[g], T[g]);
                    const float still = DESCEND ? (float)(at[g] + 1) * part_of[g] : 1.f - (float)at[g] * part_of[g];
                    left = left || more;
                    if (more && still > most && __builtin_amdgcn_readlane(have, g) >= need) {
                        sel = g;
                        most = still;
                    }
                }
                if (sel >= 0 || !left) break;
                if ((++spins & 255) == 0 && (spins > REC_SPIN_LIMIT || ld_agent(w.err) != 0)) {
                    if (lane == 0) st_agent(w.err, 1);
                    break;
                }
                have = lane < PIPE_GROUPS ? ld_agent(w.sync + lane) : 0;
            }
            if (lane == 0) s_sel[0] = sel;
        }
        bar_lds();
        const int sel = __builtin_amdgcn_readfirstlane(s_sel[0]);
        if (sel < 0) return;   // nothing left, or the wait was abandoned
        int g_lo = lo[0], g_cap = cap[0], g_T = T[0], g_ct = ct[0], g_share = share[0], c = at[0];
#pragma unroll
        for (int g = 0; g < PIPE_GROUPS; ++g)
            if (sel == g) {
                g_lo = lo[g]; g_cap = cap[g]; g_T = T[g]; g_ct = ct[g]; g_share = share[g]; c = at[g];
                at[g] += step[g];
            }
        // The group's rows of the chunk in time order: lane k holds what is needed of its timestep k.
        const int t0 = c * g_ct, nt = min(g_ct, g_T - t0);
        const int tk = t0 + min(lane, nt);
        const int off_k = tk <= WORK_LDS_T ? s_toff[tk] : w.t_off[tk];
        const int off_k1 = __shfl(off_k, min(lane + 1, nt), VER_WAVE);   // (all lanes active: lane nt is read)
        const int cnt = lane < nt ? min(max(off_k1 - off_k - g_lo, 0), g_cap) : 0;
        int before = cnt;   // inclusive prefix over the lanes, then exclusive
#pragma unroll
        for (int d = 1; d < 2 * PIPE_CT_MAX; d <<= 1) {
            const int o = __shfl_up(before, d, VER_WAVE);
            if (lane >= d) before += o;
        }
        const int total = __builtin_amdgcn_readlane(before, nt - 1);
        before -= cnt;
        const int row_k = off_k + g_lo - before;   // row of slot s of timestep k: row_k + s
        // this team's share of the chunk: whole tiles
        const int mine = team & ((1 << g_share) - 1), tiles = (total + 15) >> 4;
        const int s_lo = (tiles * mine >> g_share) << 4, s_hi = min((tiles * (mine + 1) >> g_share) << 4, total);
        auto row_of = [&](int s) {
            int k = 0;
            for (int j = 1; j < nt; ++j) k += s >= __builtin_amdgcn_readlane(before, j) ? 1 : 0;
            return __shfl(row_k, k, VER_WAVE) + s;
        };
        // 16 rows at a time, their numbers from a table of up to REC_THREADS rows.  A wave's slice of the rows goes from memory
        // straight into its staging area (few_stage_product says how it lies there); the next tile's is requested as
        // soon as this one's operands have been read, and arrives behind the last MFMAs and the partial sums.  (Every store is issued, out of
        // range for rows that a tile does not have: a store that may or may not be there makes the wait for the loads
        // before it a wait for the store.)
        const bool works = n_blk > 0;
        // Requested ahead of the MFMAs where they take long enough to be worth the separation from the reads: fp32 (2 x 512
        // forward on 32768 rows in 1024 pieces 3.75 -> 3.60 ms) and wide bf16 (2 x 1024 on 4096 rows in 64 445 -> 437 us), not
        // narrow bf16 (2 x 512 on 32768 rows in 256 1.59 -> 1.62 ms).
        constexpr bool EARLY = MODE == MODE_F32 || MT == 8 || MT == 2;
        // this thread's columns of a tile: read its partial sums, add them, store them at `out`
        constexpr unsigned NOWHERE = 0xFFFFFFF0u;
        typedef typename std::conditional<FWD, f32x4_t, float>::type col_t;
        const float* mine_part = part + min(m, 15) * ROW + (tid % TPR) * PER;
        auto read_part = [&](const float* q, col_t (&o)[REC_WAVES]) {
#pragma unroll
            for (int k = 0; k < REC_WAVES; ++k) o[k] = *reinterpret_cast<const col_t*>(q + k * (16 * ROW));
        };
        auto add_store = [&](const col_t (&o)[REC_WAVES], unsigned out) {
            if constexpr (FWD) {
                f32x4_t v = bias;
#pragma unroll
                for (int k = 0; k < REC_WAVES; ++k) {
                    v[0] += o[k][0]; v[1] += o[k][1]; v[2] += o[k][2]; v[3] += o[k][3];
                }
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), rsC, out, 0, 17);
            } else {
                float v = 0.f;
#pragma unroll
                for (int k = 0; k < REC_WAVES; ++k) v += o[k];
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rsC, out, 0, 17);
            }
        };
        unsigned out_before = NOWHERE;   // two buffers: where the tile before goes, which is in buffer buf ^ 1
        int buf = 0;
        for (int b0 = s_lo; b0 < s_hi; b0 += REC_THREADS) {
            const int n = min(s_hi - b0, REC_THREADS);
            s_row[tid] = row_of(min(b0 + tid, total - 1));
            bar_lds();
            if (works) work_request<NB>(rsA, stage, s_row, (unsigned)(K * es), b_lo, n_blk);
            for (int r0 = 0; r0 < n; r0 += 16) {
                const int rows = min(16, n - r0);
                const int out_row = s_row[r0 + min(m, 15)];
                const unsigned out = m < rows ? ((unsigned)out_row * (unsigned)N + col) * 4u : NOWHERE;
                if (r0 == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(1)" ::: "memory");   // (the store of the tile before)
                col_t o[REC_WAVES];
                if (works) {
                    f32x4_t acc[MT];
#pragma unroll
                    for (int j = 0; j < MT; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                    auto next = [&] {
                        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (the operands have been read)
                        if (r0 + 16 < n) work_request<NB>(rsA, stage, s_row + r0 + 16, (unsigned)(K * es), b_lo, n_blk);
                        if (BUFS == 2) read_part(mine_part + (buf ^ 1) * few_part_floats(COLS), o);
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    few_stage_product<MODE, MT, NB, EVEN>(wreg, stage, part + COLS, n_blk, acc, [&] { if (EARLY) next(); });
                    if (!EARLY) next();
                    few_stage_write<MT>(acc, rows, part + buf * few_part_floats(COLS) + slice * (16 * ROW));
                } else if (BUFS == 2) {
                    read_part(mine_part + (buf ^ 1) * few_part_floats(COLS), o);
                }
                if (BUFS == 2) {
                    add_store(o, out_before);
                    out_before = out;
                    buf ^= 1;
                }
                bar_lds();
                if (BUFS == 1) {
                    read_part(mine_part, o);
                    add_store(o, out);
                    bar_lds();   // (the partial sums have been read)
                }
            }
        }
        if (BUFS == 2) {
            col_t o[REC_WAVES];
            read_part(mine_part + (buf ^ 1) * few_part_floats(COLS), o);
            add_store(o, out_before);
        }
        if (wave == 0) have = lane < PIPE_GROUPS ? ld_agent(w.sync + lane) : 0;   // (arrives while the stores complete)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        bar_lds();
        if (tid == 0) __hip_atomic_fetch_add(w.sync + 16 + sel * pipe_done_stride(w.M) + c, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// This workgroup's XCD and its ticket there (tickets[PIPE_XCDS], zero at launch).
__device__ __forceinline__ int xcc_ticket(int* tickets, int& xcc) {
    __shared__ int s_t, s_x;
    if (threadIdx.x == 0) {
        const int id = __builtin_amdgcn_s_getreg((3 << 11) | 20) & 0xf;   // HW_REG_XCC_ID, 4 bits
        s_x = id;
        s_t = id < PIPE_XCDS ? __hip_atomic_fetch_add(&tickets[id], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : REC_MAX_GROUP;
    }
    __syncthreads();
    xcc = __builtin_amdgcn_readfirstlane(s_x);   // (see rec_rank)
    return __builtin_amdgcn_readfirstlane(s_t);
}

struct PipeFwdArgs {
    RecFwdArgs l0, l1;   // producer (layer 0) and consumer (layer 1)
    PipeWork work;
};
template <int MODE, int TPW, int KS, int NBW, bool STATIC>
__device__ __forceinline__ void pipe_fwd_body(const PipeFwdArgs& p, unsigned char* smem) {
    int xcc;
    const int rank = xcc_ticket(p.l0.ticket, xcc);
    const int g = xcc < PIPE_GROUPS ? xcc : xcc - PIPE_GROUPS;
#ifdef VER_REC_PROF
    const bool stamp = threadIdx.x == 0 && rank == 0 && xcc < PIPE_XCDS;   // when every XCD's first workgroup starts and ends
    long long* tl = p.l0.prof + 64 + xcc * 2;
    if (stamp) tl[0] = wall_clock64();
#endif
    if (xcc < 2 * PIPE_GROUPS) {
        const PipeLink link = pipe_link_of(p.work, p.work, g);
        const PieceSet ps = pipe_pieces_of(p.work.plan, g);
        if (xcc < PIPE_GROUPS) {
            if (rank < p.l0.G)
                rec_fwd_body<MODE, TPW, KS, NBW, STATIC, PIPE_PRODUCER>(p.l0, rank, ps, link.T, p.l0.flags + xcc * REC_MAX_GROUP, link, smem);
        } else {
            if (rank < p.l1.G)
                rec_fwd_body<MODE, TPW, KS, NBW, STATIC, PIPE_CONSUMER>(p.l1, rank, ps, link.T, p.l1.flags + xcc * REC_MAX_GROUP, link, smem);
        }
    } else if (xcc < PIPE_XCDS && rank < REC_MAX_GROUP) {
        constexpr int WMT = REC_WAVES / KS * TPW;
        pipe_worker<MODE, WMT, FewBlocks<MODE, WMT == 8>::fwd, true, MODE == MODE_F32 && !STATIC>(p.work, (xcc - 2 * PIPE_GROUPS) * REC_MAX_GROUP + rank, smem);
    }
#ifdef VER_REC_PROF
    if (stamp) tl[1] = wall_clock64();
#endif
}
template <int MODE, int TPW, int KS, int NBW, bool STATIC>
__global__ __launch_bounds__(REC_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void lstm_pipe_fwd_kernel(PipeFwdArgs p_by_value) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    pipe_fwd_body<MODE, TPW, KS, NBW, STATIC>(pipe_args_in_place<PipeFwdArgs>(p_by_value), smem);
}
// The same where the plan decides whether it runs.  (With the question in the kernels above, which two-layer networks use, the
// compiler schedules their time loops otherwise: update of 2 x 512 units, backward launches 4277 us instead of 4233.)
template <int MODE, int TPW, int KS, int NBW, bool STATIC>
__global__ __launch_bounds__(REC_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void lstm_pipe_fwd_planned_kernel(PipeFwdArgs p_by_value) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const PipeFwdArgs& p = pipe_args_in_place<PipeFwdArgs>(p_by_value);
    if (*p.work.alone != 0) return;
    pipe_fwd_body<MODE, TPW, KS, NBW, STATIC>(p, smem);
}

struct PipeBwdArgs {
    RecBwdArgs l1, l0;   // producer (layer 1) and consumer (layer 0)
    PipeWork work;
};
template <int MODE, int MT, int KS, int NI>
__device__ __forceinline__ void pipe_bwd_body(const PipeBwdArgs& p, unsigned char* smem) {
    int xcc;
    const int rank = xcc_ticket(p.l1.ticket, xcc);
    const int g = xcc < PIPE_GROUPS ? xcc : xcc - PIPE_GROUPS;
#ifdef VER_REC_PROF
    const bool stamp = threadIdx.x == 0 && rank == 0 && xcc < PIPE_XCDS;
    long long* tl = p.l1.prof - 16 + 64 + xcc * 2;
    if (stamp) tl[0] = wall_clock64();
#endif
    if (xcc < 2 * PIPE_GROUPS) {
        const PipeLink link = pipe_link_of(p.work, p.work, g);
        const PieceSet ps = pipe_pieces_of(p.work.plan, g);
        if (xcc < PIPE_GROUPS) {
            if (rank < p.l1.G)
                rec_bwd_body<MODE, MT, KS, NI, PIPE_PRODUCER>(p.l1, rank, ps, link.T, p.l1.flags + xcc * REC_MAX_GROUP, link, smem);
        } else {
            if (rank < p.l0.G)
                rec_bwd_body<MODE, MT, KS, NI, PIPE_CONSUMER>(p.l0, rank, ps, link.T, p.l0.flags + xcc * REC_MAX_GROUP, link, smem);
        }
    } else if (xcc < PIPE_XCDS && rank < REC_MAX_GROUP) {
        pipe_worker<MODE, MT, FewBlocks<MODE, MT == 2>::bwd, false, false>(p.work, (xcc - 2 * PIPE_GROUPS) * REC_MAX_GROUP + rank, smem);
    }
#ifdef VER_REC_PROF
    if (stamp) tl[1] = wall_clock64();
#endif
}
template <int MODE, int MT, int KS, int NI>
__global__ __launch_bounds__(REC_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void lstm_pipe_bwd_kernel(PipeBwdArgs p_by_value) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    pipe_bwd_body<MODE, MT, KS, NI>(pipe_args_in_place<PipeBwdArgs>(p_by_value), smem);
}
template <int MODE, int MT, int KS, int NI>
__global__ __launch_bounds__(REC_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void lstm_pipe_bwd_planned_kernel(PipeBwdArgs p_by_value) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const PipeBwdArgs& p = pipe_args_in_place<PipeBwdArgs>(p_by_value);
    if (*p.work.alone != 0) return;
    pipe_bwd_body<MODE, MT, KS, NI>(p, smem);
}

// ---- three layers -------------------------------------------------------------------------------------------------
// The same with two XCDs per layer and one for each of the two products between them; the middle layer is consumer of one
// and producer of the other.  A pair and then a top layer alone walk T_max dependent timesteps twice; here the third layer ends two
// chunks after the first.  (Planned: run_fwd in lstm.hip says when it runs.)
struct TripleFwdArgs {
    RecFwdArgs l[3];     // producer, middle, consumer
    PipeWork work[2];
};
struct TripleBwdArgs {
    RecBwdArgs l[3];     // producer (the top layer), middle, consumer
    PipeWork work[2];
};
template <typename F0, typename F1, typename F2, typename W>
__device__ __forceinline__ void triple_roles(int xcc, int rank, int G, F0&& producer, F1&& middle, F2&& consumer, W&& worker) {
    const int g = xcc % TRIPLE_GROUPS;
    if (xcc < 3 * TRIPLE_GROUPS) {
        if (rank >= G) return;
        if (xcc < TRIPLE_GROUPS) producer(g);
        else if (xcc < 2 * TRIPLE_GROUPS) middle(g);
        else consumer(g);
    } else if (xcc < PIPE_XCDS && rank < TRIPLE_WORK_COUNT) {
        worker(xcc - 3 * TRIPLE_GROUPS);
    }
}
template <int MODE, int TPW, int KS, int NBW, bool STATIC>
__global__ __launch_bounds__(REC_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void lstm_triple_fwd_kernel(TripleFwdArgs p_by_value) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const TripleFwdArgs& p = pipe_args_in_place<TripleFwdArgs>(p_by_value);
    if (*p.work[0].alone != 0) return;
    int xcc;
    const int rank = xcc_ticket(p.l[0].ticket, xcc);
    triple_roles(xcc, rank, p.l[0].G,
        [&](int g) { rec_fwd_body<MODE, TPW, KS, NBW, STATIC, PIPE_PRODUCER>(p.l[0], rank, pipe_pieces_of(p.work[0].plan, g), p.work[0].plan[PLAN_T + g],
                         p.l[0].flags + xcc * REC_MAX_GROUP, pipe_link_of(p.work[0], p.work[0], g), smem); },
        [&](int g) { rec_fwd_body<MODE, TPW, KS, NBW, STATIC, PIPE_MIDDLE>(p.l[1], rank, pipe_pieces_of(p.work[0].plan, g), p.work[0].plan[PLAN_T + g],
                         p.l[1].flags + xcc * REC_MAX_GROUP, pipe_link_of(p.work[1], p.work[0], g), smem); },
        [&](int g) { rec_fwd_body<MODE, TPW, KS, NBW, STATIC, PIPE_CONSUMER>(p.l[2], rank, pipe_pieces_of(p.work[0].plan, g), p.work[0].plan[PLAN_T + g],
                         p.l[2].flags + xcc * REC_MAX_GROUP, pipe_link_of(p.work[1], p.work[1], g), smem); },
        [&](int stage) {
            constexpr int WMT = REC_WAVES / KS * TPW;
            pipe_worker<MODE, WMT, FewBlocks<MODE, WMT == 8>::fwd, true, MODE == MODE_F32 && !STATIC>(p.work[stage], rank, smem);
        });
}
template <int MODE, int MT, int KS, int NI>
__global__ __launch_bounds__(REC_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void lstm_triple_bwd_kernel(TripleBwdArgs p_by_value) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const TripleBwdArgs& p = pipe_args_in_place<TripleBwdArgs>(p_by_value);
    if (*p.work[0].alone != 0) return;
    int xcc;
    const int rank = xcc_ticket(p.l[0].ticket, xcc);
    triple_roles(xcc, rank, p.l[0].G,
        [&](int g) { rec_bwd_body<MODE, MT, KS, NI, PIPE_PRODUCER>(p.l[0], rank, pipe_pieces_of(p.work[0].plan, g), p.work[0].plan[PLAN_T + g],
                         p.l[0].flags + xcc * REC_MAX_GROUP, pipe_link_of(p.work[0], p.work[0], g), smem); },
        [&](int g) { rec_bwd_body<MODE, MT, KS, NI, PIPE_MIDDLE>(p.l[1], rank, pipe_pieces_of(p.work[0].plan, g), p.work[0].plan[PLAN_T + g],
                         p.l[1].flags + xcc * REC_MAX_GROUP, pipe_link_of(p.work[1], p.work[0], g), smem); },
        [&](int g) { rec_bwd_body<MODE, MT, KS, NI, PIPE_CONSUMER>(p.l[2], rank, pipe_pieces_of(p.work[0].plan, g), p.work[0].plan[PLAN_T + g],
                         p.l[2].flags + xcc * REC_MAX_GROUP, pipe_link_of(p.work[1], p.work[1], g), smem); },
        [&](int stage) { pipe_worker<MODE, MT, FewBlocks<MODE, MT == 2>::bwd, false, false>(p.work[stage], rank, smem); });
}

}  // namespace ver
