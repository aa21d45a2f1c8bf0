// ver_lstm_fwd / ver_lstm_bwd: multi-layer LSTM actor-critic over a packed
// minibatch and back-propagation through time.
//
// Paper: section 4 "Architecture" (embedding + state vector -> 2-layer LSTM ->
// action distribution and value), sequences for BPTT from section 2.2.
//
// Per layer the work splits into what has no time dependence and what has:
//   time-batched (one MFMA GEMM over all M rows):  W_ih x_t + b  (forward),
//       dx = W_ih^T dz, dW_ih = dz^T x, dW_hh = dz^T h_{t-1}     (backward)
//   sequential (persistent kernels, W_hh resident in registers): h_{t-1} W_hh^T + gates
//       (forward), dz_t and W_hh dz_t (backward) - see lstm_rec.h.
// Internally the 4H gate rows are interleaved (row = unit*4 + gate); user-facing
// weights and gradients keep the gate-major order i,f,g,o of the declaration.
#include <algorithm>
#include <cstring>
#include <mutex>

#include "gemm_group.h"
#include "lstm_launch.h"

namespace ver {
namespace {

// ---------------------------------------------------------------- weight preparation
// dst[q][d] = W[(q%4)*H + q/4][d] and dstT[d][q]; q = unit*4 + gate.  A block moves a 64 x 64 tile through LDS so
// that the reads of W and both writes are contiguous along their fastest index.
// Four converted elements as one store (8 bytes bf16, 16 bytes fp32).
__device__ __forceinline__ void st4(float* p, float a, float b, float c, float d) { *reinterpret_cast<f32x4_t*>(p) = f32x4_t{a, b, c, d}; }
__device__ __forceinline__ void st4(bf16_t* p, float a, float b, float c, float d) {
    u16x4_t v;
    v.x = to_bf16(a); v.y = to_bf16(b); v.z = to_bf16(c); v.w = to_bf16(d);
    *reinterpret_cast<u16x4_t*>(p) = v;
}
// A thread moves 4 adjacent elements at a time (16-byte loads, 8- or 16-byte stores; cols is a multiple of 4):
// 16 lanes cover a tile row in either direction.
// All matrices and bias vectors of a call in one launch (blockIdx.z: the job; a launch per matrix took ~10 us each,
// most of it ramp and tail).  A tile per 256 threads: workgroups of that size for a single layer, for several workgroups of
// PLAN_THREADS, so that the plan of the two-layer launches (lstm_pipe.h) can be one of them, the first to start: as a launch of its own
// it took 7 to 30 us in front of the time loops.  (A single layer in workgroups of 1024, whose four tiles wait
// for each other: 1024 units and 36 inputs 13.0 us instead of 11.3, 512 units and 16384 inputs 79 instead of 58.)
constexpr int PREP_MAX_JOBS = 26;   // 2 matrices + 1 bias per layer, 8 layers; the fp32 rows of a bf16 call; words to clear
constexpr int PREP_BIAS = 0, PREP_ROWS = -1, PREP_CLEAR = -2;
struct PrepJob {
    const float* W;      // matrix [4H, cols] gate-major, or b_ih (bias job), or rows
    const float* b_hh;   // (bias jobs)
    void* dst; void* dstT;
    int cols;            // > 0, PREP_BIAS, PREP_ROWS or PREP_CLEAR
    size_t quads;        // rows: groups of four elements; clear: words
};
struct PrepArgs { PrepJob job[PREP_MAX_JOBS]; int n; };
// Rows converted to the operand type, four elements per thread and step.
template <typename E>
__device__ __forceinline__ void convert_rows(const float* __restrict__ src, E* __restrict__ dst, size_t quads, size_t first, unsigned stride) {
    for (size_t i = first; i < quads; i += stride) {
        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(src + i * 4);
        st4(dst + i * 4, v[0], v[1], v[2], v[3]);
    }
}
__global__ __launch_bounds__(256) void convert_rows_kernel(const float* __restrict__ src, bf16_t* __restrict__ dst, size_t quads, const int* __restrict__ alone) {
    if (alone && *alone == 0) return;   // (lstm_pipe.h: PLAN_ALONE)
    convert_rows(src, dst, quads, blockIdx.x * 256 + threadIdx.x, gridDim.x * 256);
}
constexpr size_t PREP_TILE_FLOATS = 64 * 65;
inline size_t prep_lds_bytes(int threads) {
    const size_t tiles = threads / 256 * PREP_TILE_FLOATS * sizeof(float);
    return threads == PLAN_THREADS ? std::max(tiles, sizeof(PlanLds)) : tiles;
}
// blockIdx.z = 0 is the plan where there is one (plan.plan_fwd != NULL), then the jobs; what is left belongs to the last job, the
// rows where there are any: x and y are as many as the widest matrix has tiles, 20 workgroups of 1024 for 64 units and 1044 inputs
// (us per launch with those / with a thread per four groups: 8192 rows of 1044 53 / 13, 32768 315 / 50; at most a quarter as many threads: 58).
constexpr size_t PREP_ROWS_QUADS = 4, PREP_ROWS_THREADS = 2048 * 1024;   // per thread; at most
template <typename E, int PREP_THREADS>
__global__ __launch_bounds__(PREP_THREADS) void prep_weights_kernel(PrepArgs a, int H, PlanArgs plan) {
    extern __shared__ __attribute__((aligned(16))) unsigned char prep_smem[];
    constexpr int PREP_TILES = PREP_THREADS / 256;
    const int planned = PREP_THREADS == PLAN_THREADS && plan.plan_fwd != nullptr ? 1 : 0;
    if constexpr (PREP_THREADS == PLAN_THREADS)
        if ((int)blockIdx.z < planned) {
            if (blockIdx.x == 0 && blockIdx.y == 0) plan_launches(plan, *reinterpret_cast<PlanLds*>(prep_smem));
            return;
        }
    const int z = blockIdx.z - planned, job = min(z, a.n - 1);
    const PrepJob& jb = a.job[job];   // (uniform index into the kernel arguments: scalar loads)
    const int cols = jb.cols;
    const unsigned wgs = gridDim.x * gridDim.y, wg = blockIdx.y * gridDim.x + blockIdx.x;
    if (cols == PREP_ROWS) {
        const unsigned layers = gridDim.z - planned - job;   // of the grid
        convert_rows(jb.W, static_cast<E*>(jb.dst), jb.quads, ((size_t)(z - job) * wgs + wg) * PREP_THREADS + threadIdx.x, layers * wgs * PREP_THREADS);
        return;
    }
    const unsigned first = wg * PREP_THREADS + threadIdx.x, stride = wgs * PREP_THREADS;
    if (cols == PREP_CLEAR) {
        for (unsigned i = first; i < jb.quads; i += stride) static_cast<int32_t*>(jb.dst)[i] = 0;
        return;
    }
    if (cols == PREP_BIAS) {   // bias: dst[q] = b_ih + b_hh, gate rows interleaved
        for (unsigned q = first; q < 4u * H; q += stride) {
            const int src = (q & 3) * H + (q >> 2);
            static_cast<float*>(jb.dst)[q] = jb.W[src] + jb.b_hh[src];
        }
        return;
    }
    const int tid = threadIdx.x & 255, sub = threadIdx.x >> 8;
    float (*tile)[65] = reinterpret_cast<float (*)[65]>(prep_smem) + sub * 64;
    const int q0 = blockIdx.y * 64, d0 = (blockIdx.x * PREP_TILES + sub) * 64;
    if ((int)blockIdx.x * PREP_TILES * 64 >= cols) return;   // (the whole workgroup)
    const float* __restrict__ W = jb.W;
    E* __restrict__ dst = static_cast<E*>(jb.dst);
    E* __restrict__ dstT = static_cast<E*>(jb.dstT);
    const int c4 = (tid & 15) * 4, r0 = tid >> 4;
#pragma unroll
    for (int r = r0; r < 64; r += 16) {
        const int q = q0 + r, d = d0 + c4;   // 4H is a multiple of 64: q is always a valid row
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
        if (d < cols) {
            v = *reinterpret_cast<const f32x4_t*>(W + ((size_t)(q & 3) * H + (q >> 2)) * cols + d);
            st4(dst + (size_t)q * cols + d, v[0], v[1], v[2], v[3]);
        }
        tile[r][c4] = v[0]; tile[r][c4 + 1] = v[1]; tile[r][c4 + 2] = v[2]; tile[r][c4 + 3] = v[3];
    }
    __syncthreads();
#pragma unroll
    for (int r = r0; r < 64; r += 16) {
        const int d = d0 + r, q = q0 + c4;
        if (d < cols) st4(dstT + (size_t)d * 4 * H + q, tile[c4][r], tile[c4 + 1][r], tile[c4 + 2][r], tile[c4 + 3][r]);
    }
}

// ---------------------------------------------------------------- heads
// head_out[p][a] = W_a[a] . h[p] + b_a[a];  value[p] = w_v . h[p] + b_v: a skinny fp32 GEMM (at most 64 columns)
// bound by reading h once.  One workgroup per 16 rows, fp32 MFMA 16x16x4 with the heads (action outputs, then the
// value) on the N dimension, 16 at a time; its four waves take a quarter of the contraction each (H is a multiple
// of 64) and the partial tiles are added in LDS in a fixed order: four times as many waves in flight as with one
// wave per block, which is what a latency-bound streaming read needs.
__global__ __launch_bounds__(256) void heads_fwd_kernel(const float* __restrict__ h, int M, int H, int A,
                                                        const float* __restrict__ W_a, const float* __restrict__ b_a,
                                                        const float* __restrict__ w_v, const float* __restrict__ b_v,
                                                        float* __restrict__ head_out, float* __restrict__ value) {
    __shared__ f32x4_t s_part[3][64];
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4, wave = threadIdx.x >> 6;
    const int p0 = blockIdx.x * 16;
    const bool row_ok = p0 + lr < M;
    const int kq = H / 4;   // this wave's share of the contraction: [wave * kq, (wave + 1) * kq)
    const float* hrow = h + (size_t)(row_ok ? p0 + lr : p0) * H + wave * kq + lk * 4;
    for (int ht = 0; ht * 16 <= A; ++ht) {
        const int hd = ht * 16 + lr;   // this lane's head as B operand
        const float* wrow = (hd < A ? W_a + (size_t)hd * H : w_v) + wave * kq + lk * 4;
        const bool head_ok = hd <= A;
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int k0 = 0; k0 < kq; k0 += 16) {
            f32x4_t av = *reinterpret_cast<const f32x4_t*>(hrow + k0);
            f32x4_t wv = *reinterpret_cast<const f32x4_t*>(wrow + k0);
            if (!row_ok) av = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (!head_ok) wv = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = mfma_f32_16x16x4(av[e], wv[e], acc);
        }
        __syncthreads();   // s_part may still be read from the previous head tile
        if (wave > 0) s_part[wave - 1][lane] = acc;
        __syncthreads();
        if (wave > 0) continue;
#pragma unroll
        for (int w = 0; w < 3; ++w) {
            const f32x4_t o = s_part[w][lane];
            acc[0] += o[0]; acc[1] += o[1]; acc[2] += o[2]; acc[3] += o[3];
        }
        // element r of the lane: row lk*4 + r, head ht*16 + lr
        if (head_ok) {
            const float bias = hd < A ? b_a[hd] : b_v[0];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int p = p0 + lk * 4 + r;
                if (p >= M) continue;
                if (hd < A) head_out[(size_t)p * A + hd] = acc[r] + bias;
                else value[p] = acc[r] + bias;
            }
        }
    }
}

// The heads' part of the backward pass, one launch (nothing in it depends on anything else in it); blockIdx.x says which:
//  * dh[p][j] = sum_a d_u[p][a] W_a[a][j] + d_v[p] w_v[j].  A thread owns 4 adjacent columns (16-byte stores; H is a
//    multiple of 64) for a block of HB_ROWS rows, so a head weight is read once per block instead of once per row.  Bound by
//    writing dh once.  These blocks also clear the synchronisation words of the time loop that follows.
//  * The weight gradients' partial sums over blocks of HW_ROWS rows: part[rb][a][j] = sum_{p in block rb} du(p,a) h[p][j], a =
//    0..A (A = value head), and the same of the bias gradients.  A wave takes 64 columns and the block's rows on fp32 MFMAs,
//    heads on M (16 at a time), rows on K: 4 rows and 64 columns (16 bytes per lane) per load of h, all loads of a wave in
//    flight at once.  Bound by reading h once.  (A thread per 4 columns walking over the rows four at a time, eight
//    dependent rounds: 11 us where this takes 4, on 59 rows as on 1000.)
// (The fp32 rows of a bf16 call, which the first layer's weight gradient reads, are still there in the operand type from the
// forward call: converted here again they took 34 us for 32768 rows of 1044, and 35 more in the time loop behind, 64 units.)
constexpr int HB_ROWS = 8, HW_ROWS = 32;
struct HeadsBwdArgs {
    const float* d_u; const float* d_v; const float* W_a; const float* w_v; const float* h;
    float* dh; float* part; float* part_b;
    int32_t* clear;
    int M, H, A, n_clear;
    int dh_blocks;           // blockIdx.x below dh_blocks: dh; then weight-gradient blocks
};
__device__ __forceinline__ void heads_dh_block(const HeadsBwdArgs& a, int block) {
    __shared__ float s_g[HB_ROWS][64];   // the block's loss gradients: heads 0..A-1, then the value head
    const int M = a.M, H = a.H, A = a.A;
    const int j = threadIdx.x * 4;   // (H <= 1024)
    const int p0 = block * HB_ROWS;
    for (int i = block * 256 + threadIdx.x; i < a.n_clear; i += a.dh_blocks * 256) a.clear[i] = 0;
    for (int i = threadIdx.x; i < HB_ROWS * 64; i += 256) {
        const int r = i >> 6, e = i & 63, p = p0 + r;
        s_g[r][e] = (p < M) ? (e < A ? a.d_u[(size_t)p * A + e] : (e == A ? a.d_v[p] : 0.f)) : 0.f;
    }
    __syncthreads();
    if (j >= H) return;
    f32x4_t s[HB_ROWS];
    const f32x4_t wv = *reinterpret_cast<const f32x4_t*>(a.w_v + j);
#pragma unroll
    for (int r = 0; r < HB_ROWS; ++r) {
        const float g = s_g[r][A];
        s[r] = f32x4_t{g * wv[0], g * wv[1], g * wv[2], g * wv[3]};
    }
#pragma unroll 4
    for (int e = 0; e < A; ++e) {
        const f32x4_t w = *reinterpret_cast<const f32x4_t*>(a.W_a + (size_t)e * H + j);
#pragma unroll
        for (int r = 0; r < HB_ROWS; ++r) {
            const float g = s_g[r][e];   // same address in every lane: a broadcast read
            s[r][0] += g * w[0]; s[r][1] += g * w[1]; s[r][2] += g * w[2]; s[r][3] += g * w[3];
        }
    }
#pragma unroll
    for (int r = 0; r < HB_ROWS; ++r)
        if (p0 + r < M) *reinterpret_cast<f32x4_t*>(a.dh + (size_t)(p0 + r) * H + j) = s[r];
}
__device__ __forceinline__ void heads_wgrad_block(const HeadsBwdArgs& a, int block) {
    const int M = a.M, H = a.H, A = a.A, groups = H / 64;   // groups of 64 columns
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    const int unit = block * 4 + (threadIdx.x >> 6), rb = unit / groups, j = unit % groups * 64 + lr * 4;
    const int p0 = rb * HW_ROWS + lk;   // this lane's rows: p0 + 4 s
    if (rb * HW_ROWS >= M) return;
    constexpr int STEPS = HW_ROWS / 4;
    f32x4_t hv[STEPS];
#pragma unroll
    for (int k = 0; k < STEPS; ++k) hv[k] = *reinterpret_cast<const f32x4_t*>(a.h + (size_t)min(p0 + 4 * k, M - 1) * H + j);
    for (int a0 = 0; a0 <= A; a0 += 16) {
        const int e = a0 + lr;   // this lane's head
        float g[STEPS], sum = 0.f;
#pragma unroll
        for (int k = 0; k < STEPS; ++k) {
            const int p = min(p0 + 4 * k, M - 1);
            const float* src = e < A ? a.d_u + (size_t)p * A + e : a.d_v + p;
            g[k] = *src;
        }
        f32x4_t acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < STEPS; ++k) {
            const bool in = e <= A && p0 + 4 * k < M;
            const float gk = in ? g[k] : 0.f;
            sum += gk;
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = mfma_f32_16x16x4(gk, p0 + 4 * k < M ? hv[k][t] : 0.f, acc[t]);
        }
        // element r of lane l: head a0 + lk * 4 + r, columns j .. j + 3 (one of each of the four products)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = a0 + lk * 4 + r;
            if (o <= A) *reinterpret_cast<f32x4_t*>(a.part + ((size_t)rb * (A + 1) + o) * H + j) = f32x4_t{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
        }
        if (unit % groups == 0) {   // bias gradients: the four lanes of a head together
            sum += __shfl_xor(sum, 16, VER_WAVE);
            sum += __shfl_xor(sum, 32, VER_WAVE);
            if (lk == 0 && e <= A) a.part_b[(size_t)rb * 64 + e] = sum;
        }
    }
}
__global__ __launch_bounds__(256) void heads_bwd_kernel(HeadsBwdArgs a) {
    if ((int)blockIdx.x < a.dh_blocks) heads_dh_block(a, blockIdx.x);
    else heads_wgrad_block(a, blockIdx.x - a.dh_blocks);
}
// One workgroup adds the row blocks' partial sums for 64 columns of one head: its four waves take a quarter of the
// row blocks each (in index order, 8 loads in flight), and the four shares are added in wave order.
constexpr int HF_COLS = 64;
struct HeadsFinalArgs {
    const float* part; const float* part_b;
    float* dW_a; float* dw_v; float* db_a; float* db_v;
    int n_rb, H, A;
};
__device__ __forceinline__ void heads_final_block(const HeadsFinalArgs& q, int bx, int a) {
    __shared__ float red[256];
    const int lane = threadIdx.x & 63, share = threadIdx.x >> 6, n_rb = q.n_rb, H = q.H, A = q.A;
    const int j = bx * HF_COLS + lane;
    const int per = (n_rb + 3) / 4, rb_end = min(n_rb, (share + 1) * per);
    float s = 0.f;
    int rb = share * per;
    if (j < H) {
        for (; rb + 8 <= rb_end; rb += 8) {   // 8 loads in flight, added in index order
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = q.part[((size_t)(rb + u) * (A + 1) + a) * H + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; rb < rb_end; ++rb) s += q.part[((size_t)rb * (A + 1) + a) * H + j];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (share == 0 && j < H) {
        s = ((red[lane] + red[64 + lane]) + red[128 + lane]) + red[192 + lane];
        if (a < A) q.dW_a[(size_t)a * H + j] = s; else q.dw_v[j] = s;
    }
    if (bx != 0) return;
    float sb = 0.f;
    for (int i = threadIdx.x; i < n_rb; i += 256) sb += q.part_b[(size_t)i * 64 + a];
    __syncthreads();
    red[threadIdx.x] = sb;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (a < A) q.db_a[a] = red[0]; else q.db_v[0] = red[0];
    }
}

// The bias gradients of a layer (sets = 1) or of the two or three layers of a launch: out[(c % 4) * H + c / 4] (and out2) = sum over the n_rb
// rows of part[n_rb][4H], in row order (deterministic); the next set's sums follow at part_stride.
struct BiasFinalArgs {
    const float* part; size_t part_stride;
    float* out[3]; float* out2[3];
    int n_rb, H, sets;
    const int* groups;   // groups of the time loops: of the first two sets, of the third (NULL: n_rb)
};
__device__ __forceinline__ void bias_final_block(const BiasFinalArgs& q, int bx, int set) {
    const int n_rb = q.groups ? q.groups[set / 2] : q.n_rb;
    const int c = bx * 256 + threadIdx.x, cols = 4 * q.H;
    if (c >= cols) return;
    const float* part = q.part + set * q.part_stride;
    float s = 0.f;
    int rb = 0;
    for (; rb + 8 <= n_rb; rb += 8) {   // 8 loads in flight, added in index order
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(rb + u) * cols + c];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; rb < n_rb; ++rb) s += part[(size_t)rb * cols + c];
    const int dst = (c & 3) * q.H + (c >> 2);
    (set == 2 ? q.out[2] : set == 1 ? q.out[1] : q.out[0])[dst] = s;
    (set == 2 ? q.out2[2] : set == 1 ? q.out2[1] : q.out2[0])[dst] = s;
}
// Both in one launch behind the first time loop of the backward pass (blockIdx.y: the bias sets, then the heads).
__global__ __launch_bounds__(256) void grads_final_kernel(BiasFinalArgs b, HeadsFinalArgs h) {
    if ((int)blockIdx.y < b.sets) bias_final_block(b, blockIdx.x, blockIdx.y);
    else if ((int)blockIdx.x * HF_COLS < h.H) heads_final_block(h, blockIdx.x, blockIdx.y - b.sets);
}

// ---------------------------------------------------------------- workspace
constexpr int REC_FLAG_WORDS = 8 * REC_MAX_GROUP + 64;   // flags[group][32], then one ticket per group

struct LayerWs {
    void* wih;    // [4H, D_l]  operand type, interleaved rows
    void* wihT;   // [D_l, 4H]
    void* whh;    // [4H, H]
    void* whhT;   // [H, 4H]
    float* bias;  // [4H]
    float* gates; // [M, 4H]
    float* c;     // [M, H]
    float* hout;  // [M, H]
    void* hprev;  // [M, H] operand type
    void* hcopy;  // [M, H] operand type: h_t, for what contracts it: the layer above, in a two-layer launch its workers (fp32: hout itself)
};
struct LstmWs {
    int* err;          // word 0 of the workspace
    int* flags;        // [REC_FLAG_WORDS]: per-workgroup flags of a recurrent launch, then its ticket counters
    int* flags_alone[2];   // [REC_FLAG_WORDS]: the same for a second and third launch behind the same clearing (may_run_alone)
    long long* prof;   // [128] phase counters of the recurrent kernels (forward 0..15, backward 16..31; +32: consumer layer), timeline, workers
    LayerWs layer[8];
    void* dz[3];       // [M, 4H] operand type; as many as layers share a launch
    int* pipe;         // hand-over words of a launch of several layers: progress[8], done[][] from [16]; three layers: twice
    int pipe_words;
    int* plan[2];      // which pieces every group of such a launch runs, and its chunks (lstm_pipe.h): forward, backward
    float* plan_scratch;
    float* dh[3];      // [M, H] in turn: gradient arriving at a layer's h (the third with three layers only)
    float* dh_state;   // [M, H]
    float* dc_state;   // [M, H]
    float* part;       // partial sums of the two-stage reductions
    float* part_b;     // [row blocks][64]: the heads' bias gradients per row block
    float* gemm_part;  // partial results of split contractions
    bf16_t* x_op;      // [M, input_dim]: fp32 input rows of a bf16 call in the operand type
    char* ring;        // [8 groups] exchange rings of the time loops (lstm_few.h)
    char* ring_many;   // [8 groups] the same for more than 16 pieces (lstm_many.h)
    float* db_part;    // [2 or 3][8][4H]: per layer of a launch and group, the sum of the gate gradients over the group's rows
    size_t bytes;
};

inline size_t part_floats(const ver_lstm_cfg& c, int M) {
    const size_t rb_heads = (size_t)(M + HW_ROWS - 1) / HW_ROWS;
    return rb_heads * (c.act_dim + 1) * c.hidden;   // the row-block partial sums of the heads' weight gradient
}

// Largest scratch that any contraction of the forward or backward pass asks for: partial results of a contraction that is split.
inline size_t gemm_part_max(const ver_lstm_cfg& c, int M) {
    const int bk = c.compute ? GemmGeom<MODE_BF16>::BK : GemmGeom<MODE_F32>::BK, H4 = 4 * c.hidden;
    const GemmGroup rows(false, c.compute != 0), dw(true, c.compute != 0);
    size_t m = 0;
    for (int l = 0; l < c.n_layers; ++l) {
        const int D = l == 0 ? c.input_dim : c.hidden;
        if (!c.compute) m = std::max({m, GemmGroup::row_part_floats(M, H4, D), GemmGroup::row_part_floats(M, D, H4)});
        if (!rows.fits(D, D, H4, M, H4, D)) m = std::max(m, gemm_part_floats(M, H4, D, bk));
        if (!rows.fits(H4, H4, D, M, D, H4)) m = std::max(m, gemm_part_floats(M, D, H4, bk));
        for (int n : {D, c.hidden})
            if (!dw.fits(H4, n, n, H4, n, M)) m = std::max(m, gemm_part_floats(H4, n, M, bk));
    }
    if (c.compute) m = std::max(m, GemmGroup::part_floats((size_t)H4 * (std::max(c.input_dim, c.hidden) + (size_t)c.hidden * (c.n_layers >= 2 ? 3 : 1)), M));   // (a launch takes up to two layers' weight gradients)
    return m;
}

// How the backward time loops split a width over a workgroup's waves: one wave per (16 units, share of the 4H contraction): 2 tiles x 4
// when H / 16 > 32 workgroups, else 1 x 8.
struct BwdSplit {
    bool wide;
    int mt, ks, ni;   // tiles, shares, operand blocks of a share
};
inline BwdSplit bwd_split(int mode, int H) {
    const bool wide = H / 16 > REC_MAX_GROUP;
    const int ks = wide ? 4 : 8, kblk = mode == MODE_BF16 ? RecGeom<MODE_BF16>::KBLK : RecGeom<MODE_F32>::KBLK;
    return BwdSplit{wide, wide ? 2 : 1, ks, 4 * H / ks / kblk};
}
inline int many_rows_bwd_of(int mode, int H, int M) {
    const BwdSplit b = bwd_split(mode, H);
    return many_rows_bwd(mode, H, b.mt, b.ni, M);
}

inline void lstm_ws_layout(const ver_lstm_cfg& c, int M, void* base, LstmWs* ws) {
    const size_t es = c.compute ? 2 : 4;
    const size_t H = c.hidden, Mz = (size_t)M;
    Carver cv(base);
    int* head = cv.take<int>(64);
    ws->err = head;
    ws->flags = cv.take<int>(REC_FLAG_WORDS);
    for (int*& f : ws->flags_alone) f = cv.take<int>(REC_FLAG_WORDS);
    const bool three = c.n_layers == 3;   // (three_layers, which may be switched off between the calls)
    ws->prof = cv.take<long long>(128);
    // the hand-over words sit right behind, so that one fill clears everything a launch needs cleared
    ws->pipe_words = pipe_sync_words(M) * (three ? 2 : 1);
    ws->pipe = cv.take<int>(ws->pipe_words);
    ws->plan[0] = cv.take<int>(PLAN_WORDS);
    ws->plan[1] = cv.take<int>(PLAN_WORDS);
    ws->plan_scratch = cv.take<float>(plan_scratch_floats(M));
    for (int l = 0; l < c.n_layers; ++l) {
        const size_t D = l == 0 ? c.input_dim : H;
        LayerWs& L = ws->layer[l];
        L.wih = cv.take<char>(4 * H * D * es);
        L.wihT = cv.take<char>(4 * H * D * es);
        L.whh = cv.take<char>(4 * H * H * es);
        L.whhT = cv.take<char>(4 * H * H * es);
        L.bias = cv.take<float>(4 * H);
        L.gates = cv.take<float>(Mz * 4 * H);
        L.c = cv.take<float>(Mz * H);
        L.hout = cv.take<float>(Mz * H);
        L.hprev = cv.take<char>(Mz * H * es);
        L.hcopy = l + 1 == c.n_layers ? nullptr : (c.compute ? static_cast<void*>(cv.take<char>(Mz * H * es)) : L.hout);
    }
    ws->dz[0] = cv.take<char>(Mz * 4 * H * es);
    ws->dz[1] = c.n_layers >= 2 ? cv.take<char>(Mz * 4 * H * es) : ws->dz[0];
    ws->dz[2] = three ? cv.take<char>(Mz * 4 * H * es) : ws->dz[0];
    ws->dh[0] = cv.take<float>(Mz * H);
    ws->dh[1] = cv.take<float>(Mz * H);
    ws->dh[2] = three ? cv.take<float>(Mz * H) : nullptr;
    ws->dh_state = cv.take<float>((three ? 3 : 2) * Mz * H);
    ws->dc_state = cv.take<float>((three ? 3 : 2) * Mz * H);
    ws->part = cv.take<float>(part_floats(c, M));
    ws->part_b = cv.take<float>((size_t)(M + HW_ROWS - 1) / HW_ROWS * 64);
    ws->gemm_part = cv.take<float>(gemm_part_max(c, M));
    ws->x_op = c.compute && !c.x_bf16 ? cv.take<bf16_t>(Mz * c.input_dim) : nullptr;
    ws->db_part = cv.take<float>((size_t)(three ? 3 : 2) * REC_GROUPS * 4 * H);
    const int mode = c.compute ? MODE_BF16 : MODE_F32;
    ws->ring = cv.take<char>(REC_GROUPS * few_ring_bytes(mode, 4 * c.hidden));
    ws->ring_many = cv.take<char>(REC_GROUPS * std::max(many_ring_bytes(mode, c.hidden, many_rows(mode, c.hidden, M)),
                                                        many_ring_bytes(mode, 4 * c.hidden, many_rows_bwd_of(mode, c.hidden, M))));
    ws->bytes = cv.used;
}

inline int check_cfg(const ver_lstm_cfg* c, int M) {
    if (!c || M <= 0) return VER_EINVAL;
    if (c->compute != 0 && c->compute != 1) return VER_EINVAL;
    if (c->layer_by_layer != 0 && c->layer_by_layer != 1) return VER_EINVAL;
    if (c->x_bf16 && !c->compute) return VER_EINVAL;
    if (c->n_layers < 1 || c->n_layers > 8 || c->act_dim < 1 || c->act_dim > 63) return VER_EUNSUPPORTED;
    if (c->hidden < 64 || c->hidden % 64 != 0 || c->input_dim < 4 || c->input_dim % 4 != 0) return VER_EUNSUPPORTED;
    // a wave keeps its [16, H] share of W_hh in 128 registers; a 16-row tile of dz ([16, 4H]) must fit in LDS
    if (c->hidden > (c->compute ? 1024 : 512)) return VER_EUNSUPPORTED;
    // the time-loop kernels address the rows of an activation array with 32-bit byte offsets
    if ((long long)M * 16 * c->hidden >= (1LL << 31)) return VER_EUNSUPPORTED;
    return VER_OK;
}

// How many 16-row tiles of exchanged rows fit in a CU's 160 KB of LDS next to the reduction buffer.
inline int rec_tiles(size_t tile_bytes, size_t red_bytes_per_tile) {
    int n = (int)((160 * 1024) / (tile_bytes + red_bytes_per_tile));
    return n < 1 ? 1 : (n > REC_NTC ? REC_NTC : n);
}

// C[M, N] = A[M, K] B[N, K]^T (+ bias), all three row-major, A and B in the operand type.  bf16 in 64 x 64 tiles while those
// are at most four per CU (us, 64 x 64 and 128 x 256 tiles: 1024 tiles, 1000 x 4096 x 1044 28 and 28, 2048 x 2048 x 516 15.4 and
// 16.5; 940, 3001 x 1280 x 320 9.0 and 12; 235, 3001 x 320 x 1280 8.8 and 21; 4096, 8192 x 4096 x 1044 210 and 114); where one column of
// 128 x 256 tiles covers the matrix, and so reads the rows once, at most TILES_64_NARROW of them (768 tiles, 12288 x 256 x 4096 57 and 62; 876, 14000 x
// 224 x 4096 65 and 61; 1024, 16384 x 256 x 4096 75 and 62, 32768 x 128 x 2048 47 and 37).  Beyond that one
// tile per CU at a time: 256 x 256 or 128 x 256, whichever's rounds take less; a round of the larger ones takes 1.6 times as long
// (45 and 28 us at K = 1044), and more where the contraction is short and the time that of the stores, with nothing beside them in
// a CU (8192 x 4096: K = 36 35 and 30, 192 41 and 36, 256 44 and 44; 32768 x 4096: 36 121 and 111, 260 194 and 218; 32768 x 1044: 256 72 and 50).  What lies beyond the 32-bit byte offsets of these kernels (only rows of the caller's can) goes
// to the general kernel.
constexpr int LARGE_FROM_K = 260, TILES_64_NARROW = 832;
template <int MODE>
inline int contract_rows(const typename RecGeom<MODE>::E* A, const typename RecGeom<MODE>::E* B, float* C, const float* bias, int M, int N, int K, float* part, hipStream_t s, const int* alone = nullptr) {
    GemmGroup g(false, MODE == MODE_BF16, part);
    g.a.alone = alone;
    if (!g.add(A, K, B, K, C, N, M, N, K, bias, 0)) {
        gemm_launch<MODE, false>(A, K, B, K, C, N, M, N, K, bias, 0, part, alone, s);
        return VER_OK;
    }
    if (MODE == MODE_BF16 && g.lay_out(64) > (N <= PIPE_BN ? TILES_64_NARROW : 4 * REC_GRID)) {
        auto rounds = [](int tiles) { return (tiles + REC_GRID - 1) / REC_GRID; };
        if (K >= LARGE_FROM_K && 8 * rounds(g.lay_out(GemmGroup::LARGE_TILE)) <= 5 * rounds(g.lay_out(PIPE_BM, PIPE_BN))) return g.launch_large(s) ? VER_OK : VER_EHIP;
        if (!set_lds(lstm_proj_dma_kernel, (size_t)PIPE_STAGES * PIPE_STAGE_BYTES)) return VER_EHIP;
        const ProjWork pw = {A, B, C, bias, K, N, M, alone};
        const int tiles_n = (N + PIPE_BN - 1) / PIPE_BN, tiles_m = (M + PIPE_BM - 1) / PIPE_BM;
        hipLaunchKernelGGL(lstm_proj_dma_kernel, dim3(tiles_m * tiles_n), dim3(REC_THREADS), (size_t)PIPE_STAGES * PIPE_STAGE_BYTES, s,
                           pw, tiles_n);
        return VER_OK;
    }
    g.launch(s);
    return VER_OK;
}

// The persistent time-loop kernels are written for the whole of one MI355X: a grid of one workgroup per CU that
// must be co-resident, grouped by the XCD it runs on (8 XCDs of 32 CUs).  On any other device (another
// architecture, a partition of the chip with fewer CUs) their groups would be incomplete and the bounded waits
// would give up, so the entry points refuse to launch there.  Looked up once per device.
inline int device_fits_time_loops() {
    static std::mutex lock;
    static signed char known[64];   // 0 unknown, 1 fits, -1 does not
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return VER_EHIP;
    if (dev < 0 || dev >= 64) return VER_EUNSUPPORTED;
    std::lock_guard<std::mutex> hold(lock);
    if (known[dev] == 0) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return VER_EHIP;
        const bool ok = prop.multiProcessorCount == REC_GRID && std::strncmp(prop.gcnArchName, "gfx950", 6) == 0;
        known[dev] = ok ? 1 : -1;
    }
    return known[dev] > 0 ? VER_OK : VER_EUNSUPPORTED;
}

// stage: 1 for the second of the two products of a three-layer launch.
inline void pipe_work(const LstmWs& ws, int dir, int M, const int32_t* t_off, const int* alone, PipeWork* pw, int count = WORK_COUNT, int stage = 0) {
    pw->M = M;
    pw->count = count;
    pw->t_off = t_off;
    pw->plan = ws.plan[dir];
    pw->sync = ws.pipe + stage * pipe_sync_words(M);
    pw->err = ws.err;
    pw->alone = alone;
}

// Networks of several layers run two layers at a time in one launch each (lstm_pipe.h), the layers numbered 2i and 2i + 1;
// the top layer of an odd number from five on has a launch of its own.  A pair's time loops advance side by side on three XCDs each,
// where one after the other would have all eight: us per forward and backward pass of two layers, a launch per layer
// -> one for both: 300 rows (longest piece 98) at 512 units 632 -> 357, 8192 (473) at 1024 4204 -> 2417; closest where
// hundreds of short pieces keep every XCD busy: 8192 rows in 538 pieces (86) at 320 units 1121 -> 1103.
inline bool pairs_of_layers(const ver_lstm_cfg& c) { return c.n_layers >= 2 && !c.layer_by_layer; }
// Three layers run in one launch, on two XCDs each and an XCD for each of the two products: one walk over the dependent timesteps instead of
// two.  us per forward and backward pass of 3001 rows in 30 to 36 pieces at 320 units (bf16), a pair and a top layer -> three: 1523 -> 1196
// (and 1680 to 2080 where timesteps of few pieces took longer).
inline bool three_layers(const ver_lstm_cfg& c) { return c.n_layers == 3 && !c.layer_by_layer; }
// From three layers on a shared launch is for minibatches of few alive pieces per timestep (rows / timesteps): many are bound by
// throughput, of which two or three XCDs per layer have less than eight for one layer after the other (and finding the cuts for
// thousands of pieces takes milliseconds).  Only the device knows the timesteps: the forms are launched one behind the other, and what the
// plan has not chosen does nothing (15 us in all for pairs); up to THREE_ROWS rows three layers are launched in the form of one launch alone, up
// to PAIRS_ROWS rows without the form of a launch per layer.
constexpr int PAIRS_ROWS = 768;
// The lines.  Three layers in a launch instead of a pair and a top layer, times of the one over the other, forward and backward pass of equally long
// pieces (those of different length favour the former, whose time follows the longest):
//   pieces (timesteps)     16 (8) 16 (96)  24 (16) 24 (32)  32 (16) 32 (96)  36 (8) 36 (32) 36 (96)  48 (32) 48 (96)  64 (8) 64 (96)
//   bf16, 64 units           0.84    0.67     0.84    0.80     0.83    0.69    0.84    0.86    0.92     0.87    0.92    0.81    0.64
//         256                0.94    0.70     0.99    0.88     0.99    0.74    0.85    0.89    0.94     0.89    0.93    0.84    0.71
//         320                0.98    0.71     1.05    0.92     1.08    0.81   (40:) 0.95    1.09    1.13
//         384                0.91    0.68     0.95    0.89     0.98    0.82    0.88    1.00    1.14     0.96    1.09    0.96    0.91
//         576                0.89    0.68     0.91    0.85     0.94    0.85    0.98    1.06    1.10     0.99    1.02    0.98    0.76
//         1024               0.88    0.68     0.87    0.82     0.90    0.84    0.85    1.03    1.07     0.93    0.96    0.93    0.88
//   fp32, 64 units           1.02    0.74     1.01    0.91     0.99    0.73    0.69    0.70    0.75     0.71    0.74    0.83    0.74
//         256                0.99    0.73     1.00    0.90     0.99    0.73    0.84    0.86    0.91     0.98    0.94    1.17    0.79
//         384                1.06    0.77     1.11    0.97     1.14    0.89    0.94    0.95    1.11     1.06    1.04    1.15    1.04
// What decides: whether the products' workers keep up, which are half as many as a pair's (above 256 units one team instead of two, at 320
// instead of three), and from 33 alive pieces on whether 16 pieces at a time, two groups' worth instead of a pair's three, cost more than the
// second walk.  (With what is launched and does nothing: 1.03 to 1.05 at fp32, 64 to 256 units, 24 and 32 pieces over 16 timesteps, and 0.97 to
// 0.98 as pairs.)
// Pairs instead of a launch per layer (of three layers): bf16, 320 units 35 (29) 423 / 440, 51 (59) 782 / 787, 70 (117) 1675 / 1642, 76 (27) 562 /
// 512, 104 (29) 763 / 607, 910 (36) 8807 / 3677; fp32, 256 units 44 (68) 1027 / 1106, 70 (117) 2197 / 2263, 76 (27) 733 / 651; from 384 units on,
// where the workers hold the weights twice at most, 512 units 20 (51) 866 / 931, 24 (21) 533 / 514, 28 (36) 791 / 792, 35 (29) 847 / 766, 44
// (68) 1808 / 1805, 51 (59) 1818 / 1693, 70 (117) 4177 / 3976.
inline int three_rows(const ver_lstm_cfg& c) { return c.hidden > 256 && (!c.compute || c.hidden == 320) ? (c.compute ? 128 : 64) : c.compute ? 512 : 128; }
inline bool may_run_alone(const ver_lstm_cfg& c, int M) { return c.n_layers > 2 && pairs_of_layers(c) && M > PAIRS_ROWS; }
// Three layers: whether other forms than that of one launch are launched.
inline bool may_be_pairs(const ver_lstm_cfg& c, int M) { return three_layers(c) && M > three_rows(c); }
inline void pair_lines(const ver_lstm_cfg& c, int M, PlanArgs* p) {
    const bool low = !c.compute && c.hidden > 320;
    p->base = low ? 12 : 45;
    p->per = low ? 2 : 4;
    p->most = !may_run_alone(c, M) ? 0 : low ? 60 : 80;
    p->three = !three_layers(c) ? 0 : may_be_pairs(c, M) ? 1 : 2;
    p->n2 = p->n3 = p->t2 = p->s2 = p->t3 = 0;
    if (c.hidden <= 256) {   // two teams of workers for each product, or more
        if (c.compute) {
            p->n1 = 64;
        } else {
            p->n1 = 16; p->n2 = 40; p->t2 = 40; p->n3 = 64; p->t3 = c.hidden <= 128 ? 20 : 40;
        }
    } else if (c.compute) {
        p->n1 = c.hidden == 320 ? 16 : 32; p->n2 = 32; p->t2 = 48;
    } else {
        p->n1 = 0; p->n2 = 32; p->t2 = 16; p->s2 = 3;
    }
}

// What the first launch of the forward pass does for the launches of several layers: zeroes the flags, ticket counters, hand-over words
// and the sticky time-out word at the start of the workspace, and writes the plans of both directions of the minibatch (the
// backward call runs on the packing of the forward call whose activations it finds in the workspace).
inline PlanArgs pipe_plan(const LstmWs& ws, int mode, bool wide, int G, int M, const int32_t* info, const int32_t* batch_sizes, const ver_lstm_cfg& c) {
    PlanArgs p{};
    p.info = info; p.batch_sizes = batch_sizes; p.M = M;
    p.plan_fwd = ws.plan[0]; p.plan_bwd = ws.plan[1]; p.scratch = ws.plan_scratch;
    p.clear = ws.err; p.n_clear = (int)(ws.pipe + ws.pipe_words - ws.err);
    p.fwd = plan_cost(mode, wide, true, G, WORK_COUNT);
    p.bwd = plan_cost(mode, wide, false, G, WORK_COUNT);
    p.fwd_three = plan_cost(mode, wide, true, G, TRIPLE_WORK_COUNT);
    p.bwd_three = plan_cost(mode, wide, false, G, TRIPLE_WORK_COUNT);
    p.rows = PAIRS_ROWS;
    pair_lines(c, M, &p);
    return p;
}

// The rows that layer l contracts, in the operand type.
template <int MODE>
inline const typename RecGeom<MODE>::E* layer_input(const ver_lstm_cfg& c, const LstmWs& ws, const void* x, int l) {
    typedef const typename RecGeom<MODE>::E* rows_t;
    if (l == 0) return ws.x_op ? reinterpret_cast<rows_t>(ws.x_op) : static_cast<rows_t>(x);
    return static_cast<rows_t>(ws.layer[l - 1].hcopy);
}

template <int MODE>
int run_fwd(const ver_lstm_cfg& c, const void* x, int M, const int32_t* info, const int32_t* batch_sizes,
            const int32_t* t_off, const float* h0, const float* c0, int seq_cap, const float* const* w,
            float* head_out, float* value, LstmWs& ws, hipStream_t s) {
    typedef typename RecGeom<MODE>::E E;
    const int H = c.hidden, A = c.act_dim;
    const bool pairs = pairs_of_layers(c);   // two layers' time loops in one launch

    // 8 waves = row groups x shares of the contraction (TPW tiles of 16 gate rows per wave): a workgroup owns
    // 8 tiles (32 units) when 32 workgroups need all of H/32 units each, else 4 tiles (16 units)
    const bool wide = H / 16 > REC_MAX_GROUP;
    // Shares of the contraction in timesteps with more than 16 alive pieces of a group: with 8 tiles per workgroup two (a
    // wave then reads 16 operand blocks per piece tile and the cell update adds two partial sums; four read less from LDS
    // but reduce more: H = 1024, one layer, 32 / 48 / 64 pieces 5.70 / 9.04 / 12.3 us per timestep with two, 5.83 / 9.41 / 12.5 with
    // four, the same below 24), with 4 tiles four (H = 512, one layer, 17 / 32 / 64 pieces 3.28 / 3.53 / 5.9 us with four, 3.35 /
    // 3.70 / 6.2 with two; H = 256 3.55 / 3.87 / 6.6 and 4.06 / 4.38 / 7.8).
    const bool quarter = MODE == MODE_F32 || (!wide && H % 128 == 0);   // a quarter of H is a whole number of operand blocks
    const int ks = quarter ? 4 : 2;
    const int mt = wide ? 8 : 4;
    const size_t tile = (size_t)16 * (H + RecGeom<MODE>::PAD) * sizeof(E);
    const size_t red_per_tile = (size_t)ks * mt * 64 * 16 + (size_t)16 * 4 * mt * sizeof(E);   // partial sums + new h
    const int ntc = rec_tiles(tile, red_per_tile);
    size_t lds = ntc * (tile + red_per_tile);
    const int few_nb = wide ? FewBlocks<MODE, true>::fwd : FewBlocks<MODE, false>::fwd;
    if (few_lds_bytes(16 * mt, few_nb) > lds) lds = few_lds_bytes(16 * mt, few_nb);
    if (many_lds_bytes(16 * mt, few_nb) > lds) lds = many_lds_bytes(16 * mt, few_nb);
    const size_t work_lds = work_lds_bytes(16 * mt, few_nb, work_bufs<MODE, true>());
    if (pairs && work_lds > lds) lds = work_lds;
    const int nb = (H / ks) / RecGeom<MODE>::KBLK;

    // operand-type copies of every layer's weights (and their transposes) and the summed biases: one launch
    auto prep_all = [&]() {
        ProfScope prof(VER_PROF_LSTM_PREP, s);
        PrepArgs pa{};
        int n = 0, max_cols = H;
        for (int l = 0; l < c.n_layers; ++l) {
            const int D = l == 0 ? c.input_dim : H;
            LayerWs& L = ws.layer[l];
            max_cols = D > max_cols ? D : max_cols;
            pa.job[n++] = PrepJob{w[4 * l], nullptr, L.wih, L.wihT, D, 0};
            pa.job[n++] = PrepJob{w[4 * l + 1], nullptr, L.whh, L.whhT, H, 0};
            pa.job[n++] = PrepJob{w[4 * l + 2], w[4 * l + 3], L.bias, nullptr, PREP_BIAS, 0};
        }
        // without a pair, also the time-out word and the flags of the first time loop (else: the plan clears them)
        if (!pairs) pa.job[n++] = PrepJob{nullptr, nullptr, ws.err, nullptr, PREP_CLEAR, (size_t)(ws.flags + REC_FLAG_WORDS - ws.err)};
        const unsigned threads = pairs ? PLAN_THREADS : 256, cols = threads / 4;   // columns of a workgroup's tiles
        const unsigned gx = (max_cols + cols - 1) / cols, gy = 4 * H / 64;
        size_t layers = 1;   // of the grid, for the last job
        if (ws.x_op) {
            const size_t quads = (size_t)M * c.input_dim / 4;
            pa.job[n++] = PrepJob{static_cast<const float*>(x), nullptr, ws.x_op, nullptr, PREP_ROWS, quads};
            const size_t wgs = std::min(PREP_ROWS_THREADS / threads, (quads + PREP_ROWS_QUADS * threads - 1) / (PREP_ROWS_QUADS * threads));
            layers = (wgs + gx * gy - 1) / (gx * gy);
        }
        pa.n = n;
        const PlanArgs plan = pairs ? pipe_plan(ws, MODE, wide, H / (4 * mt), M, info, batch_sizes, c) : PlanArgs{};
        auto launch = [&](auto kernel) {
            if (!set_lds(kernel, prep_lds_bytes(threads))) return false;
            hipLaunchKernelGGL(kernel, dim3(gx, gy, n - 1 + (unsigned)layers + (pairs ? 1 : 0)), dim3(threads), prep_lds_bytes(threads), s, pa, H, plan);
            return true;
        };
        return pairs ? launch(prep_weights_kernel<E, PLAN_THREADS>) : launch(prep_weights_kernel<E, 256>);
    };
    // time-batched input projection: gates[M, 4H] = x W_ih^T + (b_ih + b_hh), interleaved columns
    auto project = [&](int l, const int* alone = nullptr) {
        const int D = l == 0 ? c.input_dim : H;
        LayerWs& L = ws.layer[l];
        ProfScope prof(VER_PROF_LSTM_GEMM_FWD, s);
        return contract_rows<MODE>(layer_input<MODE>(c, ws, x, l), static_cast<const E*>(L.wih), L.gates, L.bias, M, 4 * H, D, ws.gemm_part, s, alone) == VER_OK;
    };
    auto rec_args = [&](int l, int groups_before = 0) {   // (of the layers before in the same launch)
        LayerWs& L = ws.layer[l];
        RecFwdArgs ra;
        ra.info = info; ra.batch_sizes = batch_sizes; ra.t_off = t_off;
        ra.gates = L.gates; ra.c = L.c; ra.hout = L.hout; ra.hprev = L.hprev; ra.hcopy = L.hcopy; ra.whh = L.whh;
        ra.ring = ws.ring + groups_before * few_ring_bytes(MODE, H);
        ra.many_rows = many_rows(MODE, H, M);
        ra.ring_many = ws.ring_many + groups_before * many_ring_bytes(MODE, H, ra.many_rows);
        ra.h0 = h0 ? h0 + (size_t)l * seq_cap * H : nullptr;
        ra.c0 = c0 ? c0 + (size_t)l * seq_cap * H : nullptr;
        ra.H = H; ra.seq_cap = seq_cap; ra.M = M; ra.flags = ws.flags; ra.ticket = ws.flags + 8 * REC_MAX_GROUP;
        ra.err = ws.err; ra.prof = ws.prof + (groups_before ? 32 : 0); ra.prof_all = ws.prof;
        ra.G = H / (4 * mt); ra.ntc = ntc; ra.alone = nullptr;
        return ra;
    };
    const FwdForm form{wide, quarter, nb, lds};
    // The time loop of one layer in a launch of its own.
    auto loop_alone = [&](int l, int* flags, const int* alone) {
        RecFwdArgs ra = rec_args(l);
        ra.flags = flags; ra.ticket = flags + 8 * REC_MAX_GROUP; ra.alone = alone;
        ProfScope prof(VER_PROF_LSTM_REC_FWD, s);
        return launch_fwd_loop<MODE>(form, ra, s);
    };
    // bf16: what the layer above layer l contracts (a two-layer launch writes that of its lower layer itself)
    auto copy_h = [&](int l, const int* alone) {
        if constexpr (MODE == MODE_BF16) {
            const size_t quads = (size_t)M * H / 4;
            hipLaunchKernelGGL(convert_rows_kernel, dim3((unsigned)((quads + 1023) / 1024)), dim3(256), 0, s, ws.layer[l].hout,
                               static_cast<bf16_t*>(ws.layer[l].hcopy), quads, alone);
        }
    };
    // Layers l and l + 1 in a launch; not_chosen: points to anything but a zero if the plan has chosen another form (NULL: it always runs).
    auto pair = [&](int l, const int* not_chosen) {
        PipeFwdArgs pa;
        pa.l0 = rec_args(l);
        pa.l1 = rec_args(l + 1, PIPE_GROUPS);
        pa.work.A = ws.layer[l].hcopy; pa.work.B = ws.layer[l + 1].wih; pa.work.C = ws.layer[l + 1].gates;
        pa.work.bias = ws.layer[l + 1].bias; pa.work.K = H; pa.work.N = 4 * H;
        pipe_work(ws, 0, M, t_off, not_chosen, &pa.work);
        pa.work.G = pa.l0.G;
        ProfScope prof(VER_PROF_LSTM_REC_FWD, s);
        return launch_fwd_pair<MODE>(form, pa, not_chosen != nullptr, s);
    };
    if (!prep_all()) return VER_EHIP;
    const int* alone = may_run_alone(c, M) ? ws.plan[0] + PLAN_ALONE : nullptr;
    for (int l = 0; l < c.n_layers;) {
        if (!project(l)) return VER_EHIP;
        if (three_layers(c)) {
            if (may_be_pairs(c, M)) {   // the two lower layers one after the other or in a launch, then the top one; what does nothing leaves the words as they are
                const int* top = ws.plan[0] + PLAN_TOP;
                if (alone) {
                    if (!loop_alone(0, ws.flags, alone)) return VER_EHIP;
                    copy_h(0, alone);
                    if (!project(1, alone) || !loop_alone(1, ws.flags_alone[0], alone)) return VER_EHIP;
                }
                if (!pair(0, ws.plan[0] + PLAN_NO_PAIR)) return VER_EHIP;
                copy_h(1, top);
                if (!project(2, top) || !loop_alone(2, ws.flags_alone[1], top)) return VER_EHIP;
            }
            TripleFwdArgs ta;
            for (int k = 0; k < 3; ++k) ta.l[k] = rec_args(k, k * TRIPLE_GROUPS);
            for (int k = 0; k < 2; ++k) {
                ta.work[k].A = ws.layer[k].hcopy; ta.work[k].B = ws.layer[k + 1].wih; ta.work[k].C = ws.layer[k + 1].gates;
                ta.work[k].bias = ws.layer[k + 1].bias; ta.work[k].K = H; ta.work[k].N = 4 * H;
                pipe_work(ws, 0, M, t_off, ws.plan[0] + PLAN_NO_TRIPLE, &ta.work[k], TRIPLE_WORK_COUNT, k);
                ta.work[k].G = ta.l[0].G;
            }
            ProfScope prof(VER_PROF_LSTM_REC_FWD, s);
            if (!launch_fwd_triple<MODE>(form, ta, s)) return VER_EHIP;
            l = 3;
        } else if (pairs && l + 1 < c.n_layers) {
            // (the plan, of the packing, is the same for every pair)
            if (l > 0) fill_words(ws.flags, (size_t)(ws.pipe + ws.pipe_words - ws.flags), 0, s);
            if (alone) {   // the same two layers one after the other; where they do nothing they leave the words as they are
                if (!loop_alone(l, ws.flags, alone)) return VER_EHIP;
                copy_h(l, alone);
                if (!project(l + 1, alone) || !loop_alone(l + 1, ws.flags_alone[0], alone)) return VER_EHIP;
            }
            if (!pair(l, alone)) return VER_EHIP;
            l += 2;
        } else {
            if (l > 0) fill_words(ws.flags, REC_FLAG_WORDS, 0, s);
            if (!loop_alone(l, ws.flags, nullptr)) return VER_EHIP;
            l += 1;
        }
        if (l < c.n_layers) copy_h(l - 1, nullptr);
    }
    ProfScope prof(VER_PROF_HEADS_FWD, s);
    hipLaunchKernelGGL(heads_fwd_kernel, dim3((M + 15) / 16), dim3(256), 0, s, ws.layer[c.n_layers - 1].hout, M, H, A,
                       w[4 * c.n_layers], w[4 * c.n_layers + 1], w[4 * c.n_layers + 2], w[4 * c.n_layers + 3],
                       head_out, value);
    return launch_status();
}

template <int MODE>
int run_bwd(const ver_lstm_cfg& c, const void* x, int M, const int32_t* info, const int32_t* batch_sizes,
            const int32_t* t_off, const float* c0, int seq_cap, const float* const* w, const float* d_u,
            const float* d_v, float* const* gw, float* d_x, LstmWs& ws, hipStream_t s) {
    typedef typename RecGeom<MODE>::E E;
    const int H = c.hidden, A = c.act_dim, nl = c.n_layers;
    const float* h_top = ws.layer[nl - 1].hout;
    const bool pairs = pairs_of_layers(c), three = three_layers(c), top_pair = three || (pairs && nl % 2 == 0);   // several layers' time loops in one launch
    // heads
    {
    ProfScope prof(VER_PROF_HEADS_BWD, s);
    const int rb_h = (M + HW_ROWS - 1) / HW_ROWS;
    HeadsBwdArgs ha;
    ha.d_u = d_u; ha.d_v = d_v; ha.W_a = w[4 * nl]; ha.w_v = w[4 * nl + 2]; ha.h = h_top;
    ha.dh = ws.dh[0]; ha.part = ws.part; ha.part_b = ws.part_b;
    ha.M = M; ha.H = H; ha.A = A;
    ha.clear = ws.flags; ha.n_clear = top_pair ? (int)(ws.pipe + ws.pipe_words - ws.flags) : REC_FLAG_WORDS;
    ha.dh_blocks = (M + HB_ROWS - 1) / HB_ROWS;
    hipLaunchKernelGGL(heads_bwd_kernel, dim3(ha.dh_blocks + (rb_h * (H / 64) + 3) / 4), dim3(256), 0, s, ha);
    }
    HeadsFinalArgs hf{ws.part, ws.part_b, gw[4 * nl], gw[4 * nl + 2], gw[4 * nl + 1], gw[4 * nl + 3], (M + HW_ROWS - 1) / HW_ROWS, H, A};

    const BwdSplit split = bwd_split(MODE, H);
    const bool wide = split.wide;
    const int mt = split.mt, ks = split.ks, ni = split.ni;
    const size_t tile = (size_t)16 * (4 * H + RecGeom<MODE>::PAD) * sizeof(E);
    const size_t red_per_tile = (size_t)ks * mt * 64 * 16 + (size_t)16 * 16 * mt * sizeof(float);   // partial sums + carried dh
    const int ntc = rec_tiles(tile, red_per_tile);
    size_t lds = ntc * (tile + red_per_tile);
    const int few_nb = wide ? FewBlocks<MODE, true>::bwd : FewBlocks<MODE, false>::bwd;
    if (few_lds_bytes(16 * mt, few_nb) > lds) lds = few_lds_bytes(16 * mt, few_nb);
    const size_t work_lds = work_lds_bytes(16 * mt, few_nb, work_bufs<MODE, false>());
    if (pairs && work_lds > lds) lds = work_lds;

    // dz_of(l): layer l's gate gradients.  The two layers of a pair (l & 1: the upper one, which is the producer here) carry
    // their state in separate halves of the scratch, three layers in thirds; a top layer without a partner has an even number.
    auto half = [&](int l) { return three ? l : pairs ? l & 1 : 0; };
    auto dz_of = [&](int l) { return ws.dz[half(l)]; };
    auto rec_args = [&](int l, const float* dh_above, int groups_before = 0) {
        LayerWs& L = ws.layer[l];
        RecBwdArgs ra;
        ra.info = info; ra.batch_sizes = batch_sizes; ra.t_off = t_off;
        ra.gates = L.gates; ra.c = L.c; ra.c0 = c0 ? c0 + (size_t)l * seq_cap * H : nullptr;
        ra.dh_above = dh_above; ra.dz = dz_of(l); ra.whhT = L.whhT;
        ra.ring = ws.ring + groups_before * few_ring_bytes(MODE, 4 * H);
        ra.many_rows = many_rows_bwd_of(MODE, H, M);
        ra.ring_many = ws.ring_many + groups_before * many_ring_bytes(MODE, 4 * H, ra.many_rows);
        ra.dh_state = ws.dh_state + (size_t)half(l) * M * H;
        ra.dc_state = ws.dc_state + (size_t)half(l) * M * H;
        ra.db_part = ws.db_part + (size_t)half(l) * REC_GROUPS * 4 * H;
        ra.H = H; ra.seq_cap = seq_cap; ra.flags = ws.flags; ra.ticket = ws.flags + 8 * REC_MAX_GROUP;
        ra.err = ws.err; ra.prof = ws.prof + 16 + (groups_before ? 32 : 0); ra.prof_all = ws.prof;
        ra.G = H / (16 * mt); ra.ntc = ntc; ra.alone = nullptr;
        return ra;
    };
    bool ok = true;
    const BwdForm form{wide, ni, lds};
    auto loop_alone = [&](int l, const float* dh_above, int* flags, const int* alone) {
        RecBwdArgs ra = rec_args(l, dh_above);
        ra.flags = flags; ra.ticket = flags + 8 * REC_MAX_GROUP; ra.alone = alone;
        ProfScope prof(VER_PROF_LSTM_REC_BWD, s);
        return launch_bwd_loop<MODE>(form, ra, s);
    };
    // gradient w.r.t. the layer input: dx[M, D] = dz[M, 4H] . W_ih[4H, D]
    auto input_grad = [&](int l, float* dx, const int* alone) {
        ProfScope prof(VER_PROF_LSTM_GEMM_DX, s);
        ok = contract_rows<MODE>(static_cast<const E*>(dz_of(l)), static_cast<const E*>(ws.layer[l].wihT), dx, nullptr, M, l == 0 ? c.input_dim : H, 4 * H,
                                 ws.gemm_part, s, alone) == VER_OK;
    };
    const int* alone = may_run_alone(c, M) ? ws.plan[1] + PLAN_ALONE : nullptr;
    // Everything of layer l that is not the time loop: dx (optional), dW_ih, dW_hh, db.  The upper layers of a launch of `with` layers come
    // first and leave their weight gradients and bias sums to the launches of the lowest one (last).
    GemmGroup dw(true, MODE == MODE_BF16, ws.gemm_part);
    auto layer_grads = [&](int l, float* dx, int with, bool last) {
        const int D = l == 0 ? c.input_dim : H;
        LayerWs& L = ws.layer[l];
        const E* dz = static_cast<const E*>(dz_of(l));
        if (dx) input_grad(l, dx, nullptr);
        // dW_ih[4H, D] = dz^T x ; dW_hh[4H, H] = dz^T h_{t-1}; stored gate-major.  The contractions of a layer or pair leave in
        // one launch.
        {
        ProfScope prof(VER_PROF_LSTM_GEMM_DW, s);
        auto contract = [&](const E* B, float* C, int Nc) {
            if (!dw.add(dz, 4 * H, B, Nc, C, Nc, 4 * H, Nc, M, nullptr, H))
                gemm_launch<MODE, true>(dz, 4 * H, B, Nc, C, Nc, 4 * H, Nc, M, nullptr, H, ws.gemm_part, nullptr, s);
        };
        contract(layer_input<MODE>(c, ws, x, l), gw[4 * l], D);
        contract(static_cast<const E*>(L.hprev), gw[4 * l + 1], H);
        if ((last || dw.a.n == GEMM_GROUP_MAX) && (MODE == MODE_F32 || !launch_tn_group(dw, s))) dw.launch(s);
        }
        // db_ih = db_hh = column sums of dz: the time loop left one partial sum per group (a pair: both layers' sums in
        // one launch; the heads' gradients join the first)
        if (last) {
        ProfScope prof(VER_PROF_LSTM_DBIAS, s);
        float* const* g = gw + 4 * l;
        const int* groups = with > 1 && (alone || may_be_pairs(c, M)) ? ws.plan[1] + PLAN_GROUPS : nullptr;
        BiasFinalArgs bf{ws.db_part, (size_t)REC_GROUPS * 4 * H, {}, {}, with == 1 ? REC_GROUPS : with == 2 ? PIPE_GROUPS : TRIPLE_GROUPS, H, with, groups};
        for (int k = 0; k < with; ++k) { bf.out[k] = g[4 * k + 2]; bf.out2[k] = g[4 * k + 3]; }
        const bool heads = l + with == nl;
        hipLaunchKernelGGL(grads_final_kernel, dim3(std::max((4 * H + 255) / 256, (H + HF_COLS - 1) / HF_COLS), bf.sets + (heads ? A + 1 : 0)),
                           dim3(256), 0, s, bf, hf);
        }
    };

    // Layers l and l - 1 in a launch, with the gradients that arrive at their h (see the forward pass)
    auto pair = [&](int l, float* dh_above, float* dh_below, const int* not_chosen) {
        PipeBwdArgs pa;
        pa.l1 = rec_args(l, dh_above);
        pa.l0 = rec_args(l - 1, dh_below, PIPE_GROUPS);
        pa.work.A = dz_of(l); pa.work.B = ws.layer[l].wihT; pa.work.C = dh_below; pa.work.bias = nullptr;
        pa.work.K = 4 * H; pa.work.N = H;
        pipe_work(ws, 1, M, t_off, not_chosen, &pa.work);
        pa.work.G = pa.l1.G;
        ProfScope prof(VER_PROF_LSTM_REC_BWD, s);
        return launch_bwd_pair<MODE>(form, pa, not_chosen != nullptr, s);
    };

    int cur = 0;  // ws.dh[cur] holds the gradient arriving at the current layer's h
    for (int l = nl - 1; l >= 0;) {
        if (three) {
            if (may_be_pairs(c, M)) {   // (as in the forward pass)
                const int* top = ws.plan[1] + PLAN_TOP;
                if (!loop_alone(2, ws.dh[0], ws.flags_alone[1], top)) return VER_EHIP;
                input_grad(2, ws.dh[1], top);
                if (!ok) return VER_EHIP;
                if (alone) {
                    if (!loop_alone(1, ws.dh[1], ws.flags_alone[0], alone)) return VER_EHIP;
                    input_grad(1, ws.dh[2], alone);
                    if (!ok || !loop_alone(0, ws.dh[2], ws.flags, alone)) return VER_EHIP;
                }
                if (!pair(1, ws.dh[1], ws.dh[2], ws.plan[1] + PLAN_NO_PAIR)) return VER_EHIP;
            }
            TripleBwdArgs ta;
            for (int k = 0; k < 3; ++k) ta.l[k] = rec_args(2 - k, ws.dh[k], k * TRIPLE_GROUPS);
            for (int k = 0; k < 2; ++k) {
                ta.work[k].A = ws.dz[2 - k]; ta.work[k].B = ws.layer[2 - k].wihT; ta.work[k].C = ws.dh[k + 1]; ta.work[k].bias = nullptr;
                ta.work[k].K = 4 * H; ta.work[k].N = H;
                pipe_work(ws, 1, M, t_off, ws.plan[1] + PLAN_NO_TRIPLE, &ta.work[k], TRIPLE_WORK_COUNT, k);
                ta.work[k].G = ta.l[0].G;
            }
            {
            ProfScope prof(VER_PROF_LSTM_REC_BWD, s);
            if (!launch_bwd_triple<MODE>(form, ta, s)) return VER_EHIP;
            }
            layer_grads(2, nullptr, 3, false);
            layer_grads(1, nullptr, 3, false);
            layer_grads(0, d_x, 3, true);
            if (!ok) return VER_EHIP;
            l = -1;
        } else if (pairs && l % 2 == 1) {
            if (l != nl - 1) fill_words(ws.flags, (size_t)(ws.pipe + ws.pipe_words - ws.flags), 0, s);   // (the top layers': heads_bwd_kernel)
            if (alone) {   // (as in the forward pass)
                if (!loop_alone(l, ws.dh[cur], ws.flags, alone)) return VER_EHIP;
                input_grad(l, ws.dh[cur ^ 1], alone);
                if (!ok || !loop_alone(l - 1, ws.dh[cur ^ 1], ws.flags_alone[0], alone)) return VER_EHIP;
            }
            if (!pair(l, ws.dh[cur], ws.dh[cur ^ 1], alone)) return VER_EHIP;
            layer_grads(l, nullptr, 2, false);   // the weight gradients of both layers leave in one grouped launch
            layer_grads(l - 1, l > 1 ? ws.dh[cur] : d_x, 2, true);
            if (!ok) return VER_EHIP;
            l -= 2;
        } else {
            if (l != nl - 1) fill_words(ws.flags, REC_FLAG_WORDS, 0, s);
            if (!loop_alone(l, ws.dh[cur], ws.flags, nullptr)) return VER_EHIP;
            layer_grads(l, l > 0 ? ws.dh[cur ^ 1] : d_x, 1, true);
            if (!ok) return VER_EHIP;
            cur ^= 1;
            l -= 1;
        }
    }
    return launch_status();
}

}  // namespace
}  // namespace ver

extern "C" size_t ver_lstm_workspace_bytes(const ver_lstm_cfg* cfg, int32_t M) {
    if (ver::check_cfg(cfg, M) != VER_OK) return 0;
    ver::LstmWs ws;
    ver::lstm_ws_layout(*cfg, M, nullptr, &ws);
    return ws.bytes;
}

extern "C" int ver_lstm_fwd(const ver_lstm_cfg* cfg, const void* x_packed, int32_t M, const int32_t* info,
                            const int32_t* batch_sizes, const int32_t* t_off, const float* h0, const float* c0,
                            int32_t seq_cap, const float* const* weights, float* head_out, float* value,
                            void* workspace, size_t workspace_bytes, void* stream) {
    const int st = ver::check_cfg(cfg, M);
    if (st != VER_OK) return st;
    if (!x_packed || !info || !batch_sizes || !t_off || !weights || !head_out || !value) return VER_EINVAL;
    if ((h0 || c0) && seq_cap <= 0) return VER_EINVAL;
    for (int i = 0; i < 4 * cfg->n_layers + 4; ++i)
        if (!weights[i]) return VER_EINVAL;
    if (!workspace || workspace_bytes < ver_lstm_workspace_bytes(cfg, M)) return VER_EWORKSPACE;
    const int dev_st = ver::device_fits_time_loops();
    if (dev_st != VER_OK) return dev_st;
    ver::LstmWs ws;
    ver::lstm_ws_layout(*cfg, M, workspace, &ws);
    hipStream_t s = static_cast<hipStream_t>(stream);
    return cfg->compute ? ver::run_fwd<ver::MODE_BF16>(*cfg, x_packed, M, info, batch_sizes, t_off, h0, c0, seq_cap,
                                                       weights, head_out, value, ws, s)
                        : ver::run_fwd<ver::MODE_F32>(*cfg, x_packed, M, info, batch_sizes, t_off, h0, c0, seq_cap,
                                                      weights, head_out, value, ws, s);
}

extern "C" int ver_lstm_bwd(const ver_lstm_cfg* cfg, const void* x_packed, int32_t M, const int32_t* info,
                            const int32_t* batch_sizes, const int32_t* t_off, const float* h0, const float* c0,
                            int32_t seq_cap, const float* const* weights, const float* d_head_out,
                            const float* d_value, float* const* weight_grads, float* d_x, void* workspace,
                            size_t workspace_bytes, void* stream) {
    (void)h0;  // h_{t-1} of every row, including the initial state, was saved by the forward pass
    const int st = ver::check_cfg(cfg, M);
    if (st != VER_OK) return st;
    if (!x_packed || !info || !batch_sizes || !t_off || !weights || !d_head_out || !d_value || !weight_grads)
        return VER_EINVAL;
    if (c0 && seq_cap <= 0) return VER_EINVAL;
    for (int i = 0; i < 4 * cfg->n_layers + 4; ++i)
        if (!weights[i] || !weight_grads[i]) return VER_EINVAL;
    if (!workspace || workspace_bytes < ver_lstm_workspace_bytes(cfg, M)) return VER_EWORKSPACE;
    const int dev_st = ver::device_fits_time_loops();
    if (dev_st != VER_OK) return dev_st;
    ver::LstmWs ws;
    ver::lstm_ws_layout(*cfg, M, workspace, &ws);
    hipStream_t s = static_cast<hipStream_t>(stream);
    return cfg->compute ? ver::run_bwd<ver::MODE_BF16>(*cfg, x_packed, M, info, batch_sizes, t_off, c0, seq_cap,
                                                       weights, d_head_out, d_value, weight_grads, d_x, ws, s)
                        : ver::run_bwd<ver::MODE_F32>(*cfg, x_packed, M, info, batch_sizes, t_off, c0, seq_cap,
                                                      weights, d_head_out, d_value, weight_grads, d_x, ws, s);
}
