// bf16 contractions of the LSTM on v_mfma_f32_16x16x32_bf16 in 64 x 64 tiles, for the sizes whose larger tiles (lstm_proj_dma_kernel,
// the grouped kernels of gemm.h) would leave CUs idle.  gfx950 only.
//
// Same frame as gemm_f32.hip: K-tiles of 64 straight from global memory into LDS, two stages, one barrier per K-tile, the operands
// of the next K-tile read before the MFMAs of this one, several workgroups per CU.  A wave's 32 x 32 needs 4 KB of LDS reads for 64
// MFMA cycles, so a full chip is bound by LDS at half the MFMA rate; these launches are bound by the latency of their few
// K-tiles instead (K-minor ones, whose contraction runs over the rows of a minibatch, are split to that end: gemm_group.h).
// K-minor operands are read with the transposing LDS load (its lane layout: gemm.h).
#include "gemm_group.h"
#include "mfma.h"

namespace ver {
namespace {

constexpr int T = 64, BK = 64, WT = 2;                           // tile, K-tile, MFMA tiles per side of a wave's square
constexpr int OPERAND = T * BK * 2, STAGE = 2 * OPERAND, STAGES = 2;
constexpr int NL = OPERAND / 1024 / 4;                           // load instructions per wave, operand and stage
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef unsigned long long u64_t;

// Chunk (16 bytes) position p of LDS row r (128 bytes) holds chunk p ^ swz(r): 16 rows read at one chunk (K-major), or rows
// k .. k + 3 and k + 8 .. k + 11 at two neighbouring chunks (K-minor), touch every bank once.
template <bool KMIN> __device__ __forceinline__ int swz(int r) {
    return KMIN ? (r & 2) | ((r >> 1) & 4) : (r >> 1) & 7;
}

template <bool KMIN>
__device__ __forceinline__ void tile(const GemmProblem& q, int t, unsigned char* smem) {
#if defined(__HIP_DEVICE_COMPILE__)   // (the transposing-load builtin only exists in the device pass)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const int m0 = t / q.tiles_n * T, n0 = t % q.tiles_n * T;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int nk = (q.K + BK - 1) / BK;
    const int rowsA = KMIN ? q.K : q.Mr, rowsB = KMIN ? q.K : q.Nc;
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.A), 0, rowsA * q.lda * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.B), 0, rowsB * q.ldb * 2, 0x00020000);
    // a load instruction fills 8 rows of LDS (lane -> row lane / 8, position lane % 8); the swizzle is applied on the global side
    unsigned offA[NL], offB[NL];
    int kc[NL];   // K-major: this lane's first k in the K-tile
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const int row = (wave * NL + j) * 8 + (lane >> 3), c = (lane & 7) ^ swz<KMIN>(row);
        kc[j] = c * 8;
        if (KMIN) {   // rows beyond K are beyond the buffer and read zero; columns beyond the matrix feed outputs that are not stored
            offA[j] = ((unsigned)row * q.lda + m0 + c * 8) * 2;
            offB[j] = ((unsigned)row * q.ldb + n0 + c * 8) * 2;
        } else {      // rows beyond the matrix repeat its last one
            offA[j] = ((unsigned)min(m0 + row, q.Mr - 1) * q.lda + c * 8) * 2;
            offB[j] = ((unsigned)min(n0 + row, q.Nc - 1) * q.ldb + c * 8) * 2;
        }
    }
    auto issue = [&](int kt) {
        unsigned char* st = smem + kt % STAGES * STAGE + wave * NL * 1024;
        const unsigned stepA = KMIN ? (unsigned)(kt * BK) * q.lda * 2 : kt * BK * 2, stepB = KMIN ? (unsigned)(kt * BK) * q.ldb * 2 : kt * BK * 2;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const bool in = KMIN || kt * BK + kc[j] < q.K;   // (chunks beyond K: read zero)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_ptr_t)(st + j * 1024), 16, in ? offA[j] + stepA : 0xFFFFFFF0u, 0, 0, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (lds_ptr_t)(st + OPERAND + j * 1024), 16, in ? offB[j] + stepB : 0xFFFFFFF0u, 0, 0, 0);
        }
    };
    f32x4_t acc[WT][WT];
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    constexpr int STEPS = BK / 32;
    struct Operands { u16x8_t a[STEPS][WT], b[STEPS][WT]; };
    auto read_one = [&](const unsigned char* op, int ks, int first) -> u16x8_t {
        if constexpr (KMIN) {
            s16x4_t h[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const int k = ks * 32 + lk * 8 + (lr >> 2) + 4 * x, col = (first + 4 * (lr & 3)) * 2;
                h[x] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(op + k * 128 + (((col >> 4) ^ swz<KMIN>(k)) << 4) + (col & 8)));
            }
            return u16x8_t{(bf16_t)h[0][0], (bf16_t)h[0][1], (bf16_t)h[0][2], (bf16_t)h[0][3], (bf16_t)h[1][0], (bf16_t)h[1][1], (bf16_t)h[1][2], (bf16_t)h[1][3]};
        } else {
            const int r = first + lr;
            return *reinterpret_cast<const u16x8_t*>(op + r * 128 + (((ks * 4 + lk) ^ swz<KMIN>(r)) << 4));
        }
    };
    auto read = [&](int kt, Operands& o) {
        const unsigned char* st = smem + kt % STAGES * STAGE;
#pragma unroll
        for (int ks = 0; ks < STEPS; ++ks)
#pragma unroll
            for (int i = 0; i < WT; ++i) {
                o.a[ks][i] = read_one(st, ks, wm + i * 16);
                o.b[ks][i] = read_one(st + OPERAND, ks, wn + i * 16);
            }
    };
    auto multiply = [&](const Operands& o) {
#pragma unroll
        for (int ks = 0; ks < STEPS; ++ks)
#pragma unroll
            for (int i = 0; i < WT; ++i)
#pragma unroll
                for (int j = 0; j < WT; ++j) acc[i][j] = mfma_bf16_16x16x32(o.a[ks][i], o.b[ks][j], acc[i][j]);
    };
    // this wave's loads have landed, and after the barrier so have everyone's
    auto arrived = [&] {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        bar_lds();
    };
    // K-major with K not a multiple of 8: the chunk that straddles K also holds 4 elements of the next row, which a thread per
    // row of the last K-tile clears
    auto trim = [&] {
        if (KMIN || q.K % 8 == 0) return;
        const int row = tid & (T - 1), c = (q.K % BK) >> 3;
        if (tid < 2 * T)
            *reinterpret_cast<u64_t*>(smem + (nk - 1) % STAGES * STAGE + (tid / T) * OPERAND + row * 128 + ((c ^ swz<KMIN>(row)) << 4) + 8) = 0;
        bar_lds();
    };
    issue(0);
    if (nk > 1) {
        issue(1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NL) : "memory");
        bar_lds();
    } else {
        arrived();
        trim();
    }
    Operands even, odd;
    auto step = [&](int kt, const Operands& now, Operands& next) {
        arrived();   // (and everyone has read the stage of kt, which is the one that is filled again)
        if (kt + STAGES < nk) issue(kt + STAGES);
        if (kt + 2 == nk) trim();
        read(kt + 1, next);
        __builtin_amdgcn_sched_barrier(0);
        multiply(now);
        __builtin_amdgcn_sched_barrier(0);
    };
    read(0, even);
    int kt = 0;
    for (; kt + 2 < nk; kt += 2) {
        step(kt, even, odd);
        step(kt + 1, odd, even);
    }
    if (kt + 1 < nk) {
        step(kt, even, odd);
        multiply(odd);
    } else {
        multiply(even);
    }
    // element r of lane l: row lk * 4 + r, column lr of the MFMA tile; what lies outside the matrix is stored out of the
    // buffer's range, i.e. dropped.  (16-byte stores of a transposed product: 1 to 5 % slower.)
    const __amdgpu_buffer_rsrc_t rsC = __builtin_amdgcn_make_buffer_rsrc(q.C, 0, q.Mr * q.ldc * 4, 0x00020000);
#pragma unroll
    for (int j = 0; j < WT; ++j) {
        const int n = n0 + wn + j * 16 + lr;
        const float bv = q.bias && n < q.Nc ? q.bias[n] : 0.f;
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm + i * 16 + lk * 4 + r, out = q.unperm_h > 0 ? (m & 3) * q.unperm_h + (m >> 2) : m;
                const unsigned at = m < q.Mr && n < q.Nc ? ((unsigned)out * q.ldc + n) * 4 : 0xFFFFFFF0u;
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][r] + bv), rsC, at, 0, 0);
            }
    }
#endif
}

__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmGroupArgs g) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[STAGES * STAGE];
    const int t = group_tile(g.tiles);
    if (t < 0 || (g.alone && *g.alone == 0)) return;
    const GemmProblem q = group_problem(g, t);
    tile<false>(q, t - q.tile_first, smem);
}
__global__ __launch_bounds__(256) void gemm_bf16_k_minor_kernel(GemmGroupArgs g) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[STAGES * STAGE];
    const int all = group_tile(g.tiles * g.parts);
    if (all < 0) return;
    const int part = all / g.tiles, t = all - part * g.tiles;
    GemmProblem q = group_problem(g, t);
    if (g.parts > 1) {   // rows [part * k_part, ...) of both operands, into the part's own results
        const int k0 = part * g.k_part;
        q.A = static_cast<const bf16_t*>(q.A) + (size_t)k0 * q.lda;
        q.B = static_cast<const bf16_t*>(q.B) + (size_t)k0 * q.ldb;
        q.K = min(q.K - k0, g.k_part);
        q.C = q.part + (size_t)part * q.Mr * q.Nc;
        q.ldc = q.Nc;
        q.unperm_h = 0;
    }
    tile<true>(q, t - q.tile_first, smem);
}
// C = sum of the parts in index order (+ bias), 8 loads in flight; blockIdx.y: the problem.
__global__ __launch_bounds__(256) void gemm_add_parts_kernel(GemmGroupArgs g) {
    if (g.alone && *g.alone == 0) return;
    const GemmProblem& q = g.p[blockIdx.y];   // (uniform index into the kernel arguments: scalar loads)
    const unsigned total = (unsigned)q.Mr * q.Nc;
    for (unsigned i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
        float s = 0.f;
        int z = 0;
        for (; z + 8 <= g.parts; z += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = q.part[(size_t)(z + u) * total + i];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; z < g.parts; ++z) s += q.part[(size_t)z * total + i];
        const unsigned m = i / q.Nc, n = i - m * q.Nc, out = q.unperm_h > 0 ? (m & 3) * q.unperm_h + (m >> 2) : m;
        q.C[(size_t)out * q.ldc + n] = q.bias ? s + q.bias[n] : s;
    }
}

// ---- large K-major contractions: 256 x 256 tiles, 8 waves (2 x 4 of 128 x 64), one workgroup per CU ------------------------
// K-tiles of 64 in two stages of 64 KB, one barrier per K-tile (2048 MFMA cycles per SIMD).  A K-tile is multiplied in two halves
// of 32; the operands of a half are read between the MFMAs of the half before it, one read after two MFMAs: read in one go
// they hold the wave's MFMAs up while the LDS serves all eight waves at once (2 to 5 % slower).  1169 TFLOP/s on 8192 x 8192 x
// 8192 (the library 1132).  The projections have short contractions and write 4 bytes per 2 K flops: 8192 x 4096 x 1044 bf16 takes 91
// us, of which 27 are the 134 MB of results (after each round of tiles, with no MFMAs beside them), and rows of 1044 are not
// aligned to cache lines (83 us with 1088); 114 us with 128 x 256 tiles, 424 against 475 on 32768 rows.  Tried: K-tiles of 32 in four stages
// (64-byte row pieces: 101 us), 16-byte stores of a transposed product (97).
constexpr int LT = 256, L_THREADS = 512, L_OPERAND = LT * BK * 2, L_STAGE = 2 * L_OPERAND, L_NL = L_OPERAND / 1024 / 8, L_STAGES = 2;
__global__ __launch_bounds__(L_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_bf16_large_kernel(GemmGroupArgs g) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_l[];
    const int t = group_tile(g.tiles);
    if (t < 0 || (g.alone && *g.alone == 0)) return;
    const GemmProblem& q = g.p[0];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    // tiles in bands of 4 rows of tiles, column by column: the 32 workgroups of an XCD that run at a time share 4 rows and 8 columns
    const int band = t / (4 * q.tiles_n), rows_m = (q.Mr + LT - 1) / LT, in_band = min(4, rows_m - band * 4), rem = t - band * 4 * q.tiles_n;
    const int m0 = (band * 4 + rem % in_band) * LT, n0 = rem / in_band * LT;
    const int wm = (wave >> 2) * 128, wn = (wave & 3) * 64;
    const int nk = (q.K + BK - 1) / BK;
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.A), 0, q.Mr * q.lda * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.B), 0, q.Nc * q.ldb * 2, 0x00020000);
    // a load instruction fills 8 rows (lane -> row lane / 8, position lane % 8); rows beyond the matrix repeat its last one
    unsigned offA[L_NL], offB[L_NL];
    const int kc0 = ((lane & 7) ^ ((lane >> 4) & 3)) * 8;   // this lane's first k in the K-tile for even j; odd j: ^ 32 (the swizzle (row >> 1) & 7)
#pragma unroll
    for (int j = 0; j < L_NL; ++j) {
        const int row = (wave * L_NL + j) * 8 + (lane >> 3), kc = (j & 1) ? kc0 ^ 32 : kc0;
        offA[j] = ((unsigned)min(m0 + row, q.Mr - 1) * q.lda + kc) * 2;
        offB[j] = ((unsigned)min(n0 + row, q.Nc - 1) * q.ldb + kc) * 2;
    }
    auto issue = [&](int kt) {
        unsigned char* st = smem_l + (kt & 1) * L_STAGE + wave * L_NL * 1024;
        const bool in[2] = {kt * BK + kc0 < q.K, kt * BK + (kc0 ^ 32) < q.K};
#pragma unroll
        for (int j = 0; j < L_NL; ++j) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_ptr_t)(st + j * 1024), 16, in[j & 1] ? offA[j] + kt * (BK * 2) : 0xFFFFFFF0u, 0, 0, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (lds_ptr_t)(st + L_OPERAND + j * 1024), 16, in[j & 1] ? offB[j] + kt * (BK * 2) : 0xFFFFFFF0u, 0, 0, 0);
        }
    };
    f32x4_t acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    struct Operands { u16x8_t a[8], b[4]; };
    // row wm + i * 16 + lr: (row >> 1) & 7 = lr >> 1, the same for every i
    const int sw = lr >> 1, rowA = (wm + lr) * 128, rowB = L_OPERAND + (wn + lr) * 128;
    auto read = [&](int kt, int half, Operands& o) {
        const unsigned char* st = smem_l + (kt & 1) * L_STAGE + (((half * 4 + lk) ^ sw) << 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) o.b[j] = *reinterpret_cast<const u16x8_t*>(st + rowB + j * 2048);
#pragma unroll
        for (int i = 0; i < 8; ++i) o.a[i] = *reinterpret_cast<const u16x8_t*>(st + rowA + i * 2048);
    };
    auto multiply = [&](const Operands& o) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = mfma_bf16_16x16x32(o.a[i], o.b[j], acc[i][j]);
    };
    auto trim = [&] {   // (as above)
        if (q.K % 8 == 0) return;
        const int row = tid & (LT - 1), c = (q.K % BK) >> 3;
        *reinterpret_cast<u64_t*>(smem_l + (nk - 1) % L_STAGES * L_STAGE + (tid / LT) * L_OPERAND + row * 128 + ((c ^ ((row >> 1) & 7)) << 4) + 8) = 0;
        bar_lds();
    };
    issue(0);
    if (nk > 1) {
        issue(1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * L_NL) : "memory");
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    bar_lds();
    if (nk == 1) trim();
    Operands lo, hi;
    read(0, 0, lo);
    for (int kt = 0; kt < nk - 1; ++kt) {
        read(kt, 1, hi);
        multiply(lo);
#pragma unroll
        for (int x = 0; x < 12; ++x) {   // two MFMAs, one LDS read
            __builtin_amdgcn_sched_group_barrier(0x8, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x8, 8, 0);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's loads of K-tile kt + 1 have landed,
        bar_lds();                                         // everyone's have, and everyone has read K-tile kt
        if (kt + 2 < nk) issue(kt + 2);
        if (kt + 2 == nk) trim();
        __builtin_amdgcn_sched_barrier(0);
        read(kt + 1, 0, lo);
        multiply(hi);
#pragma unroll
        for (int x = 0; x < 12; ++x) {
            __builtin_amdgcn_sched_group_barrier(0x8, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x8, 8, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    read(nk - 1, 1, hi);
    multiply(lo);
    multiply(hi);
    const __amdgpu_buffer_rsrc_t rsC = __builtin_amdgcn_make_buffer_rsrc(q.C, 0, q.Mr * q.ldc * 4, 0x00020000);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = n0 + wn + j * 16 + lr;
        const float bv = q.bias && n < q.Nc ? q.bias[n] : 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // (rows beyond the matrix are beyond the buffer: dropped)
                const unsigned at = n < q.Nc ? ((unsigned)(m0 + wm + i * 16 + lk * 4 + r) * q.ldc + n) * 4 : 0xFFFFFFF0u;
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][j][r] + bv), rsC, at, 0, 0);
            }
    }
}

}  // namespace

void GemmGroup::launch_bf16(hipStream_t s) {
    const int tiles = lay_out(T);
    if (!k_minor) {
        hipLaunchKernelGGL(gemm_bf16_kernel, dim3(group_grid(tiles)), dim3(256), 0, s, a);
        return;
    }
    split(tiles, PART_ROWS, BK);
    hipLaunchKernelGGL(gemm_bf16_k_minor_kernel, dim3(group_grid(tiles * a.parts)), dim3(256), 0, s, a);
    add_parts(s);
}

void GemmGroup::add_parts(hipStream_t s) {
    if (a.parts <= 1) return;
    unsigned most = 0;
    for (int i = 0; i < a.n; ++i) most = std::max(most, (unsigned)a.p[i].Mr * a.p[i].Nc);
    hipLaunchKernelGGL(gemm_add_parts_kernel, dim3(std::min(1024u, (most + 255) / 256), a.n), dim3(256), 0, s, a);
}

bool GemmGroup::launch_large(hipStream_t s) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_bf16_large_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            L_STAGES * L_STAGE) != hipSuccess) return false;
    lay_out(LT);
    hipLaunchKernelGGL(gemm_bf16_large_kernel, dim3(group_grid(a.tiles)), dim3(L_THREADS), L_STAGES * L_STAGE, s, a);
    a.n = 0;
    return true;
}

}  // namespace ver
