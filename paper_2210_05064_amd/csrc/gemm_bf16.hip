// bf16 contractions of the LSTM on v_mfma_f32_16x16x32_bf16 in 64 x 64 tiles, for the sizes whose larger tiles (lstm_proj_dma_kernel,
// the grouped kernels of gemm.h) would leave CUs idle.  gfx950 only.
//
// Same frame as gemm_f32.hip: K-tiles of 64 straight from global memory into LDS, two stages, one barrier per K-tile, the operands
// of the next K-tile read before the MFMAs of this one, several workgroups per CU.  A wave's 32 x 32 needs 4 KB of LDS reads for 64
// MFMA cycles, so a full chip is bound by LDS at half the MFMA rate; these launches are bound by the latency of their few
// K-tiles instead.  K-minor operands are read with the transposing LDS load (its lane layout: gemm.h).
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
    if (t < 0) return;
    const GemmProblem q = group_problem(g, t);
    tile<false>(q, t - q.tile_first, smem);
}
__global__ __launch_bounds__(256) void gemm_bf16_k_minor_kernel(GemmGroupArgs g) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[STAGES * STAGE];
    const int t = group_tile(g.tiles);
    if (t < 0) return;
    const GemmProblem q = group_problem(g, t);
    tile<true>(q, t - q.tile_first, smem);
}

}  // namespace

void GemmGroup::launch_bf16(hipStream_t s) {
    lay_out(T);
    if (k_minor) hipLaunchKernelGGL(gemm_bf16_k_minor_kernel, dim3(group_grid(a.tiles)), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(gemm_bf16_kernel, dim3(group_grid(a.tiles)), dim3(256), 0, s, a);
}

}  // namespace ver
