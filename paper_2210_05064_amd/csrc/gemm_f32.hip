// fp32 contractions of the LSTM on v_mfma_f32_16x16x4_f32: input projections and input gradients (K-major operands) and
// weight gradients (K-minor operands: the contraction runs over the packed rows).  gfx950 only.
//
// Bound by the MFMAs (157 TFLOP/s at 2.4 GHz; these launches run at 2.0 to 2.1), so what matters is that every SIMD always has
// one to issue:
//  * K-tiles of 32 go from global memory straight into LDS (buffer_load ... lds), one barrier per K-tile.  Neither direction
//    needs a transposition: the MFMA takes one value per lane and any assignment of contraction indices to lanes works as
//    long as A and B agree, so K-major rows are read 16 bytes (4 k) at a time, and K-minor rows are read along the
//    output index (with 64 x 64 tiles two adjacent outputs per lane, which go to two MFMAs: the tile's rows and columns
//    are permuted, and the store puts them back);
//  * two stages of LDS, so that four workgroups share a CU and one multiplies while another waits (three or four stages with
//    fewer workgroups: 8 to 15 % slower);
//  * square tiles of 64, or of 32 where their rounds of the chip take less (launch rule below), without splitting the
//    contraction (but for few rows of very wide inputs: gemm_group.h): no partial tiles in memory and no pass that adds
//    them.  A running sum is moved to a second set of registers every 128 k, so chains of additions stay as short as with a split;
//  * all weight gradients of a minibatch share a launch, so the last, partly filled round of the chip is paid once.
// us, the 128 x 128 register-staged tiles with a split contraction that ran here before -> now: the four weight gradients of 2 x
// 512 units over 1024 rows (8.7 GFLOP) 235 -> 88, input projection 1024 x 2048 x 516 55 -> 26, input gradient 1024 x
// 516 x 2048 55 -> 35.  Counters of the first (tiles of 64): the CUs are busy 84 % of the launch (its last round is partly filled), the MFMAs 79 % of that.
#include "gemm_group.h"
#include "mfma.h"

namespace ver {
namespace {

constexpr int BK = 32;
// T: rows and columns of a workgroup's tile (4 waves, 2 x 2)
template <int T> struct Geom {
    static constexpr int W = T / 2, WT = W / 16;       // a wave's square, in MFMA tiles
    static constexpr int OPERAND = T * BK * 4, STAGE = 2 * OPERAND;
    static constexpr int STAGES = 2;
    static constexpr int NL = OPERAND / 1024 / 4;      // load instructions per wave, operand and stage
    static constexpr int ACCS = T == 32 ? 2 : 1;       // running sums per MFMA tile (a wave with a single tile alternates)
};

// Chunk (16 bytes) position p of LDS row r holds chunk p ^ swz(r).
template <int T, bool KMIN> __device__ __forceinline__ int swz(int r) {
    if (!KMIN) return (r >> 1) & 7;                    // rows of 8 chunks, read by 16 lanes of one chunk column
    return T == 64 ? (r & 1) << 3 : ((r >> 1) & 1) << 2;   // 16 or 8 chunks, read by 16 lanes along each of 4 rows
}

template <int T, bool KMIN>
__device__ __forceinline__ void tile(const GemmProblem& q, int t, unsigned char* smem) {
    typedef Geom<T> G;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const int m0 = t / q.tiles_n * T, n0 = t % q.tiles_n * T;
    const int wm = (wave >> 1) * G::W, wn = (wave & 1) * G::W;
    const int nk = (q.K + BK - 1) / BK;
    const int rowsA = KMIN ? q.K : q.Mr, rowsB = KMIN ? q.K : q.Nc;
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.A), 0, rowsA * q.lda * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.B), 0, rowsB * q.ldb * 4, 0x00020000);
    // A load instruction fills 1 KB of LDS (8 rows K-major; 1024 / (4 T) rows K-minor); the swizzle is applied on the global side.
    constexpr int CHUNKS = KMIN ? T / 4 : BK / 4;
    unsigned offA[G::NL], offB[G::NL];
    int kc[G::NL];   // K-major: this lane's first k in the K-tile
#pragma unroll
    for (int j = 0; j < G::NL; ++j) {
        const int row = (wave * G::NL + j) * (64 / CHUNKS) + lane / CHUNKS, c = (lane % CHUNKS) ^ swz<T, KMIN>(row);
        kc[j] = c * 4;
        if (KMIN) {   // rows beyond K are beyond the buffer and read zero; columns beyond the matrix feed outputs that are not stored
            offA[j] = ((unsigned)row * q.lda + m0 + c * 4) * 4;
            offB[j] = ((unsigned)row * q.ldb + n0 + c * 4) * 4;
        } else {      // rows beyond the matrix repeat its last one
            offA[j] = ((unsigned)min(m0 + row, q.Mr - 1) * q.lda + c * 4) * 4;
            offB[j] = ((unsigned)min(n0 + row, q.Nc - 1) * q.ldb + c * 4) * 4;
        }
    }
    auto issue = [&](int kt) {
        unsigned char* st = smem + kt % G::STAGES * G::STAGE + wave * G::NL * 1024;
        const unsigned stepA = KMIN ? (unsigned)(kt * BK) * q.lda * 4 : kt * BK * 4, stepB = KMIN ? (unsigned)(kt * BK) * q.ldb * 4 : kt * BK * 4;
#pragma unroll
        for (int j = 0; j < G::NL; ++j) {
            const bool in = KMIN || kt * BK + kc[j] < q.K;   // (K is a multiple of 4 when K-major; beyond it: read zero)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_ptr_t)(st + j * 1024), 16, in ? offA[j] + stepA : 0xFFFFFFF0u, 0, 0, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (lds_ptr_t)(st + G::OPERAND + j * 1024), 16, in ? offB[j] + stepB : 0xFFFFFFF0u, 0, 0, 0);
        }
    };
    f32x4_t acc[G::ACCS][G::WT][G::WT], sum[G::WT][G::WT];
#pragma unroll
    for (int i = 0; i < G::WT; ++i)
#pragma unroll
        for (int j = 0; j < G::WT; ++j) {
            sum[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < G::ACCS; ++s) acc[s][i][j] = sum[i][j];
        }
    auto fold = [&] {
#pragma unroll
        for (int s = 0; s < G::ACCS; ++s)
#pragma unroll
            for (int i = 0; i < G::WT; ++i)
#pragma unroll
                for (int j = 0; j < G::WT; ++j) {
                    sum[i][j] += acc[s][i][j];
                    acc[s][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                }
    };
    // A wave's operands of one K-tile.  K-major: 16 bytes along k; K-minor: WT adjacent outputs for each of 8 k.
    constexpr int STEPS = KMIN ? BK / 4 : BK / 16, VALS = KMIN ? 1 : G::WT;
    typedef float op_t __attribute__((ext_vector_type(KMIN ? G::WT : 4)));
    struct Operands { op_t a[STEPS][VALS], b[STEPS][VALS]; };
    auto read = [&](int kt, Operands& o) {
        const unsigned char* sA = smem + kt % G::STAGES * G::STAGE;
        const unsigned char* sB = sA + G::OPERAND;
#pragma unroll
        for (int ks = 0; ks < STEPS; ++ks)
#pragma unroll
            for (int i = 0; i < VALS; ++i) {
                if constexpr (KMIN) {
                    const int k = ks * 4 + lk, ca = wm + lr * G::WT, cb = wn + lr * G::WT;
                    o.a[ks][i] = *reinterpret_cast<const op_t*>(sA + k * (T * 4) + (((ca >> 2) ^ swz<T, KMIN>(k)) << 4) + (ca & 3) * 4);
                    o.b[ks][i] = *reinterpret_cast<const op_t*>(sB + k * (T * 4) + (((cb >> 2) ^ swz<T, KMIN>(k)) << 4) + (cb & 3) * 4);
                } else {
                    const int ra = wm + i * 16 + lr, rb = wn + i * 16 + lr;
                    o.a[ks][i] = *reinterpret_cast<const op_t*>(sA + ra * 128 + (((ks * 4 + lk) ^ swz<T, KMIN>(ra)) << 4));
                    o.b[ks][i] = *reinterpret_cast<const op_t*>(sB + rb * 128 + (((ks * 4 + lk) ^ swz<T, KMIN>(rb)) << 4));
                }
            }
    };
    auto multiply = [&](const Operands& o) {
#pragma unroll
        for (int ks = 0; ks < STEPS; ++ks)
#pragma unroll
            for (int e = 0; e < (KMIN ? 1 : 4); ++e)
#pragma unroll
                for (int i = 0; i < G::WT; ++i)
#pragma unroll
                    for (int j = 0; j < G::WT; ++j) {
                        f32x4_t& c = acc[(ks + e) % G::ACCS][i][j];
                        c = KMIN ? mfma_f32_16x16x4(o.a[ks][0][KMIN ? i : 0], o.b[ks][0][KMIN ? j : 0], c)
                                 : mfma_f32_16x16x4(o.a[ks][KMIN ? 0 : i][e], o.b[ks][KMIN ? 0 : j][e], c);
                    }
    };
    // this wave's loads have landed, and after the barrier so have everyone's
    auto arrived = [&] {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        bar_lds();
    };
    for (int kt = 0; kt < G::STAGES && kt < nk; ++kt) issue(kt);
    if (nk >= G::STAGES) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((G::STAGES - 1) * 2 * G::NL) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    bar_lds();
    // The operands of K-tile kt + 1 are read before the MFMAs of K-tile kt are issued; K-minor, whose 8 paired reads keep a small
    // tile's 8 MFMAs waiting for longest, between them (two layers of 64 units, 2048 rows 18.0 -> 14.8 us, of 512, 1024 rows in
    // tiles of 32 92.7 -> 87.5; K-major in tiles of 32 3 % slower).
    Operands even, odd;
    auto step = [&](int kt, const Operands& now, Operands& next) {
        arrived();   // (and everyone has read the stage of kt, which is the one that is filled again)
        if (kt + G::STAGES < nk) issue(kt + G::STAGES);
        __builtin_amdgcn_sched_barrier(0);
        read(kt + 1, next);
        if (!KMIN) __builtin_amdgcn_sched_barrier(0);
        multiply(now);
        if constexpr (KMIN) {
            constexpr int MFMAS = 8 * G::WT * G::WT, READS = 8, PER = MFMAS / READS / 2 > 0 ? MFMAS / READS / 2 : 1;
#pragma unroll
            for (int x = 0; x < READS; ++x) {   // PER MFMAs, one (paired) LDS read
                __builtin_amdgcn_sched_group_barrier(0x8, PER, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x8, MFMAS - READS * PER, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    read(0, even);
    int kt = 0;
    for (; kt + 2 < nk; kt += 2) {
        step(kt, even, odd);
        step(kt + 1, odd, even);
        if ((kt & 2) != 0) fold();   // every 4 K-tiles
    }
    if (kt + 1 < nk) {
        step(kt, even, odd);
        multiply(odd);
    } else {
        multiply(even);
    }
    fold();
    // element r of lane l: row lk * 4 + r, column lr of the MFMA tile; what lies outside the matrix is stored out of the
    // buffer's range, i.e. dropped
    const __amdgpu_buffer_rsrc_t rsC = __builtin_amdgcn_make_buffer_rsrc(q.C, 0, q.Mr * q.ldc * 4, 0x00020000);
    float bv[G::WT];
#pragma unroll
    for (int j = 0; j < G::WT; ++j) {
        const int n = n0 + wn + (KMIN ? lr * G::WT + j : j * 16 + lr);
        bv[j] = q.bias && n < q.Nc ? q.bias[n] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < G::WT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + wm + (KMIN ? (lk * 4 + r) * G::WT + i : i * 16 + lk * 4 + r);
            const int out = q.unperm_h > 0 ? (m & 3) * q.unperm_h + (m >> 2) : m;
#pragma unroll
            for (int j = 0; j < G::WT; ++j) {
                const int n = n0 + wn + (KMIN ? lr * G::WT + j : j * 16 + lr);
                const unsigned at = m < q.Mr && n < q.Nc ? ((unsigned)out * q.ldc + n) * 4 : 0xFFFFFFF0u;
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sum[i][j][r] + bv[j]), rsC, at, 0, 0);
            }
        }
}

template <int T, bool KMIN>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmGroupArgs g) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int all = group_tile(g.tiles * g.parts);
    if (all < 0 || (g.alone && *g.alone == 0)) return;
    const int part = g.parts > 1 ? all / g.tiles : 0, t = all - part * g.tiles;
    GemmProblem q = group_problem(g, t);
    if (!KMIN && g.parts > 1) {   // columns [part * k_part, ...) of both operands, into the part's own results
        const int k0 = part * g.k_part;
        q.A = static_cast<const float*>(q.A) + k0;
        q.B = static_cast<const float*>(q.B) + k0;
        q.K = min(q.K - k0, g.k_part);
        q.C = q.part + (size_t)part * q.Mr * q.Nc;
        q.ldc = q.Nc;
        q.bias = nullptr;
    }
    tile<T, KMIN>(q, t - q.tile_first, smem);
}

template <int T, bool KMIN>
void start(const GemmGroupArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((gemm_f32_kernel<T, KMIN>), dim3(group_grid(a.tiles * a.parts)), dim3(256), Geom<T>::STAGES * Geom<T>::STAGE, s, a);
}

// A round of 256 tiles of 64, one per CU, lasts as long as ROUND_OF_32 tiles of 32 (a CU's workgroups share its MFMAs: it is the
// count per CU that matters, not how many workgroups are resident), and tiles of 64 need two rounds, so that a CU has another
// workgroup while one waits.  us with tiles of 64 / 32, by tiles of 64 (of 32).  K-minor, 4096 rows: 336 (1188) 132 / 110, 544 (2112) 191 / 168, 800
// (3200) 262 / 234, 928 (3648) 261 / 267, 960 (3800) 262 / 301, 1056 (4160) 326 / 306, 1224 (4848) 327 / 369, 1440 (5696) 387 / 444, 2080 (8320) 567 /
// 634; 1024 rows: 544 54 / 48, 992 (3904) 76 / 80, 1056 91 / 85, 1312 (5184) 106 / 99.  K-major, K = 516: 256 (1024) 17.4 / 17.7, 384 (1536) 25 / 22, 448
// (1792) 26 / 24, 576 (2304) 34 / 32, 768 (3072) 35 / 39, 2048 (8192) 80 / 90; K = 2048 and 2052: 252 (952) 44 / 41, 384 74 / 65, 462 (1820) 74 / 77, 576
// (2176) 103 / 91, 640 (2560) 106 / 114, 1056 (4160) 167 / 160, 2048 269 / 335.
constexpr int ROUND = 256, ROUND_OF_32 = 850;
// Of a split contraction: tiles of 64 where all parts' tiles are as many as the chip holds (us with 64 / 32: 256 rows, 512 units, 16384
// inputs, 8 parts of 128 tiles 149 / 192; 1024 rows, 256 units, 4 parts of 256 tiles 282 / 309).

}  // namespace

void GemmGroup::launch_f32(hipStream_t s) {
    a.parts = 1;
    const int tiles_32 = lay_out(32);
    int tiles = lay_out(64);
    const int rounds = (tiles + ROUND - 1) / ROUND;
    bool of_64 = rounds >= 2 && ROUND_OF_32 * rounds <= tiles_32;
    const bool whole = k_minor || of_64;
    if (!whole) of_64 = tiles * parts(tiles, PART_COLS) >= PART_TILES;
    if (!of_64) tiles = lay_out(32);
    if (!whole) split(tiles, PART_COLS, BK);
    if (of_64) k_minor ? start<64, true>(a, s) : start<64, false>(a, s);
    else k_minor ? start<32, true>(a, s) : start<32, false>(a, s);
    add_parts(s);
}

}  // namespace ver
