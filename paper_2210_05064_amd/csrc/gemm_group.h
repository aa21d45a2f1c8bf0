// Contractions of the LSTM outside the time loops, several to a launch: host interface of gemm_f32.hip and gemm_bf16.hip.
#pragma once
#include <algorithm>

#include "common.h"

namespace ver {

constexpr int GEMM_GROUP_MAX = 4;
struct GemmProblem {
    const void* A; const void* B; float* C; const float* bias;
    int lda, ldb, ldc, Mr, Nc, K, unperm_h;
    int tiles_n, tile_first;   // column tiles; first tile of the problem in the launch
    float* part;               // parts > 1: [parts][Mr][Nc]
};
// parts > 1: that many workgroups per tile take k_part of the contraction each.
// alone: the launch does nothing if it points to a zero (lstm_pipe.h: PLAN_ALONE); NULL: it always runs.
struct GemmGroupArgs { GemmProblem p[GEMM_GROUP_MAX]; int n, tiles, parts, k_part; const int* alone; };

// Up to four contractions in one launch, all with the contraction index contiguous (K-major: C = A[Mr, K] B[Nc, K]^T + bias)
// or all with it outermost (K-minor: C = A[K, Mr]^T B[K, Nc]); operands fp32 or bf16, C and bias fp32.  Leading dimensions,
// Nc, K (K-major) and Mr (K-minor) are multiples of 4; unperm_h > 0 stores output row m at row (m % 4) * unperm_h + m / 4.
struct GemmGroup {
    GemmGroupArgs a{};
    bool k_minor, bf16;
    float* part;   // scratch of part_floats (bf16, K-minor) or row_part_floats (fp32, K-major), or NULL
    GemmGroup(bool k_minor_, bool bf16_, float* part_ = nullptr) : k_minor(k_minor_), bf16(bf16_), part(part_) {}
    // K-minor bf16 contractions in 64 x 64 tiles are split into parts of at least PART_ROWS rows (a part takes a few us whatever its
    // length, and one more pass adds the parts) while all parts' tiles are at most PART_TILES, what the chip holds at a time.
    // us per launch (bf16), one part -> several: 32 inputs, 64 units, 2048 rows 23 -> 12, 8192 75 -> 13, 131072 1501 -> 34; 256 units, 8192
    // rows 76 -> 21, 131072 1560 -> 166; 1044 inputs, 320 units, 1500 rows 21 -> 25, 8192 81 -> 67.  At least 256 / 512 / 1024 rows: 64
    // units, 8192 rows 11.3 / 12.6 / 16.3; 320 units, 1000 rows 22 / 16 / 16.  At most 512 / 1024 / 2048 tiles: 256 units, 32768 rows 78 /
    // 50 / 55; 320 units, 32768 rows 400 / 248 / 269.
    static constexpr int PART_ROWS = 512, PART_TILES = 1024;
    // Bound of the scratch for contractions over K rows of up to `outputs` results per launch.
    static size_t part_floats(size_t outputs, int K) {
        return K < 2 * PART_ROWS ? 0 : std::min((size_t)PART_TILES * 64 * 64, outputs * (K / PART_ROWS));
    }
    // K-major fp32 contractions of few tiles over wide inputs are split in the same way, into parts of at least PART_COLS.  us per
    // projection, one part -> several (128 x 128 tiles split up to eight ways, before: in brackets): 59 rows, 64 units, 4096
    // inputs 46 -> 30 (54), 16384 183 -> 31 (166); 59 rows, 512 units, 16384 inputs 294 -> 72 (168); 256 rows, 512 units 301 -> 149 (178).
    static constexpr int PART_COLS = 2048;
    static size_t row_part_floats(int Mr, int Nc, int K) {
        return K < 2 * PART_COLS ? 0 : std::min((size_t)PART_TILES * 64 * 64, (size_t)Mr * Nc * (K / PART_COLS));
    }
    // Whether all arrays are within the kernels' 32-bit byte offsets.
    bool fits(int lda, int ldb, int ldc, int Mr, int Nc, int K) const {
        const size_t rowsA = k_minor ? K : Mr, rowsB = k_minor ? K : Nc, es = bf16 ? 2 : 4, lim = 0x7fffffff;
        constexpr size_t over = 256;   // rows that a last tile may address beyond the arrays (they read zero)
        return (rowsA + over) * lda * es < lim && (rowsB + over) * ldb * es < lim && (size_t)Mr * ldc * 4 < lim;
    }
    // False if they are not (or the launch is full): not added.
    bool add(const void* A, int lda, const void* B, int ldb, float* C, int ldc, int Mr, int Nc, int K, const float* bias, int unperm_h) {
        if (a.n >= GEMM_GROUP_MAX || !fits(lda, ldb, ldc, Mr, Nc, K)) return false;
        a.p[a.n++] = GemmProblem{A, B, C, bias, lda, ldb, ldc, Mr, Nc, K, unperm_h, 0, 0, nullptr};
        return true;
    }
    // Tiles of TM rows and TN columns: numbers the tiles of all problems and returns how many there are.
    int lay_out(int T) { return lay_out(T, T); }
    int lay_out(int TM, int TN) {
        int tiles = 0;
        for (int i = 0; i < a.n; ++i) {
            GemmProblem& q = a.p[i];
            q.tiles_n = (q.Nc + TN - 1) / TN;
            q.tile_first = tiles;
            tiles += q.tiles_n * ((q.Mr + TM - 1) / TM);
        }
        return a.tiles = tiles;
    }
    void launch(hipStream_t s) {
        if (a.n > 0) bf16 ? launch_bf16(s) : launch_f32(s);
        a.n = 0;
    }
    // One K-major bf16 contraction in 256 x 256 tiles (false: not launched).
    static constexpr int LARGE_TILE = 256;
    bool launch_large(hipStream_t s);

private:
    // Parts of at least `least` of the contraction (the same in all problems) for launches of `tiles` tiles, and where their
    // results go; add_parts, behind the launch, adds those.
    int parts(int tiles, int least) const { return part ? std::max(1, std::min(a.p[0].K / least, PART_TILES / tiles)) : 1; }
    void split(int tiles, int least, int BK) {
        const int K = a.p[0].K;
        a.parts = parts(tiles, least);
        a.k_part = ((K + a.parts - 1) / a.parts + BK - 1) / BK * BK;
        a.parts = (K + a.k_part - 1) / a.k_part;   // (none of them empty)
        float* to = part;
        for (int i = 0; a.parts > 1 && i < a.n; ++i) {
            a.p[i].part = to;
            to += (size_t)a.parts * a.p[i].Mr * a.p[i].Nc;
        }
    }
    void add_parts(hipStream_t s);
    void launch_f32(hipStream_t s);
    void launch_bf16(hipStream_t s);
};

// Which tile of a launch a workgroup computes (-1: none).  Workgroups go to the 8 XCDs round-robin: every XCD takes a stretch
// of consecutive tiles, so that the rows they share are fetched into its L2 once.
__device__ __forceinline__ int group_tile(int tiles) {
    const int per = gridDim.x / 8, t = (blockIdx.x % 8) * per + blockIdx.x / 8;
    return t < tiles ? t : -1;
}
inline int group_grid(int tiles) { return (tiles + 7) / 8 * 8; }
__device__ __forceinline__ GemmProblem group_problem(const GemmGroupArgs& g, int t) {
    GemmProblem q = g.p[0];   // uniform selects (an indexed copy of a kernel argument would live in scratch memory)
#pragma unroll
    for (int i = 1; i < GEMM_GROUP_MAX; ++i)
        if (i < g.n && t >= g.p[i].tile_first) q = g.p[i];
    return q;
}

}  // namespace ver
