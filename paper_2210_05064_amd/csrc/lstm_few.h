// The time loops while a group has few alive pieces (included by lstm_rec.h).  gfx950 only.
//
// A timestep with a handful of alive pieces is all latency: the flag protocol of lstm_rec.h passes through a store
// acknowledgement, a workgroup barrier, a flag store, a poll, a barrier, the copy of the rows into LDS and another
// barrier before the first MFMA, and every wave's wait for its stores also waits for the saved activations.  Here
// the exchanged values announce themselves:
//  * Rows are exchanged through a ring of FEW_RING slots per group that stays in the XCD's L2.  An empty 32-bit word
//    of a slot holds FEW_EMPTY, which no published word equals (see few_word), so a reader polls the values it needs
//    and has them when the poll succeeds: no flag, no wait for a store's acknowledgement, no barrier, no copy.
//  * Each of the 8 waves owns an eighth of the contraction (all gate rows of the workgroup) and polls just that
//    slice of the rows.  Up to 4 pieces (lstm_quad.h): straight into the operand registers of the product.  The 16 rows of an
//    operand hold P pieces x 16/P operand blocks, so that a load instruction is full and four neighbouring lanes
//    read 64 contiguous bytes (lanes of a quad that read different lines cost a cycle each); a block is brought to
//    its piece's first row by rotating the lanes of a row (DPP), the other rows of the operand are whatever they are (a
//    row of A only reaches the same row of the result).  fp32 reads its values as DPP broadcasts.  More pieces: in
//    the order of memory into registers, and through a piece of LDS of the wave's own into operand order.
//  * The partial sums of the waves meet in LDS; a thread (up to 4 pieces: four lanes, two buffers, one barrier per
//    timestep) then owns one (piece, unit) and keeps its cell state (backward: both carried gradients) in registers.
//  * Everything that is not on the way from one exchange to the next (saved activations, copies for other XCDs,
//    prefetches) is issued right after a poll has succeeded, so that it completes behind the product: memory
//    operations of a wave complete in order, and what is queued before a poll delays it.
// Reuse of a slot: a workgroup that has read the rows of one timestep from all workgroups knows that all of them
// are done with the rows of the timestep before; each clears its own words of that slot then, and publishes at least
// once more after the clearing stores have completed before anyone polls the slot again.
//
// Bound by the latency of its phases: about 0.6 us for the exchange alone (a kernel that does nothing else), 0.43 us for
// the MFMAs of one 16-row tile at H = 1024 (1.7 us in fp32 at H = 512), then the partial sums through LDS and the cell
// update.  Microseconds per timestep (time of a launch against its timesteps; two layers, with 16 pieces one), a thread per (piece, unit)
// throughout -> four lanes up to 4 pieces:
//     alive pieces                     1             2             4             8      16
//     bf16, H = 1024   forward    1.37 -> 1.25  1.34 -> 1.24          1.37     1.9    2.1
//                      backward   1.63 -> 1.58  1.81 -> 1.61  2.14 -> 2.01     2.4    2.9
//     bf16, H = 512    forward    1.04 -> 0.90  1.04 -> 0.88  1.05 -> 0.94     1.3    1.3
//                      backward   1.36 -> 1.16  1.36 -> 1.16  1.58 -> 1.34     1.5    2.0
//     fp32, H = 512    forward    1.23 -> 1.12  1.51 -> 1.42  2.13 -> 2.05     3.0    3.0
//                      backward   1.49 -> 1.28  2.05 -> 1.82  3.06 -> 2.74     3.5    4.2
// (the flag protocol took 2.2 to 2.4 us with one piece and 3.3 to 5.7 with 16.)
// What mattered after the exchange itself: four neighbouring lanes on contiguous memory (16 pieces forward 2.74 -> 2.04 us,
// backward 5.25 -> 2.99), reading the eight partial sums without a branch per share (0.2 us per timestep), and no wait
// for a prefetch before the next poll (0.1 us).
#pragma once

namespace ver {

constexpr int FEW_RING = 4;
constexpr unsigned FEW_EMPTY = 0xffffffffu;
// Alive pieces up to which a group runs this form: one MFMA tile.
constexpr int FEW_MAX = 16;
// Operand blocks per wave: the contraction (H forward, 4H backward) over 8 waves.
template <int MODE, bool WIDE> struct FewBlocks {
    static constexpr int fwd = MODE == MODE_BF16 ? (WIDE ? 4 : 2) : 4;
    static constexpr int bwd = MODE == MODE_BF16 ? (WIDE ? 16 : 8) : 16;
};
inline __host__ __device__ size_t few_slot_bytes(int mode, int row_elems) {
    return (size_t)FEW_MAX * (mode == MODE_BF16 ? 2 : 4) * row_elems;
}
inline __host__ __device__ size_t few_ring_bytes(int mode, int row_elems) { return FEW_RING * few_slot_bytes(mode, row_elems); }
// LDS: partial sums, [8 waves][16 pieces][columns + 4] or two buffers of [8 waves][4 pieces][columns + 4], then (more than
// 4 pieces) 16 rows of NB operand blocks per wave.
constexpr int few_row(int cols) { return cols + 4; }   // (16 bytes more, always zero: 16 pieces of a fragment hit different banks)
constexpr int few_part_floats(int cols) { return REC_WAVES * 16 * few_row(cols); }
constexpr int few_stage_bytes(int nb) { return 16 * nb * 64; }   // per wave
inline __host__ __device__ size_t few_lds_bytes(int cols, int nb) {
    return (size_t)few_part_floats(cols) * sizeof(float) + (size_t)REC_WAVES * few_stage_bytes(nb);
}

template <int I> struct FewIdx { static constexpr int value = I; };
template <int N, int I = 0, typename F> __device__ __forceinline__ void few_for(F&& f) {
    if constexpr (I < N) {
        f(FewIdx<I>{});
        few_for<N, I + 1>(f);
    }
}
template <int CTRL> __device__ __forceinline__ unsigned few_dpp(unsigned v) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
// Lane i of every row of 16 gets the value of lane (i + S) % 16.
template <int S> __device__ __forceinline__ f32x4_t few_rot(u32x4_t v) {
    if constexpr (S != 0) {
        constexpr int CTRL = 0x120 + 16 - S;   // row_ror:(16 - S)
        v = u32x4_t{few_dpp<CTRL>(v[0]), few_dpp<CTRL>(v[1]), few_dpp<CTRL>(v[2]), few_dpp<CTRL>(v[3])};
    }
    return __builtin_bit_cast(f32x4_t, v);
}
// acc + sum of w[e] * (v[e] of lane I of the lane's row of 16).  Written out because the compiler makes a move and a
// multiply-add of every term; the wait states are those between a write of a register and its use through DPP.
template <int I> __device__ __forceinline__ float few_fma4(float acc, u32x4_t v, f32x4_t w) {
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %1, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %2, %6 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %3, %7 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %4, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
        : "+v"(acc)
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "n"(I));
    return acc;
}
__device__ __forceinline__ void few_swap16(float& a, float& b) {   // odd rows of a <-> even rows of b
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void few_swap32(float& a, float& b) {   // upper half of a <-> lower half of b
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}
// A use of registers whose loads are known to have completed (the wait of a poll is written out, which the compiler does
// not see): without it the first real use, in the middle of a timestep, waits for everything requested since.
__device__ __forceinline__ void few_touch(f32x4_t& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void few_touch(float& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void few_touch(int& v) { asm volatile("" : "+v"(v)); }
// A word to publish: never FEW_EMPTY (only a pair of NaNs, or an fp32 NaN, has these bits; it stays NaN).
__device__ __forceinline__ unsigned few_word(unsigned v) { return v == FEW_EMPTY ? FEW_EMPTY - 1 : v; }

// few_fwd and few_bwd take the address of the kernel's arguments and load them once more, and take everything else as values that
// are made scalar here: their time loops shared the scalar registers with what the kernel keeps for its other forms and roles, and
// fetched their own constants from spill lanes (64 to 88 v_readlane per backward timestep of a consumer, now 2 to 18).  (As calls, with
// registers of their own, they save and restore a hundred vector registers per lane: 16 us per launch at H = 1024.)
template <typename T> __device__ __forceinline__ T few_scalar(T v) {
    if constexpr (sizeof(T) == 8) {
        const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
        const unsigned long long u = (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)b) |
                                     (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32;
        return __builtin_bit_cast(T, u);
    } else {
        return __builtin_bit_cast(T, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
    }
}
// A pointer that the compiler knows to be global (of one read from memory it does not, and a generic access also counts
// as one to LDS).
template <typename T> __device__ __forceinline__ void few_global(T*& p) { p = (T*)(__attribute__((address_space(1))) T*)p; }
// Kept in vector registers: what a timestep rarely asks for, or asks for with a lane's address.
template <typename T> __device__ __forceinline__ void few_away(T& v) {
    if constexpr (std::is_pointer<T>::value) {
        unsigned long long b = reinterpret_cast<unsigned long long>(v);
        asm volatile("" : "+v"(b));
        typedef typename std::remove_pointer<T>::type V;
        v = (T)(__attribute__((address_space(1))) V*)b;
    } else {
        asm volatile("" : "+v"(v));
    }
}

// Reads L x 16 bytes per lane at from + off[j]; with `check` again and again until no word is empty.  The loads
// bypass the CU's L1 (sc0 sc1) and are written out because the compiler waits for every volatile load by itself.
// Lanes that do not `take` part keep what raw holds.  False: the wait was abandoned (time-out here or in another
// workgroup).
template <int L>
__device__ __forceinline__ bool few_read(const unsigned char* from, const unsigned (&off)[L], bool take, bool check, u32x4_t (&raw)[L], int* err) {
    static_assert(L == 1 || L == 2 || L == 4 || L == 8, "loads per poll");
    // (the same for all lanes, which the asm needs and the compiler does not always see)
    const unsigned long long at = reinterpret_cast<unsigned long long>(from);
    const unsigned char* base = reinterpret_cast<const unsigned char*>(
        (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)at) | (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(at >> 32)) << 32);
    long long spins = 0;
    for (;;) {
        unsigned m = 0;
        if (take) {
            if constexpr (L == 1)
                asm volatile("global_load_dwordx4 %0, %1, %2 sc0 sc1\n\ts_waitcnt vmcnt(0)" : "+&v"(raw[0]) : "v"(off[0]), "s"(base) : "memory");
            else if constexpr (L == 2)
                asm volatile("global_load_dwordx4 %0, %2, %4 sc0 sc1\n\tglobal_load_dwordx4 %1, %3, %4 sc0 sc1\n\ts_waitcnt vmcnt(0)"
                             : "+&v"(raw[0]), "+&v"(raw[1]) : "v"(off[0]), "v"(off[1]), "s"(base) : "memory");
            else if constexpr (L == 4)
                asm volatile("global_load_dwordx4 %0, %4, %8 sc0 sc1\n\tglobal_load_dwordx4 %1, %5, %8 sc0 sc1\n\t"
                             "global_load_dwordx4 %2, %6, %8 sc0 sc1\n\tglobal_load_dwordx4 %3, %7, %8 sc0 sc1\n\ts_waitcnt vmcnt(0)"
                             : "+&v"(raw[0]), "+&v"(raw[1]), "+&v"(raw[2]), "+&v"(raw[3])
                             : "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base) : "memory");
            else
                asm volatile("global_load_dwordx4 %0, %8, %16 sc0 sc1\n\tglobal_load_dwordx4 %1, %9, %16 sc0 sc1\n\t"
                             "global_load_dwordx4 %2, %10, %16 sc0 sc1\n\tglobal_load_dwordx4 %3, %11, %16 sc0 sc1\n\t"
                             "global_load_dwordx4 %4, %12, %16 sc0 sc1\n\tglobal_load_dwordx4 %5, %13, %16 sc0 sc1\n\t"
                             "global_load_dwordx4 %6, %14, %16 sc0 sc1\n\tglobal_load_dwordx4 %7, %15, %16 sc0 sc1\n\ts_waitcnt vmcnt(0)"
                             : "+&v"(raw[0]), "+&v"(raw[1]), "+&v"(raw[2]), "+&v"(raw[3]), "+&v"(raw[4]), "+&v"(raw[5]), "+&v"(raw[6]), "+&v"(raw[7])
                             : "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "v"(off[4]), "v"(off[5]), "v"(off[6]), "v"(off[7]), "s"(base)
                             : "memory");
#pragma unroll
            for (int j = 0; j < L; ++j) m = max(max(m, max(raw[j][0], raw[j][1])), max(raw[j][2], raw[j][3]));
        }
        if (!check || __all(m != FEW_EMPTY)) return true;
        ++spins;
        if ((spins & 1023) == 0 && (spins > REC_SPIN_LIMIT || __builtin_amdgcn_readfirstlane(ld_agent(err)) != 0)) {
            st_agent(err, 1);
            return false;
        }
    }
}
// The last slice of a wide bf16 layer may have half of the blocks (n_blk = NB / 2; every other slice is whole).  The
// weights of the blocks it does not have are zero, but zero times an infinite value would not be: they are skipped, or
// multiplied with zeros where a branch costs more (forward, 4 blocks: 445 us instead of 473 for two layers of 1024 on
// 4096 rows in 64 pieces).
template <int MODE, int MT> constexpr bool few_always_whole() { return !(MODE == MODE_BF16 && (MT == 8 || MT == 2)); }
// Offsets of the L loads of a lane: block blk + j * BPL of the slice, or block blk again where the slice has no such
// block (which is not multiplied).
template <int L, int BPL>
__device__ __forceinline__ void few_offsets(unsigned (&off)[L], unsigned first, int blk, int n_blk) {
#pragma unroll
    for (int j = 0; j < L; ++j) off[j] = first + (blk + j * BPL < n_blk ? j * BPL * 16 : 0);
}

// ---- up to 4 pieces: operands in the registers they were loaded into --------------------------------------------
// Register j of lane (lr, lk) holds, of piece lr / BPL, the 16 bytes lk of operand block j * BPL + lr % BPL, BPL = 16 / P.
// Adds the product with all tiles of the wave into acc.  bf16: pieces are the rows 0, BPL, 2 BPL, ... of A, so that lane
// group p * BPL / 4 holds piece p of the result, element 0.  fp32: acc[tile][piece] on the vector ALUs, a lane's share.
template <int MODE, int MT, int NB, int P, int L>
__device__ __forceinline__ void few_product(const f32x4_t (&w)[MT * NB], const u32x4_t (&raw)[L], int bs, int n_blk, f32x4_t (&acc)[MT]) {
    constexpr int BPL = 16 / P;
    if constexpr (MODE == MODE_BF16) {
        auto half = [&](auto first) {
            few_for<NB / 2>([&](auto ib) {
                constexpr int b = decltype(first)::value + decltype(ib)::value;
                const f32x4_t op = few_rot<b % BPL>(raw[b / BPL]);
#pragma unroll
                for (int j = 0; j < MT; ++j) acc[j] = mfma_block<MODE>(op, w[j * NB + b], acc[j]);
            });
        };
        half(FewIdx<0>{});
        // (a single load: the lanes of the blocks that are not there read nothing and keep their zeros)
        if (few_always_whole<MODE, MT>() || L == 1 || n_blk == NB) half(FewIdx<NB / 2>{});
    } else {
        few_for<P>([&](auto ip) {
            constexpr int p = decltype(ip)::value;
            if (p < bs)
                few_for<NB>([&](auto ib) {
                    constexpr int b = decltype(ib)::value;
#pragma unroll
                    for (int j = 0; j < MT; ++j) acc[j][p] = few_fma4<p * BPL + b % BPL>(acc[j][p], raw[b / BPL], w[j * NB + b]);
                });
        });
    }
}
// Leaves the wave's partial sums in LDS: s[piece * few_row(16 MT) + column].
template <int MODE, int MT, int P>
__device__ __forceinline__ void few_write(const f32x4_t (&acc)[MT], int bs, float* s) {
    constexpr int ROW = few_row(16 * MT), BPL = 16 / P;
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    if constexpr (MODE == MODE_BF16) {
        const int p = lk * 4 / BPL;   // the piece of this lane group, if it has one
        if (lk * 4 % BPL == 0 && p < bs)
#pragma unroll
            for (int j = 0; j < MT; ++j) s[p * ROW + j * 16 + lr] = acc[j][0];
    } else {   // fp32: the four lane groups hold shares of every sum
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (p < bs) {
                if constexpr (MT == 4) {
                    float a = acc[0][p], b = acc[1][p], c = acc[2][p], d = acc[3][p];
                    few_swap16(a, b);
                    few_swap16(c, d);
                    float u = a + b, v = c + d;
                    few_swap32(u, v);
                    s[p * ROW + lane] = u + v;
                } else {
                    static_assert(MT == 1, "tiles of the fp32 loops");
                    float a = acc[0][p], b = a;
                    few_swap32(a, b);
                    float u = a + b, v = u;
                    few_swap16(u, v);
                    if (lane < 16) s[p * ROW + lane] = u + v;
                }
            }
    }
}

// ---- up to 16 rows through LDS ----------------------------------------------------------------------------------
// A wave's staging area: 16 rows of C = 4 NB chunks of 16 bytes; position q of row r holds chunk q ^ key(r), which makes
// the operand reads (the same chunk of 16 rows) hit all banks.  Lane i of load j fills position i % C of row
// j * (64 / C) + i / C, i.e. 1 KB in lane order.
template <int NB> struct FewStage {
    static constexpr int C = 4 * NB, RPL = 64 / C, LOADS = 16 / RPL;   // chunks per row, rows per load, loads for 16 rows
    static_assert((C & (C - 1)) == 0 && C <= 64 && C >= 8, "blocks per wave");
    static __device__ __forceinline__ int key(int r) { return C >= 16 ? (r & 15) : ((r >> 1) & 7); }
    static __device__ __forceinline__ int row(int j) { return j * RPL + (int)(threadIdx.x & 63) / C; }
    // byte offset, inside the slice, of what this lane loads of row r (chunk 0 where the slice has no such chunk, which is
    // not multiplied)
    static __device__ __forceinline__ unsigned src(int r, int n_blk) {
        const int c = ((int)(threadIdx.x & 63) % C) ^ key(r);
        return (unsigned)(c < 4 * n_blk ? c : 0) * 16u;
    }
};
// Product of the staged rows with all tiles, added into acc: rows are columns of the result, lane l holds row l % 16 and
// columns (l / 16) * 4 + e of a tile.  zero: 16 bytes of zeros.  Calls read() once no operand is left to be fetched, ahead of
// the last (up to 8) blocks' MFMAs.  RAGGED: any number of blocks.
template <int MODE, int MT, int NB, bool RAGGED, typename F>
__device__ __forceinline__ void few_stage_product(const f32x4_t (&w)[MT * NB], const unsigned char* stage, const float* zero, int n_blk,
                                                  f32x4_t (&acc)[MT], F&& read) {
    constexpr int GRP = NB < 8 ? NB : 8;   // operands in flight
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    const unsigned char* row = stage + lr * (FewStage<NB>::C * 16);
    const int key = FewStage<NB>::key(lr);
#pragma unroll
    for (int b0 = 0; b0 < NB; b0 += GRP) {
        if (!few_always_whole<MODE, MT>() && GRP < NB && b0 >= n_blk) break;
        f32x4_t op[GRP];
#pragma unroll
        for (int b = 0; b < GRP; ++b) {
            const unsigned char* src = row + (((RAGGED ? min(lk * n_blk + b0 + b, 4 * n_blk - 1) : lk * n_blk + b0 + b) ^ key) << 4);
            if (!few_always_whole<MODE, MT>() && GRP == NB && b0 + b >= NB / 2 && n_blk < NB) src = reinterpret_cast<const unsigned char*>(zero);
            op[b] = *reinterpret_cast<const f32x4_t*>(src);
        }
        if (b0 + GRP >= NB || (!few_always_whole<MODE, MT>() && b0 + GRP >= n_blk)) read();
#pragma unroll
        for (int b = 0; b < GRP; ++b)
            if (!RAGGED || b0 + b < n_blk)
#pragma unroll
                for (int j = 0; j < MT; ++j) acc[j] = mfma_block<MODE>(w[j * NB + b0 + b], op[b], acc[j]);
    }
}
template <int MT>
__device__ __forceinline__ void few_stage_write(const f32x4_t (&acc)[MT], int rows, float* s) {
    constexpr int ROW = few_row(16 * MT);
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    if (lr < rows)
#pragma unroll
        for (int j = 0; j < MT; ++j) *reinterpret_cast<f32x4_t*>(s + lr * ROW + j * 16 + lk * 4) = acc[j];
}
// Polls rows 0 .. bs-1 (row_bytes apart from base) and leaves this wave's slice of them in its staging area.
template <int NB>
__device__ __forceinline__ bool few_stage_read(const unsigned char* base, unsigned row_bytes, unsigned slice_off, int n_blk, int bs, bool check,
                                               unsigned char* stage, int* err) {
    typedef FewStage<NB> S;
    constexpr int L = S::LOADS < 8 ? S::LOADS : 8;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j0 = 0; j0 < S::LOADS; j0 += L) {
        if (j0 * S::RPL >= bs) break;
        u32x4_t raw[L];
        unsigned off[L];
#pragma unroll
        for (int j = 0; j < L; ++j) {   // (a row beyond the last: the last one again)
            raw[j] = u32x4_t{0u, 0u, 0u, 0u};
            const int r = S::row(j0 + j);
            off[j] = (unsigned)min(r, bs - 1) * row_bytes + slice_off + S::src(r, n_blk);
        }
        if (L == 8 && bs - j0 * S::RPL <= 4 * S::RPL) {   // half of the loads cover the rows that are there
            u32x4_t half[4] = {raw[0], raw[1], raw[2], raw[3]};
            const unsigned off4[4] = {off[0], off[1], off[2], off[3]};
            if (!few_read<4>(base, off4, true, check, half, err)) return false;
#pragma unroll
            for (int j = 0; j < 4; ++j) *reinterpret_cast<u32x4_t*>(stage + (j0 + j) * 1024 + lane * 16) = half[j];
        } else {
            if (!few_read<L>(base, off, true, check, raw, err)) return false;
#pragma unroll
            for (int j = 0; j < L; ++j) *reinterpret_cast<u32x4_t*>(stage + (j0 + j) * 1024 + lane * 16) = raw[j];
        }
    }
    return true;
}

// Zeroes the partial sums: a wave without a share of the contraction never writes its own, and the sum over all eight
// is read without a branch (guarded reads come one after the other).
template <int COLS>
__device__ __forceinline__ void few_clear_part(float* part) {
    for (int i = threadIdx.x; i < few_part_floats(COLS); i += REC_THREADS) part[i] = 0.f;
}

// Batch sizes of 128 consecutive timesteps, two per lane: a scalar read costs no memory access.  DIR = 1: the
// window moves up, -1: down.
template <int DIR>
struct FewWindow {
    const int32_t* bs;
    int T, lo;       // cur: timesteps lo .. lo + 63; other: the 64 after (DIR = 1) or before (DIR = -1)
    int cur, other;
    __device__ __forceinline__ int fetch(int first) const {
        const int t = first + (int)(threadIdx.x & 63);
        return t >= 0 && t < T ? bs[t] : 0;
    }
    __device__ __forceinline__ void init(const int32_t* b, int n, int t) {
        bs = b; T = n;
        lo = DIR > 0 ? t : t - 63;
        cur = fetch(lo);
        other = fetch(lo + DIR * 64);
    }
    __device__ __forceinline__ int at(int t) const {
        const int d = t - lo;
        const bool in = d >= 0 && d < 64;
        return in ? __builtin_amdgcn_readlane(cur, d) : __builtin_amdgcn_readlane(other, d - DIR * 64);
    }
    __device__ __forceinline__ void advance(int t) {   // t: the timestep read next
        const int d = t - lo;
        if (d >= 0 && d < 64) return;
        cur = other;
        lo += DIR * 64;
        other = fetch(lo + DIR * 64);
    }
};

// Empties this workgroup's words of every slot (cols elements from column j0).
template <int MODE>
__device__ __forceinline__ void few_clear_ring(unsigned char* ring, int row_elems, int j0, int cols) {
    constexpr int es = (int)sizeof(typename RecGeom<MODE>::E);
    const int words = cols * es / 4;
    for (int i = threadIdx.x; i < FEW_RING * FEW_MAX * words; i += REC_THREADS)
        reinterpret_cast<unsigned*>(ring)[(size_t)(i / words) * (row_elems * es / 4) + j0 * es / 4 + i % words] = FEW_EMPTY;
}

// Up to QUAD_MAX pieces: lstm_quad.h.
constexpr int QUAD_MAX = 4;
// Forward the widths above 512 units, with 32 units per workgroup, run it up to 2 pieces, 3 and 4 with a thread per (piece, unit): with four lanes all
// eight waves own a share of the cell update, two per SIMD, where two waves do with a thread.  us per forward pass of two layers over 256 timesteps of 4
// pieces per group, four lanes -> a thread: 576 units 409 -> 403, 768 429 -> 424, 1024 458 -> 442; one layer of 576 378 -> 367.  (Backward the same
// made the consumer's timesteps longer: 1024 units 746 -> 922.)
template <int MT> constexpr int QUAD_FWD = MT == 8 ? 2 : QUAD_MAX;
template <int MODE, int MT, int NB> struct FewFwd;
template <int MODE, int MT, int NB> struct FewBwd;
template <int MODE, int MT, int NB, int PIPE>
__device__ __forceinline__ bool quad_fwd(FewFwd<MODE, MT, NB>& s, const RecFwdArgs& a, const PieceSet& ps, int rank, int* flags, unsigned char* ring, const PipeLink& pl, int& t,
                         int T);
template <int MODE, int MT, int NB, int PIPE>
__device__ __forceinline__ bool quad_bwd(FewBwd<MODE, MT, NB>& s, const RecBwdArgs& a, const PieceSet& ps, int rank, unsigned char* ring, const PipeLink& pl, int& t, int T,
                         int t_stop);

// ---- forward ------------------------------------------------------------------------------------------------
// What a group's workgroup carries through its timesteps with few pieces.
template <int MODE, int MT, int NB>
struct FewFwd {
    f32x4_t w[MT * NB];
    FewWindow<1> win;
    int bs_a, bs_b;              // alive pieces of all groups at t, t + 1
    int base, base_prev;         // first row of timesteps t, t - 1
    int t0;                      // first timestep of this form
    int c_wait;                  // consumer: the chunk it has to wait for next
    bool ready;                  // that chunk has been seen finished
    int have;                    // its counter, requested a timestep ago
    int n_slices, slice, n_blk;  // slices with work, this wave's slice, its operand blocks
    float c;                     // this thread's cell state
    f32x4_t z;                   // its input projection of timestep t
    f32x4_t s_g; float s_c, s_h; unsigned s_w;   // results of the timestep before, not yet stored
    int* fail;                   // LDS: a wait was abandoned; the counter of a chunk
    float* part;                 // LDS
};

// A word at `rows` + `off` bytes of an array (`rows`: the same for all lanes).  Consumers, which run out of scalar registers, store through a
// pointer: two of them instead of a buffer's four (40 -> 16 v_readlane in two timesteps at 256 units; us per forward pass of two layers of
// 256 units over 256 timesteps of 8 pieces per group 363 -> 347); one layer alone is faster with buffers (512 units 366 -> 360).
template <int PIPE>
__device__ __forceinline__ void few_store(void* array, unsigned rows, unsigned off, unsigned v) {
    if constexpr ((PIPE & PIPE_CONSUMER) != 0) {
        __attribute__((address_space(1))) unsigned char* at = (__attribute__((address_space(1))) unsigned char*)array + rows;
        *(__attribute__((address_space(1))) unsigned*)(at + off) = v;
    } else {
        __builtin_amdgcn_raw_buffer_store_b32(v, __builtin_amdgcn_make_buffer_rsrc(array, 0, (int)0x80000000u, 0x00020000), off, rows, 0);
    }
}
template <int MODE, int MT, int NB, int PIPE>
__device__ __forceinline__ void few_fwd_store(const FewFwd<MODE, MT, NB>& s, const RecFwdArgs& a, const PieceSet& ps, int j0, int bs_prev,
                                              int base, int bs) {
    typedef typename RecGeom<MODE>::E E;
    constexpr int UH = 4 * MT, es = (int)sizeof(E);
    const int m = threadIdx.x / UH, u = threadIdx.x % UH, n = m * ps.X + ps.x, H = a.H;
    if (m >= bs_prev) return;
    constexpr int WHOLE = (int)0x80000000u;
    const unsigned col = (unsigned)(n * H + j0 + u);
    const unsigned so = (unsigned)s.base_prev * (unsigned)H;   // elements of an [M, H] array
    const __amdgpu_buffer_rsrc_t rs_g = __builtin_amdgcn_make_buffer_rsrc(a.gates, 0, WHOLE, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, s.s_g), rs_g, col * 16u, so * 16u, 0);
    few_store<PIPE>(a.c, so * 4u, col * 4u, __float_as_uint(s.s_c));
    if (!(PIPE & PIPE_PRODUCER)) few_store<PIPE>(a.hout, so * 4u, col * 4u, __float_as_uint(s.s_h));
    if (MODE == MODE_F32 || (u & 1) == 0) {   // operand type: a bf16 pair per even lane
        if (m < bs) few_store<PIPE>(a.hprev, (unsigned)base * (unsigned)(H * es), col * es, s.s_w);
        if (PIPE & PIPE_PRODUCER) {   // written through: input of the workers' GEMM
            const __amdgpu_buffer_rsrc_t rs_hc = __builtin_amdgcn_make_buffer_rsrc(a.hcopy, 0, WHOLE, 0x00020000);
            __builtin_amdgcn_raw_buffer_store_b32(s.s_w, rs_hc, col * es, so * es, 17);
        }
    }
}

// Runs timesteps while more than down_to (and at most P) pieces are alive.  P = 16: rows through LDS; P = 4: polled into operand registers, two
// buffers of partial sums, sums and gates in the order of lstm_quad.h.  False: a wait was abandoned.
template <int MODE, int MT, int NB, int P, int PIPE>
__device__ __forceinline__ bool few_fwd_phase(FewFwd<MODE, MT, NB>& s, const RecFwdArgs& a, const PieceSet& ps, int rank, int* flags,
                                              unsigned char* ring, const PipeLink& pl, int& t, int T, int down_to) {
    typedef typename RecGeom<MODE>::E E;
    constexpr int es = (int)sizeof(E);
    constexpr int UH = 4 * MT, COLS = 16 * MT, ROW = few_row(COLS);
    constexpr bool STAGED = P > 4;
    constexpr int BPL = STAGED ? 1 : 16 / P, L = STAGED ? 1 : (NB + BPL - 1) / BPL;
    const int X = ps.X, x = ps.x, H = a.H;
    const int tid = threadIdx.x, lr = tid & 15, lk = (tid & 63) >> 4;
    const int piece = lr / BPL, blk = lr % BPL;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = tid / UH, u = tid % UH, j0 = rank * UH;
    const unsigned slice_off = (unsigned)(s.slice * NB) * 64u;                          // bytes: an operand block is 64
    const unsigned slot = (unsigned)few_slot_bytes(MODE, H);
    const unsigned w_off = (unsigned)(m * H + j0 + u) * es;   // where this thread's value goes inside a slot
    const bool polls = s.slice < s.n_slices;
    unsigned char* stage = reinterpret_cast<unsigned char*>(s.part + few_part_floats(COLS)) + wave * few_stage_bytes(NB);
    const unsigned k_off = slice_off + (unsigned)(lk * s.n_blk + blk) * 16u;   // this lane's first 16 bytes inside a row
    unsigned off[L];
    few_offsets<L, BPL>(off, (unsigned)(piece * H) * es + k_off, blk, s.n_blk);
    u32x4_t raw[L];
#pragma unroll
    for (int j = 0; j < L; ++j) raw[j] = u32x4_t{0u, 0u, 0u, 0u};
    bar_lds();   // (the partial sums of the phase before have been read)
    few_clear_part<COLS>(s.part);
    bar_lds();
    constexpr int WHOLE = (int)0x80000000u;
    const __amdgpu_buffer_rsrc_t rs_g = __builtin_amdgcn_make_buffer_rsrc(a.gates, 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_ring = __builtin_amdgcn_make_buffer_rsrc(ring, 0, (int)(FEW_RING * slot), 0x00020000);

    auto step = [&](f32x4_t& z, f32x4_t& z_next) __attribute__((always_inline)) -> bool {
        const int bs = grp_count(s.bs_a, ps), bs_next = t + 1 < T ? grp_count(s.bs_b, ps) : 0;
        const int base_next = s.base + s.bs_a;
        s.win.advance(t + 2);
        if ((PIPE & PIPE_CONSUMER) && t + 1 < T && t + 1 == s.c_wait * pl.ct) {
            if (!s.ready && !pipe_wait_chunk(pl, s.c_wait, a.err)) return false;
            ++s.c_wait;
            s.ready = false;
        }
        bool ok = true;
        if (t == s.t0) {
            // the rows were written under the flag protocol (initial states, or the timestep before with more pieces)
            if (!rec_wait(flags, a.G, t + 1, a.err)) return false;
            if ((PIPE & PIPE_PRODUCER) && rank == 0 && tid == 0 && t > 0) st_agent(pl.progress, t);
            if (polls) {
                const unsigned char* rows = reinterpret_cast<const unsigned char*>(static_cast<const E*>(a.hprev) + (size_t)(s.base + x) * H);
                if constexpr (STAGED) {
                    few_stage_read<NB>(rows, (unsigned)(X * H) * es, slice_off, s.n_blk, bs, false, stage, a.err);
                } else {
                    unsigned first[L];
                    few_offsets<L, BPL>(first, (unsigned)(piece * X * H) * es + k_off, blk, s.n_blk);
                    few_read<L>(rows, first, piece < bs && blk < s.n_blk, false, raw, a.err);
                }
            }
        } else if (polls) {
            const unsigned char* rows = ring + (unsigned)((t - 1) & (FEW_RING - 1)) * slot;
            if constexpr (STAGED) ok = few_stage_read<NB>(rows, (unsigned)H * es, slice_off, s.n_blk, bs, true, stage, a.err);
            else ok = few_read<L>(rows, off, piece < bs && blk < s.n_blk, true, raw, a.err);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (also: this wave's stores of two timesteps ago have completed)
        few_touch(z);
        few_touch(s.win.cur);
        few_touch(s.win.other);
        if (PIPE & PIPE_CONSUMER) few_touch(s.have);
        if (!ok) *s.fail = 1;
        const int bs_c = s.win.at(t + 2);
        // off the critical path: results of the timestep before, the input projection of the next one
        if (m < bs_next)
            z_next = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs_g, (unsigned)((m * X + x) * H + j0 + u) * 16u,
                                                                                        (unsigned)base_next * (unsigned)H * 16u, 0));
        // A look at the chunk that the next timestep asks for: usually finished, which saves that wait its round trip.  Its
        // counter was requested a timestep earlier (a load waited for in the timestep that requests it, under a condition,
        // makes the compiler wait in every timestep).
        const bool look = (PIPE & PIPE_CONSUMER) && t + 2 < T && t + 2 == s.c_wait * pl.ct;
        if (PIPE & PIPE_CONSUMER) {
            if (look && tid == REC_THREADS - 1) s.fail[1] = s.have;
            if (look) s.have = 0;
            if (t + 3 < T && t + 3 == s.c_wait * pl.ct && tid == REC_THREADS - 1) s.have = ld_agent(&pl.done[s.c_wait]);
        }
        if (t > s.t0) few_fwd_store<MODE, MT, NB, PIPE>(s, a, ps, j0, grp_count(s.base - s.base_prev, ps), s.base, bs);
        float* part = s.part + (STAGED ? 0 : (t & 1) * (REC_WAVES * P * ROW));
        if (polls) {
            f32x4_t acc[MT];
#pragma unroll
            for (int j = 0; j < MT; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if constexpr (STAGED) {
                few_stage_product<MODE, MT, NB, false>(s.w, stage, s.part + 16 * MT, s.n_blk, acc, [] {});
                few_stage_write<MT>(acc, bs, part + s.slice * (P * ROW));
            } else {
                few_product<MODE, MT, NB, P, L>(s.w, raw, bs, s.n_blk, acc);
                few_write<MODE, MT, P>(acc, bs, part + s.slice * (P * ROW));
            }
        }
        bar_lds();
        const int failed = *s.fail;   // (looked at after the publication: its read is not waited for by itself)
        if (look) s.ready = __builtin_amdgcn_readfirstlane(s.fail[1]) >= few_scalar(pl.need);
        // Every workgroup has published the rows of timestep t-1, which it did after its stores for timestep t-3 had
        // completed (they are issued in timestep t-2 and waited for in timestep t-1).
        if ((PIPE & PIPE_PRODUCER) && rank == 0 && tid == REC_THREADS - 1 && t - 2 > s.t0) st_agent(pl.progress, t - 2);
        if (m < bs) {
            f32x4_t q = z, o[REC_WAVES];
            const float* p = part + m * ROW + u * 4;
#pragma unroll
            for (int k = 0; k < REC_WAVES; ++k) o[k] = *reinterpret_cast<const f32x4_t*>(p + k * (P * ROW));
            if constexpr (STAGED) {
#pragma unroll
                for (int k = 0; k < REC_WAVES; ++k) {
                    q[0] += o[k][0]; q[1] += o[k][1]; q[2] += o[k][2]; q[3] += o[k][3];
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] += ((o[0][i] + o[1][i]) + (o[2][i] + o[3][i])) + ((o[4][i] + o[5][i]) + (o[6][i] + o[7][i]));
            }
            const float gi = sigmoidf_(q[0]), gf = sigmoidf_(q[1]), gg = tanhf_(q[2]), go = sigmoidf_(q[3]);
            s.c = gf * s.c + gi * gg;
            const float h = go * tanhf_(s.c);
            s.s_g = f32x4_t{gi, gf, gg, go};
            s.s_c = s.c;
            s.s_h = h;
            if constexpr (MODE == MODE_BF16) {
                const unsigned b = to_bf16_finite(h);
                s.s_w = few_word(b | (few_dpp<0xb1>(b) << 16));   // (quad_perm 1,0,3,2: the neighbour's value)
            } else {
                s.s_w = few_word(__float_as_uint(h));
            }
            if ((MODE == MODE_F32 || (u & 1) == 0) && m < bs_next) {
                __builtin_amdgcn_raw_buffer_store_b32(s.s_w, rs_ring, w_off, (unsigned)(t & (FEW_RING - 1)) * slot, 0);
                __builtin_amdgcn_raw_buffer_store_b32(FEW_EMPTY, rs_ring, w_off, (unsigned)((t + 2) & (FEW_RING - 1)) * slot, 0);
            }
        }
        if (__builtin_amdgcn_readfirstlane(failed)) return false;
        if (STAGED) bar_lds();   // (one buffer of partial sums: it has been read)
        s.base_prev = s.base;
        s.base = base_next;
        s.bs_a = s.bs_b;
        s.bs_b = bs_c;
        ++t;
        return true;
    };
    // (two steps per iteration: a prefetched value is used where it was loaded, a move would wait for the load)
    f32x4_t z2 = s.z;
    while (t < T && grp_count(s.bs_a, ps) > down_to) {
        if (!step(s.z, z2)) return false;
        if (!(t < T && grp_count(s.bs_a, ps) > down_to)) {
            s.z = z2;
            break;
        }
        if (!step(z2, s.z)) return false;
    }
    return true;
}

template <typename A> using few_args_t = const A __attribute__((address_space(4)))*;
struct FewLink { PieceSet ps; PipeLink pl; };
template <int PIPE>
__device__ __forceinline__ FewLink few_link(int x, int cap, int id, int* progress, int* done, int need, int ct) {
    FewLink l;
    l.ps.x = few_scalar(x);
    l.ps.X = PIPE == PIPE_NONE ? REC_GROUPS : 1;   // (PieceSet: dealt round-robin, or a block)
    l.ps.cap = few_scalar(cap);
    l.ps.id = few_scalar(id);
    l.pl.progress = few_scalar(progress);
    l.pl.done = few_scalar(done);
    few_away(l.pl.progress);
    few_away(l.pl.done);
    l.pl.need = few_scalar(need);
    few_away(l.pl.need);
    l.pl.ct = few_scalar(ct);
    l.pl.T = 0;
    return l;
}

// Timesteps [t0, T): at most FEW_MAX pieces of the group are alive.  The rows of h_{t0-1} are in hprev, announced by
// flag value t0 + 1.  lds: where the dynamic LDS begins.  False: a wait was abandoned.
template <int MODE, int MT, int PIPE>
__device__ __forceinline__ bool few_fwd(few_args_t<RecFwdArgs> args, int x_, int cap_, int id_, int rank_, int t0_, int T_, int* flags_, int* progress_,
                                                  int* done_, int need_, int ct_, int c_wait_, unsigned lds_) {
    const FewLink link = few_link<PIPE>(x_, cap_, id_, progress_, done_, need_, ct_);
    const PieceSet& ps = link.ps;
    const PipeLink& pl = link.pl;
    const int rank = few_scalar(rank_), t0 = few_scalar(t0_), T = few_scalar(T_), c_wait = few_scalar(c_wait_);
    int* flags = few_scalar(flags_);
    few_away(flags);
    RecFwdArgs a = *(const RecFwdArgs*)few_scalar(args);
    few_global(a.batch_sizes); few_global(a.t_off); few_global(a.gates); few_global(a.c); few_global(a.hout);
    few_away(a.c0); few_away(a.err); few_away(a.batch_sizes); few_away(a.seq_cap);
    a.hprev = (void*)(__attribute__((address_space(1))) void*)a.hprev;
    a.whh = (const void*)(__attribute__((address_space(1))) const void*)a.whh;
    a.ring = (void*)(__attribute__((address_space(1))) void*)a.ring;
    unsigned char* ring = static_cast<unsigned char*>(a.ring) + ps.id * few_ring_bytes(MODE, a.H);
    unsigned char* smem = (unsigned char*)(__attribute__((address_space(3))) unsigned char*)few_scalar(lds_);
    typedef typename RecGeom<MODE>::E E;
    constexpr int KBLK = RecGeom<MODE>::KBLK, VEC = RecGeom<MODE>::VEC, UH = 4 * MT;
    constexpr int NB = FewBlocks<MODE, MT == 8>::fwd;
    __shared__ int s_fail[2];
    const int H = a.H, X = ps.X, x = ps.x;
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    const int m = tid / UH, u = tid % UH, j0 = rank * UH;
    FewFwd<MODE, MT, NB> s;
    s.fail = s_fail;
    s.part = reinterpret_cast<float*>(smem);
    if (tid == 0) s_fail[0] = 0;
    bar_lds();   // (LDS of the other form has been read)
    const int blocks = H / KBLK;
    s.n_slices = (blocks + NB - 1) / NB;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // which slice a wave takes rotates with the rank: the workgroups poll the same rows at the same moment
    s.slice = s.n_slices == REC_WAVES ? (wave + rank) % REC_WAVES : wave;
    s.n_blk = min(NB, blocks - s.slice * NB);
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const E* wrow = static_cast<const E*>(a.whh) + ((size_t)j0 * 4 + j * 16 + lr) * H + (s.slice * NB * 4 + lk * s.n_blk) * VEC;
#pragma unroll
        for (int b = 0; b < NB; ++b)
            s.w[j * NB + b] = b < s.n_blk ? *reinterpret_cast<const f32x4_t*>(wrow + b * VEC) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    // (a use of the registers: the loads are complete before the time loop, see rec_fwd_body)
#pragma unroll
    for (int i = 0; i < MT * NB; ++i) asm volatile("" : "+v"(s.w[i]));
    s.t0 = t0;
    s.c_wait = c_wait;
    s.ready = false;
    s.have = 0;
    s.win.init(a.batch_sizes, T, t0);
    s.bs_a = s.win.at(t0);
    s.bs_b = s.win.at(t0 + 1);
    s.base = a.t_off[t0];
    s.base_prev = t0 > 0 ? a.t_off[t0 - 1] : 0;
    s.c = 0.f;
    s.z = s.s_g = f32x4_t{0.f, 0.f, 0.f, 0.f};
    s.s_c = s.s_h = 0.f;
    s.s_w = 0;
    if (m < grp_count(s.bs_a, ps)) {
        const int n = m * X + x;
        s.z = *reinterpret_cast<const f32x4_t*>(a.gates + ((size_t)s.base + n) * 4 * H + (size_t)(j0 + u) * 4);
        if (t0 > 0) s.c = a.c[((size_t)s.base_prev + n) * H + j0 + u];
        else if (a.c0 && n < a.seq_cap) s.c = a.c0[(size_t)n * H + j0 + u];
    }
    int t = t0;
    if (!few_fwd_phase<MODE, MT, NB, 16, PIPE>(s, a, ps, rank, flags, ring, pl, t, T, QUAD_MAX)) return false;
    constexpr int QUAD = QUAD_FWD<MT>;
    if constexpr (QUAD < QUAD_MAX)
        if (t < T && grp_count(s.bs_a, ps) > QUAD && !few_fwd_phase<MODE, MT, NB, QUAD_MAX, PIPE>(s, a, ps, rank, flags, ring, pl, t, T, QUAD)) return false;
    if (t > t0) few_fwd_store<MODE, MT, NB, PIPE>(s, a, ps, j0, grp_count(s.base - s.base_prev, ps), s.base, t < T ? grp_count(s.bs_a, ps) : 0);
    if (t < T && !quad_fwd<MODE, MT, NB, PIPE>(s, a, ps, rank, flags, ring, pl, t, T)) return false;
    if (PIPE & PIPE_PRODUCER) rec_publish(few_scalar(flags), rank, T + 1);
    return true;
}

// ---- backward -----------------------------------------------------------------------------------------------
struct FewSaved {
    f32x4_t g;                 // activated gates
    float c_prev, dh_above;
    float c;                   // only loaded for a piece whose last timestep this is
};
template <int MODE, int MT, int NB>
struct FewBwd {
    f32x4_t w[MT * NB];
    FewWindow<-1> win;
    int bs_up, bs_t, bs_m1, bs_m2;   // alive pieces of all groups at t + 1, t, t - 1, t - 2
    int base;                        // first row of timestep t
    int c_wait;                      // consumer: the lowest chunk it has waited for
    bool ready;                      // the chunk below has been seen finished
    int have;                        // its counter, requested a timestep ago
    int n_slices, slice, n_blk;
    FewSaved sv, sv2;                // what the forward pass saved for timesteps t and t - 1
    float dh, dc, c;                 // carried gradients, cell state of timestep t
    float db[4];                     // sums of the gate gradients of this thread's unit
    int* fail;
    float* part;
};

// Requests the saved activations of timestep q (rows from base_q, of timestep q - 1 from base_q1).
__device__ __forceinline__ void few_load_saved(FewSaved& sv, const RecBwdArgs& a, int m, int n, int j, int q, int bs_q, int bs_q_up, int base_q,
                                               int base_q1) {
    if (m >= bs_q) return;
    constexpr int WHOLE = (int)0x80000000u;
    const unsigned H = (unsigned)a.H, col = (unsigned)n * H + (unsigned)j, so = (unsigned)base_q * H;
    const __amdgpu_buffer_rsrc_t rs_g = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.gates), 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_c = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.c), 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.dh_above), 0, WHOLE, 0x00020000);
    sv.g = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs_g, col * 16u, so * 16u, 0));
    sv.dh_above = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_a, col * 4u, so * 4u, 0));
    if (q > 0) sv.c_prev = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_c, col * 4u, (unsigned)base_q1 * H * 4u, 0));
    else sv.c_prev = (a.c0 && n < a.seq_cap) ? a.c0[(size_t)n * a.H + j] : 0.f;
    if (bs_q > bs_q_up && m >= bs_q_up) sv.c = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_c, col * 4u, so * 4u, 0));
}

// Runs timesteps t, t-1, ... >= t_stop while at most FEW_MAX pieces are alive.  False: a wait was abandoned.
template <int MODE, int MT, int NB, int PIPE>
__device__ __forceinline__ bool few_bwd_phase(FewBwd<MODE, MT, NB>& s, const RecBwdArgs& a, const PieceSet& ps, int rank, unsigned char* ring,
                                              const PipeLink& pl, int& t, int T, int t_stop) {
    typedef typename RecGeom<MODE>::E E;
    constexpr int es = (int)sizeof(E);
    constexpr int UH = 16 * MT, ROW = few_row(UH);
    const int X = ps.X, x = ps.x, H = a.H, K = 4 * H;
    const int tid = threadIdx.x;
    const int m = tid / UH, u = tid % UH, j0 = rank * UH, n = m * X + x, j = j0 + u;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned slice_off = (unsigned)(s.slice * NB) * 64u;
    const unsigned slot = (unsigned)few_slot_bytes(MODE, K);
    const unsigned w_off = (unsigned)(m * K + j * 4) * es;
    const bool polls = s.slice < s.n_slices;
    unsigned char* stage = reinterpret_cast<unsigned char*>(s.part + few_part_floats(UH)) + wave * few_stage_bytes(NB);
    bar_lds();   // (the partial sums of the phase before have been read)
    few_clear_part<UH>(s.part);
    bar_lds();
    constexpr int WHOLE = (int)0x80000000u;
    const __amdgpu_buffer_rsrc_t rs_dz = __builtin_amdgcn_make_buffer_rsrc(a.dz, 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_ring = __builtin_amdgcn_make_buffer_rsrc(ring, 0, (int)(FEW_RING * slot), 0x00020000);
    typedef unsigned wv_t __attribute__((ext_vector_type(MODE == MODE_BF16 ? 2 : 4)));
    auto store = [&](wv_t v, __amdgpu_buffer_rsrc_t rs, unsigned off, unsigned so, auto aux) {
        if constexpr (MODE == MODE_BF16) __builtin_amdgcn_raw_buffer_store_b64(v, rs, off, so, decltype(aux)::value);
        else __builtin_amdgcn_raw_buffer_store_b128(v, rs, off, so, decltype(aux)::value);
    };

    // sv: what the forward pass saved for timestep t; other: for timestep t - 1, requested a timestep ago
    auto step = [&](FewSaved& sv, FewSaved& other) __attribute__((always_inline)) -> bool {
        s.win.advance(t - 3);
        const int bs = grp_count(s.bs_t, ps), bs_up = t + 1 < T ? grp_count(s.bs_up, ps) : 0;
        wv_t word;
#pragma unroll
        for (int i = 0; i < (MODE == MODE_BF16 ? 2 : 4); ++i) word[i] = 0u;
        // A. gate gradients of this thread's (piece, unit)
        if (m < bs) {
            const bool carried = m < bs_up;
            const float gi = sv.g[0], gf = sv.g[1], gg = sv.g[2], go = sv.g[3];
            const float dh = carried ? sv.dh_above + s.dh : sv.dh_above;
            const float tc = tanhf_(carried ? s.c : sv.c);
            const float dc = (carried ? s.dc : 0.f) + dh * go * (1.f - tc * tc);
            const float dzi = dc * gg * gi * (1.f - gi), dzf = dc * sv.c_prev * gf * (1.f - gf), dzg = dc * gi * (1.f - gg * gg),
                        dzo = dh * tc * go * (1.f - go);
            if constexpr (MODE == MODE_BF16) {
                word[0] = few_word((unsigned)to_bf16_finite(dzi) | ((unsigned)to_bf16_finite(dzf) << 16));
                word[1] = few_word((unsigned)to_bf16_finite(dzg) | ((unsigned)to_bf16_finite(dzo) << 16));
            } else {
                word[0] = few_word(__float_as_uint(dzi)); word[1] = few_word(__float_as_uint(dzf));
                word[2] = few_word(__float_as_uint(dzg)); word[3] = few_word(__float_as_uint(dzo));
            }
            if (t > 0) store(word, rs_ring, w_off, (unsigned)(t & (FEW_RING - 1)) * slot, FewIdx<0>{});
            s.db[0] += dzi; s.db[1] += dzf; s.db[2] += dzg; s.db[3] += dzo;
            s.dc = dc * gf;
            s.c = sv.c_prev;
        }
        const unsigned so_dz = (unsigned)s.base * (unsigned)(K * es);
        if (t == 0) {   // nothing is carried before the first timestep
            if (m < bs) store(word, rs_dz, (unsigned)(n * K + j * 4) * es, so_dz, FewIdx<(PIPE & PIPE_PRODUCER) ? 17 : 0>{});
            --t;
            return true;
        }
        if ((PIPE & PIPE_CONSUMER) && t >= 2 && t - 2 < s.c_wait * pl.ct) {
            --s.c_wait;
            if (!s.ready && !pipe_wait_chunk(pl, s.c_wait, a.err)) return false;
            s.ready = false;
        }
        // B. dh carried to t-1: dh[piece][k] = sum_q dz[piece][q] * W_hh[q][k] for this workgroup's columns k
        const unsigned char* src = ring + (unsigned)(t & (FEW_RING - 1)) * slot;
        bool ok = true;
        if (polls) ok = few_stage_read<NB>(src, (unsigned)K * es, slice_off, s.n_blk, bs, true, stage, a.err);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (also: this wave's dz rows of timestep t+1 have completed)
        few_touch(other.g);
        few_touch(other.c_prev);
        few_touch(other.dh_above);
        few_touch(other.c);
        few_touch(s.win.cur);
        few_touch(s.win.other);
        if (PIPE & PIPE_CONSUMER) few_touch(s.have);
        if (!ok) *s.fail = 1;
        const int bs_m3 = s.win.at(t - 3);
        // off the critical path: the dz rows of this timestep, the saved activations of timestep t-2
        if (m < bs) store(word, rs_dz, (unsigned)(n * K + j * 4) * es, so_dz, FewIdx<(PIPE & PIPE_PRODUCER) ? 17 : 0>{});
        if (t >= 2) {
            const int base_2 = s.base - s.bs_m1 - s.bs_m2;
            few_load_saved(sv, a, m, n, j, t - 2, grp_count(s.bs_m2, ps), grp_count(s.bs_m1, ps), base_2, base_2 - bs_m3);
        }
        // a look at the chunk that the next timestep asks for, see the forward loop
        const bool look = (PIPE & PIPE_CONSUMER) && t >= 3 && t - 3 == s.c_wait * pl.ct - 1;
        if (PIPE & PIPE_CONSUMER) {
            if (look && tid == REC_THREADS - 1) s.fail[1] = s.have;
            if (look) s.have = 0;
            if (t >= 4 && t - 4 == s.c_wait * pl.ct - 1 && tid == REC_THREADS - 1) s.have = ld_agent(&pl.done[s.c_wait - 1]);
        }
        float* part = s.part;
        if (polls) {
            f32x4_t acc[MT];
#pragma unroll
            for (int i = 0; i < MT; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            few_stage_product<MODE, MT, NB, false>(s.w, stage, s.part + 16 * MT, s.n_blk, acc, [] {});
            few_stage_write<MT>(acc, bs, part + s.slice * (16 * ROW));
        }
        bar_lds();
        const int failed = *s.fail;
        if (look) s.ready = __builtin_amdgcn_readfirstlane(s.fail[1]) >= few_scalar(pl.need);
        // Every workgroup has published the rows of timestep t, which it did after its dz rows of timestep t+2 had
        // completed (they are stored in that timestep and waited for in timestep t+1).
        if ((PIPE & PIPE_PRODUCER) && rank == 0 && tid == REC_THREADS - 1 && t + 2 < T) st_agent(pl.progress, T - (t + 2));
        if (m < bs) {
            float q = 0.f, o[REC_WAVES];
            const float* p = part + m * ROW + u;
#pragma unroll
            for (int k = 0; k < REC_WAVES; ++k) o[k] = p[k * (16 * ROW)];
#pragma unroll
            for (int k = 0; k < REC_WAVES; ++k) q += o[k];
            s.dh = q;
            store(wv_t(FEW_EMPTY), rs_ring, w_off, (unsigned)((t + 1) & (FEW_RING - 1)) * slot, FewIdx<0>{});
        }
        if (__builtin_amdgcn_readfirstlane(failed)) return false;
        bar_lds();   // (one buffer of partial sums: it has been read)
        s.base -= s.bs_m1;
        s.bs_up = s.bs_t;
        s.bs_t = s.bs_m1;
        s.bs_m1 = s.bs_m2;
        s.bs_m2 = bs_m3;
        --t;
        return true;
    };
    while (t >= t_stop) {
        if (!step(s.sv, s.sv2)) return false;
        if (t < t_stop) break;
        if (!step(s.sv2, s.sv)) return false;
    }
    return true;
}

// What the few-pieces form leaves of a thread's (piece, unit): the carried gradients, the sums of its gate gradients; and the
// lowest chunk waited for.
struct FewBwdOut {
    float dh, dc, db[4];
    int c_wait;
    bool ok;   // false: a wait was abandoned
};
// Timesteps T-1 .. t_stop: at most FEW_MAX pieces of the group are alive.
template <int MODE, int MT, int PIPE>
__device__ __forceinline__ FewBwdOut few_bwd(few_args_t<RecBwdArgs> args, int x_, int cap_, int id_, int rank_, int t_stop_, int T_, int* progress_,
                                                       int* done_, int need_, int ct_, int c_wait_, unsigned lds_) {
    const FewLink link = few_link<PIPE>(x_, cap_, id_, progress_, done_, need_, ct_);
    const PieceSet& ps = link.ps;
    const PipeLink& pl = link.pl;
    const int rank = few_scalar(rank_), t_stop = few_scalar(t_stop_), T = few_scalar(T_), c_wait = few_scalar(c_wait_);
    RecBwdArgs a = *(const RecBwdArgs*)few_scalar(args);
    few_global(a.batch_sizes); few_global(a.t_off); few_global(a.gates); few_global(a.c); few_global(a.dh_above);
    few_away(a.c0); few_away(a.err); few_away(a.batch_sizes); few_away(a.seq_cap);
    a.dz = (void*)(__attribute__((address_space(1))) void*)a.dz;
    a.whhT = (const void*)(__attribute__((address_space(1))) const void*)a.whhT;
    a.ring = (void*)(__attribute__((address_space(1))) void*)a.ring;
    unsigned char* ring = static_cast<unsigned char*>(a.ring) + ps.id * few_ring_bytes(MODE, 4 * a.H);
    unsigned char* smem = (unsigned char*)(__attribute__((address_space(3))) unsigned char*)few_scalar(lds_);
    const FewBwdOut gave_up = {};
    typedef typename RecGeom<MODE>::E E;
    constexpr int KBLK = RecGeom<MODE>::KBLK, VEC = RecGeom<MODE>::VEC, UH = 16 * MT;
    constexpr int NB = FewBlocks<MODE, MT == 2>::bwd, LOW = 16 / NB;
    __shared__ int s_fail[2];
    const int H = a.H, K = 4 * H, X = ps.X, x = ps.x;
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    const int m = tid / UH, j = rank * UH + tid % UH, n = m * X + x;
    FewBwd<MODE, MT, NB> s;
    s.fail = s_fail;
    s.part = reinterpret_cast<float*>(smem);
    if (tid == 0) s_fail[0] = 0;
    bar_lds();
    const int blocks = K / KBLK;
    s.n_slices = (blocks + NB - 1) / NB;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    s.slice = s.n_slices == REC_WAVES ? (wave + rank) % REC_WAVES : wave;
    s.n_blk = min(NB, blocks - s.slice * NB);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const E* wrow = static_cast<const E*>(a.whhT) + ((size_t)rank * UH + i * 16 + lr) * K + (s.slice * NB * 4 + lk * s.n_blk) * VEC;
#pragma unroll
        for (int b = 0; b < NB; ++b)
            s.w[i * NB + b] = b < s.n_blk ? *reinterpret_cast<const f32x4_t*>(wrow + b * VEC) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < MT * NB; ++i) asm volatile("" : "+v"(s.w[i]));
    s.c_wait = c_wait;
    s.ready = false;
    s.have = 0;
    s.win.init(a.batch_sizes, T, T - 1);
    s.bs_up = 0;
    s.bs_t = s.win.at(T - 1);
    s.bs_m1 = s.win.at(T - 2);
    s.bs_m2 = s.win.at(T - 3);
    s.base = a.t_off[T - 1];
    s.dh = s.dc = s.c = 0.f;
    s.sv.g = s.sv2.g = f32x4_t{0.f, 0.f, 0.f, 0.f};
    s.sv.c_prev = s.sv.dh_above = s.sv.c = s.sv2.c_prev = s.sv2.dh_above = s.sv2.c = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s.db[i] = 0.f;
    int t = T - 1;
    if (!quad_bwd<MODE, MT, NB, PIPE>(s, a, ps, rank, ring, pl, t, T, t_stop)) return gave_up;
    if (t >= t_stop) {
        if (PIPE & PIPE_CONSUMER)
            while (s.c_wait > 0 && t - 1 < s.c_wait * pl.ct) {
                --s.c_wait;
                if (!pipe_wait_chunk(pl, s.c_wait, a.err)) return gave_up;
                s.ready = false;
            }
        const int base_1 = s.base - s.bs_m1;
        few_load_saved(s.sv, a, m, n, j, t, grp_count(s.bs_t, ps), t + 1 < T ? grp_count(s.bs_up, ps) : 0, s.base, base_1);
        if (t > 0) few_load_saved(s.sv2, a, m, n, j, t - 1, grp_count(s.bs_m1, ps), grp_count(s.bs_t, ps), base_1, base_1 - s.bs_m2);
        few_touch(s.sv.g); few_touch(s.sv.c_prev); few_touch(s.sv.dh_above); few_touch(s.sv.c);   // (the loads are complete before the loop)
        few_touch(s.sv2.g); few_touch(s.sv2.c_prev); few_touch(s.sv2.dh_above); few_touch(s.sv2.c);
        if (!few_bwd_phase<MODE, MT, NB, PIPE>(s, a, ps, rank, ring, pl, t, T, t_stop)) return gave_up;
    }
    return FewBwdOut{s.dh, s.dc, {s.db[0], s.db[1], s.db[2], s.db[3]}, s.c_wait, true};
}

}  // namespace ver

#include "lstm_quad.h"
#include "lstm_many.h"
