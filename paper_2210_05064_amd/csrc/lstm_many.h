// The time loops while a group has more than 16 alive pieces (included by lstm_few.h, whose exchange they use).  gfx950 only.
//
// The alive pieces of a timestep are worked through 16 at a time.  Such a unit, (timestep, tile of 16 pieces), depends on the same tile
// of the timestep before, which is at least one unit back, so that no unit has to wait for the exchange: a unit's rows, its
// input projections and its cell states are requested while the unit before is worked on.  The rows go from the ring straight into
// LDS (forward two areas per wave in turn); an operand that is still empty when it is read (lstm_few.h) is requested again.
// Memory operations of a wave complete in order, and a unit issues the same number of stores behind the next unit's loads whatever its
// pieces (those without one go beyond the buffers), so that the wait for a unit's loads leaves the stores of the unit before in flight.
// What is published in a unit is published after the stores of the unit before the last one have completed.  So whoever has the rows of a timestep
// knows that the rows of the timestep before are complete in memory, and that the words that were emptied two units earlier are.
// Bound by LDS (192 KB per unit at H = 1024, 0.64 us), the MFMAs (0.43 us) and the gates, one after the other in a wave.
// us per timestep of one layer with 17 / 32 / 64 alive pieces per group, flag form of lstm_rec.h -> this form: bf16, 1024 units 4.5 / 5.3 / 11.7 ->
// 3.5 / 4.4 / 8.2, 576 4.9 / 5.4 / 11.2 -> 3.2 / 3.7 / 6.7, 512 3.2 / 3.9 / 6.5 -> 2.6 / 3.0 / 5.7, 256 3.1 / 3.6 / 6.6 -> 2.3 / 2.4 / 4.8, 64 3.3 /
// 3.5 / 6.0 -> 2.2 / 2.1 / 4.2; fp32, 512 6.6 / 6.8 / 14.7 -> 5.9 / 6.2 / 12.7, 256 4.7 / 5.2 / 9.7 -> 4.0 / 4.1 / 8.3.
// (The next unit's rows requested at the start of a unit and not behind its MFMAs: 32 pieces at 1024 units 5.0, most of them requested before
// they are published and then once more.)
#pragma once

namespace ver {

constexpr int MANY_MAX = 512;   // rows of a slot; more alive pieces than that: the flag form of lstm_rec.h
// fp32 holds the contraction in H / 64 waves, which all take 2 us of MFMAs per unit (the flag form shares them evenly), the first four of them on
// SIMDs of their own: so 256 units and from 448 on.  us per forward pass of two layers with 17 / 32 / 64 pieces per group, 48 timesteps, flag form -> this one
// in hundredths: 192 units 97 / 96 / 104 (12 timesteps 105 / 104 / 108), 256 91 / 90 / 96, 320 109 / 105 / 111, 384 102 / 99 / 100, 448 97 / 98 /
// 96, 512 98 / 92 / 94; one layer of 64 units 3.5 / 3.6 / 6.8 -> 3.9 / 3.9 / 7.6 us per timestep.
template <int MODE> __host__ __device__ constexpr bool many_pays(int H) { return MODE == MODE_BF16 || H == 256 || H > 384; }
// In a launch of several layers it hands rows on about two timesteps later, and pays from this many timesteps on: forward passes of two layers with 17
// pieces per group over 4 / 8 / 12 / 16 / 24 timesteps, as above: bf16, 512 units 111 / 106 / 102 / 101 / 99, 1024 105 / 103 / 102 / 101 / 99, 64 98 / 90 /
// 87 / 84 / 81, 256 (6:) 100 / 98 / 96 / 93 / 90, 576 104 / 97 / 93 / 91 / 86; fp32, 256 units 109 / 103 / 100 / 98 / 96, 448 (12:) 103, 512 104 / 101 / 104 / 102 / 101.
// One layer 101 / 97 / 97 / 95 / 94 at 1024 units.  Only fp32 has the line: the forms add in another order, which in bf16 a rounding may show, and groups
// with 17 pieces for a handful of timesteps are common in updates (2 to 6 us of a launch).
template <int MODE> __host__ __device__ constexpr int many_steps_fwd(bool shared) {
    return shared && MODE == MODE_F32 ? 24 : 1;
}
// Rows of a slot for minibatches of M rows; 0 where no launch of this width runs the form.
inline int many_rows(int mode, int H, int M) {
    if (!(mode == MODE_BF16 ? many_pays<MODE_BF16>(H) : many_pays<MODE_F32>(H)) || M <= FEW_MAX) return 0;
    return M < MANY_MAX ? (M + 15) / 16 * 16 : MANY_MAX;
}
inline __host__ __device__ size_t many_ring_bytes(int mode, int row_elems, int rows) { return (size_t)FEW_RING * rows * row_elems * (mode == MODE_BF16 ? 2 : 4); }
inline __host__ __device__ size_t many_lds_bytes(int cols, int nb) { return (size_t)few_part_floats(cols) * sizeof(float) + (size_t)2 * REC_WAVES * few_stage_bytes(nb); }

// The backward loop runs the timesteps of more than 16 pieces of a group in one form: this one for up to MANY_MAX_BWD (rows of a slot; dz has
// four times the columns of h) where the lines of many_pays_bwd say so; else that of lstm_rec.h.
// In a shared launch it hands rows on about two timesteps later, 10 to 20 us in all.  Backward passes of two layers over 24 / 48 / 96 timesteps, flag form ->
// this one in hundredths (before its other lines):
//   pieces per group           17                24                32                48                64
//   bf16, 128 units            flags             flags       105 / 100 /  98   112 / 109 / 107         flags
//         192            107 / 102 / 101   104 /  99 /  96    98 /  93 /  89   102 /  98 /  95   111 / 108 / 106
//         320            102 /  97 /  93    93 /  89 /  85    87 /  80 /  76    87 /  81 /  77    83 /  79 /  77
//         448            108 / 103 /  99   100 /  95 /  93    94 /  92 /  88    89 /  86 /  79    94 /  90 /  87
//         576             82 /  75 /  71    76 /  70 /  66    72 /  65 /  61    69 /  65 /  62    69 /  65 /  63
//        1024            103 /  97 /  92    94 /  88 /  84    88 /  86 /  83    89 /  84 /  82    88 /  84 /  81
//   fp32, 320            104 / 101 / 100    98 /  94 /  92    92 /  87 /  84    91 /  89 /  85    92 /  88 /  86
//         512            104 / 100 /  98    99 /  95 /  95   100 /  98 /  95    99 /  96 /  93    98 /  95 /  95
// One layer alone: bf16, 128 units 32 pieces 96 / 92 / 91, 48 103 / 102 / 102; 192 97 / 95 / 93 to 100 / 98 / 97; 512, fp32, 97 to 87; 1024 90 to 81.
// us per timestep of one layer, 17 / 32 / 64 pieces: bf16, 1024 units 6.7 / 8.7 / 16.5 -> 5.1 / 6.1 / 12.2, 576 7.5 / 9.2 / 17.4 -> 3.5 / 4.2 / 8.5, 192 2.6 / 3.6 /
// 5.9 -> 2.4 / 2.7 / 5.6, 128 2.4 / 2.8 / 4.8 -> 2.4 / 2.4 / 5.1; fp32, 512 8.2 / 9.8 / 19.1 -> 7.3 / 7.9 / 15.8, 256 4.7 / 5.7 / 10.9 -> 5.1 / 5.3 / 10.7, 128 3.2 /
// 3.9 / 8.2 -> 4.6 / 4.7 / 9.5.  Not bf16 at 256 and 512 units, whose flag form has a loop of its own width: 512 units 3.4 / 4.3 / 8.1 -> 3.3 / 3.7 / 7.3, 256 2.6 / 3.4 /
// 6.5 -> 2.5 / 2.8 / 5.7; long launches of 25 pieces and more gain there, but with the form in the kernel the compiler spills more scalars in the loops of
// few pieces, which an update of 2 x 512 units consists of (6.89 -> 7.03 ms).
constexpr int MANY_MAX_BWD = 256;
constexpr int MANY_STEPS_BWD = 24;
// Kernels that have the form: MT tiles per workgroup, loops for NI operand blocks (0: the general ones).
constexpr bool many_bwd_form(int mode, int mt, int ni) { return mt == 2 || (ni != 4 && ni != 8 && (ni != 16 || mode == MODE_F32)); }
template <int MODE, int MT, int NI> constexpr bool MANY_BWD = many_bwd_form(MODE, MT, NI);
// pieces of a group, timesteps with more than 16 of them; shared: a launch of several layers.
template <int MODE, int MT> __host__ __device__ constexpr bool many_pays_bwd(int H, int pieces, int steps, bool shared) {
    if (steps < MANY_STEPS_BWD || pieces > MANY_MAX_BWD) return false;
    if (shared && pieces <= 24 && steps < 2 * MANY_STEPS_BWD && (MT == 1 || H == 1024)) return false;
    if (MODE == MODE_F32) return H > 256;
    if (MT == 1 && H <= 128) return pieces > 24 && pieces <= 32 && (!shared || steps >= 2 * MANY_STEPS_BWD);
    return MT == 2 || H != 192 || !shared || (pieces > 24 && pieces <= 48);
}
// Rows of a slot of the backward ring for minibatches of M rows; ni: operand blocks per wave (run_bwd).  0 where no launch runs the form.
inline int many_rows_bwd(int mode, int H, int mt, int ni, int M) {
    const int most = mode == MODE_BF16 && H <= 128 ? 32 : MANY_MAX_BWD;
    if (!many_bwd_form(mode, mt, ni) || (mode == MODE_F32 && H <= 256) || M < (FEW_MAX + 1) * MANY_STEPS_BWD) return 0;
    return M < most ? (M + 15) / 16 * 16 : most;
}

// Empties this workgroup's words (cols elements from column j0) of the first `used` rows of every slot of group id's ring.
template <int MODE>
__device__ __forceinline__ void many_clear_ring(void* rings, int id, int row_elems, int rows, int used, int j0, int cols) {
    constexpr int es = (int)sizeof(typename RecGeom<MODE>::E);
    const int words = cols * es / 4;
    unsigned* ring = reinterpret_cast<unsigned*>(static_cast<unsigned char*>(rings) + id * many_ring_bytes(MODE, row_elems, rows));
    for (int i = threadIdx.x; i < FEW_RING * used * words; i += REC_THREADS) {
        const int r = i / words, k = r / used;
        ring[((size_t)k * rows + r % used) * (row_elems * es / 4) + j0 * es / 4 + i % words] = FEW_EMPTY;
    }
}

// Timesteps [t_lo, t_hi): more than FEW_MAX pieces of the group are alive, at most MANY_MAX.  The rows of h_{t_lo-1} are in hprev, announced by
// flag value t_lo + 1; leaves those of h_{t_hi-1} there, announced by t_hi + 1.  False: a wait was abandoned.
template <int MODE, int MT, int PIPE>
__device__ __forceinline__ bool many_fwd(few_args_t<RecFwdArgs> args, const PieceSet& ps, int rank, int t_lo, int t_hi, int T, int* flags,
                                         const PipeLink& pl, int& c_wait, unsigned char* smem) {
    typedef typename RecGeom<MODE>::E E;
    constexpr int es = (int)sizeof(E), KBLK = RecGeom<MODE>::KBLK, VEC = RecGeom<MODE>::VEC;
    constexpr int NB = FewBlocks<MODE, MT == 8>::fwd, UH = 4 * MT, COLS = 16 * MT, ROW = few_row(COLS);
    typedef FewStage<NB> S;
    constexpr unsigned NOWHERE = 0xFFFFFFF0u;
    constexpr int STORES = 6;   // per unit and wave, behind the loads of the next unit
    __shared__ int s_fail_many;
    RecFwdArgs a = *(const RecFwdArgs*)few_scalar(args);
    few_global(a.batch_sizes); few_global(a.t_off); few_global(a.gates); few_global(a.c); few_global(a.hout); few_global(a.c0); few_away(a.err);
    a.whh = (const void*)(__attribute__((address_space(1))) const void*)a.whh;
    const int H = a.H, X = ps.X, x = ps.x;
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = tid / UH, u = tid % UH, j0 = rank * UH;
    float* part = reinterpret_cast<float*>(smem);
    unsigned char* stages = smem + (size_t)few_part_floats(COLS) * sizeof(float) + (size_t)wave * 2 * few_stage_bytes(NB);
    if (tid == 0) s_fail_many = 0;
    bar_lds();   // (LDS of the other form has been read)
    few_clear_part<COLS>(part);
    const int blocks = H / KBLK, n_slices = (blocks + NB - 1) / NB;
    const int slice = n_slices == REC_WAVES ? (wave + rank) % REC_WAVES : wave;   // (see few_fwd)
    const int n_blk = min(NB, blocks - slice * NB);
    const bool polls = slice < n_slices;
    f32x4_t w[MT * NB];
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const E* wrow = static_cast<const E*>(a.whh) + ((size_t)j0 * 4 + j * 16 + lr) * H + (slice * NB * 4 + lk * n_blk) * VEC;
#pragma unroll
        for (int b = 0; b < NB; ++b)
            w[j * NB + b] = b < n_blk ? *reinterpret_cast<const f32x4_t*>(wrow + b * VEC) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < MT * NB; ++i) asm volatile("" : "+v"(w[i]));
    constexpr int WHOLE = (int)0x80000000u;
    const unsigned slot = (unsigned)a.many_rows * (unsigned)(H * es);
    const __amdgpu_buffer_rsrc_t rs_ring = __builtin_amdgcn_make_buffer_rsrc(static_cast<unsigned char*>(a.ring_many) + ps.id * (size_t)FEW_RING * slot, 0,
                                                                             (int)(FEW_RING * slot), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_g = __builtin_amdgcn_make_buffer_rsrc(a.gates, 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_c = __builtin_amdgcn_make_buffer_rsrc(a.c, 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_c0 = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.c0), 0, a.c0 ? (int)min((size_t)a.seq_cap * H * 4, (size_t)0x7fffffff) : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_h = __builtin_amdgcn_make_buffer_rsrc((PIPE & PIPE_PRODUCER) ? static_cast<void*>(a.hcopy) : static_cast<void*>(a.hout), 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_hp = __builtin_amdgcn_make_buffer_rsrc(a.hprev, 0, WHOLE, 0x00020000);
    const bool word_lane = MODE == MODE_F32 || (u & 1) == 0;
    const unsigned slice_off = (unsigned)(slice * NB) * 64u;
    FewWindow<1> win;
    win.init(a.batch_sizes, T, t_lo);
    int t = t_lo, q = 0;                                    // the unit
    int all = win.at(t), all_1 = win.at(t + 1);             // alive pieces of all groups at t, t + 1
    int bs = grp_count(all, ps), bs_1 = grp_count(all_1, ps);
    int base = a.t_off[t], base_prev = t > 0 ? a.t_off[t - 1] : 0;
    few_touch(win.cur);
    few_touch(win.other);
    int edge = (PIPE & PIPE_CONSUMER) && c_wait * pl.ct < T ? c_wait * pl.ct : 0x7fffffff;
    if (!rec_wait(flags, a.G, t + 1, a.err)) return false;
    if ((PIPE & PIPE_PRODUCER) && rank == 0 && tid == 0 && t > 0) st_agent(pl.progress, t);

    // requests the rows of h_{rt-1} of tile rq, rbs pieces of which are alive at rt
    auto request = [&](unsigned char* stage, int rt, int rq, int rbs, int rbase) __attribute__((always_inline)) {
        const bool first = rt == t_lo;
        const unsigned pitch = (unsigned)((first ? X : 1) * H * es);
        const unsigned so = first ? (unsigned)((rbase + x) * H) * (unsigned)es : (unsigned)((rt - 1) & (FEW_RING - 1)) * slot;
#pragma unroll
        for (int j = 0; j < S::LOADS; ++j) {
            const int r = S::row(j);   // (a row beyond the last: the last one again)
            const unsigned off = (unsigned)min(rq * 16 + r, rbs - 1) * pitch + slice_off + S::src(r, n_blk);
            if (first) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_hp, (lds_ptr_t)(stage + j * 1024), 16, off, so, 0, 17);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_ring, (lds_ptr_t)(stage + j * 1024), 16, off, so, 0, 17);
        }
    };
    // the input projection and the cell state of this thread's piece and unit of tile rq
    auto fetch = [&](f32x4_t& z, float& c, int rt, int rq, int rbs, int rbase, int rbase_prev) __attribute__((always_inline)) {
        const int mm = rq * 16 + m;
        const unsigned off = m < 16 && mm < rbs ? (unsigned)((mm * X + x) * H + j0 + u) * 4u : NOWHERE;
        z = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs_g, off == NOWHERE ? NOWHERE : off * 4u, (unsigned)rbase * (unsigned)H * 16u, 0));
        c = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rt == 0 ? rs_c0 : rs_c, off, rt == 0 ? 0u : (unsigned)rbase_prev * (unsigned)H * 4u, 0));
    };
    f32x4_t z0, z1;
    float c0, c1;
    bool alive = true;
    if (polls) request(stages, t, 0, bs, base);
    fetch(z0, c0, t, 0, bs, base, base_prev);
    z1 = z0; c1 = c0;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the counts below hold from the second unit on)
    bar_lds();

    // false: that was the last unit, or a wait was abandoned
    auto unit = [&](f32x4_t& z, float& c, f32x4_t& z_next, float& c_next, unsigned char* stage, unsigned char* stage_next) __attribute__((always_inline)) -> bool {
        const bool step = (q + 1) * 16 >= bs;   // the timestep's last unit
        const bool more = !step || t + 1 < t_hi;
        if (q == 0) win.advance(t + 2);
        if ((PIPE & PIPE_CONSUMER) && step && t + 1 == edge) {   // (the next timestep's input is fetched in this unit)
            if (!pipe_wait_chunk(pl, c_wait, a.err)) {
                alive = false;
                return false;
            }
            ++c_wait;
            edge = c_wait * pl.ct < T ? c_wait * pl.ct : 0x7fffffff;
        }
        const int rt = step ? t + 1 : t, rq = step ? 0 : q + 1, rbs = step ? bs_1 : bs, rbase = step ? base + all : base, rbase_prev = step ? base : base_prev;
        // this unit's loads have completed (issued in the unit before, in front of its stores)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(STORES) : "memory");
        const int rows = min(bs - q * 16, 16);
        if (polls) {
            f32x4_t op[NB];
            const unsigned char* row = stage + lr * (S::C * 16);
            const int key = S::key(lr);
            int spins = 0;
            for (;;) {
                unsigned worst = 0;
#pragma unroll
                for (int b = 0; b < NB; ++b) {   // (a block that the slice does not have: another one, which is not multiplied)
                    const int bb = few_always_whole<MODE, MT>() || b < NB / 2 || n_blk == NB ? b : b - NB / 2;
                    op[b] = *reinterpret_cast<const f32x4_t*>(row + (((lk * n_blk + bb) ^ key) << 4));
                    const u32x4_t v = __builtin_bit_cast(u32x4_t, op[b]);
                    worst = max(max(worst, max(v[0], v[1])), max(v[2], v[3]));
                }
                if (t == t_lo || __all(worst != FEW_EMPTY)) break;
                ++spins;
                if ((spins & 1023) == 0 && (spins > REC_SPIN_LIMIT || __builtin_amdgcn_readfirstlane(ld_agent(a.err)) != 0)) {
                    st_agent(a.err, 1);
                    s_fail_many = 1;
                    break;
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                request(stage, t, q, bs, base);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            f32x4_t acc[MT];
#pragma unroll
            for (int j = 0; j < MT; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            auto half = [&](auto from) __attribute__((always_inline)) {
#pragma unroll
                for (int b = 0; b < NB / 2; ++b)
#pragma unroll
                    for (int j = 0; j < MT; ++j) acc[j] = mfma_block<MODE>(w[j * NB + decltype(from)::value + b], op[decltype(from)::value + b], acc[j]);
            };
            half(FewIdx<0>{});
            if (few_always_whole<MODE, MT>() || n_blk == NB) half(FewIdx<NB / 2>{});
            few_stage_write<MT>(acc, rows, part + slice * (16 * ROW));
        }
        // The next unit's loads: here, so that its rows have been published a good part of a unit ago where it is the next but one after the
        // one that made them.
        if (more) {
            if (polls) request(stage_next, rt, rq, rbs, rbase);
            fetch(z_next, c_next, rt, rq, rbs, rbase, rbase_prev);
        }
        bar_lds();
        const int failed = s_fail_many;
        // Every workgroup has published this tile's rows of timestep t-1, at least two units after its stores for timestep t-2.
        if ((PIPE & PIPE_PRODUCER) && rank == 0 && tid == REC_THREADS - 1 && q == 1 && t - 1 > t_lo) st_agent(pl.progress, t - 1);
        const bool live = m < rows;
        f32x4_t g = z;
        {
            f32x4_t o[REC_WAVES];
            const float* p = part + (m & 15) * ROW + u * 4;
#pragma unroll
            for (int k = 0; k < REC_WAVES; ++k) o[k] = *reinterpret_cast<const f32x4_t*>(p + k * (16 * ROW));
#pragma unroll
            for (int k = 0; k < REC_WAVES; ++k) {
                g[0] += o[k][0]; g[1] += o[k][1]; g[2] += o[k][2]; g[3] += o[k][3];
            }
        }
        g[0] = sigmoidf_(g[0]); g[1] = sigmoidf_(g[1]); g[2] = tanhf_(g[2]); g[3] = sigmoidf_(g[3]);
        const float cn = g[1] * c + g[0] * g[2], h = g[3] * tanhf_(cn);
        unsigned word;
        if constexpr (MODE == MODE_BF16) {
            const unsigned b = to_bf16_finite(h);
            word = few_word(b | (few_dpp<0xb1>(b) << 16));   // (quad_perm 1,0,3,2: the neighbour's value)
        } else {
            word = few_word(__float_as_uint(h));
        }
        const int mm = q * 16 + m;
        const bool goes_on = live && mm < bs_1 && word_lane;
        const unsigned in_ring = goes_on && t + 1 < t_hi ? (unsigned)(mm * H + j0 + u) * es : NOWHERE;
        __builtin_amdgcn_raw_buffer_store_b32(word, rs_ring, in_ring, (unsigned)(t & (FEW_RING - 1)) * slot, 0);
        __builtin_amdgcn_raw_buffer_store_b32(FEW_EMPTY, rs_ring, in_ring, (unsigned)((t + 2) & (FEW_RING - 1)) * slot, 0);
        const unsigned col = (unsigned)((mm * X + x) * H + j0 + u), so = (unsigned)base * (unsigned)H;
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, g), rs_g, live ? col * 16u : NOWHERE, so * 16u, 0);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(cn), rs_c, live ? col * 4u : NOWHERE, so * 4u, 0);
        if (PIPE & PIPE_PRODUCER) __builtin_amdgcn_raw_buffer_store_b32(word, rs_h, live && word_lane ? col * es : NOWHERE, so * es, 17);   // (hcopy)
        else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(h), rs_h, live ? col * 4u : NOWHERE, so * 4u, 0);
        __builtin_amdgcn_raw_buffer_store_b32(word, rs_hp, goes_on ? col * es : NOWHERE, (unsigned)(base + all) * (unsigned)(H * es), 0);
        bar_lds();   // (the partial sums have been read)
        if (__builtin_amdgcn_readfirstlane(failed)) {
            alive = false;
            return false;
        }
        if (step) {
            base_prev = base;
            base += all;
            all = all_1;
            bs = bs_1;
            ++t;
            all_1 = win.at(t + 1);
            bs_1 = grp_count(all_1, ps);
            q = 0;
        } else {
            ++q;
        }
        return more;
    };
    // (two units per iteration: what was requested is used where it was loaded)
    for (;;) {
        if (!unit(z0, c0, z1, c1, stages, stages + few_stage_bytes(NB))) break;
        few_touch(win.cur);
        few_touch(win.other);
        if (!unit(z1, c1, z0, c0, stages + few_stage_bytes(NB), stages)) break;
    }
    if (!alive) return false;
    rec_publish(flags, rank, t_hi + 1);
    return true;
}

// ---- backward -----------------------------------------------------------------------------------------------
// A unit (t, tile) turns the tile's dz rows of timestep t into dh, which is all that the gate gradients of timestep t-1 wait for, and publishes
// those.  One staging area per wave (a slice is four times as long as forward): the next unit's rows are requested when this one's have been read.
// Bound by the rows through LDS (256 KB per unit at H = 1024, 0.85 us) and out of the L2 (4 MB for the 32 CUs), one after the other with the
// gradients.  The cell-state gradient is carried in memory, by the thread that has the piece and unit.
template <typename E, int AUX, typename W>
__device__ __forceinline__ void many_dz(__amdgpu_buffer_rsrc_t rs, W word, unsigned off, unsigned so) {
    if constexpr (sizeof(E) == 2) __builtin_amdgcn_raw_buffer_store_b64(word, rs, off, so, AUX);
    else __builtin_amdgcn_raw_buffer_store_b128(word, rs, off, so, AUX);
}
struct ManySaved {
    f32x4_t g;
    float c, c_prev, dh_above, dc;   // dc: carried to the timestep
};
// Timesteps below t_few, down to 0: more than FEW_MAX pieces of the group are alive.  dh, dc: carried to timestep t_few - 1 by this
// thread's (piece, unit) of the first tile.  False: a wait was abandoned.
template <int MODE, int MT, int PIPE>
__device__ __forceinline__ bool many_bwd(few_args_t<RecBwdArgs> args, const PieceSet& ps, int rank, int t_few, int T, int* flags, const PipeLink& pl,
                                         int c_wait, unsigned char* smem, float dh_few, float dc_few, float (&db)[4]) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));   // (see rec_bwd_rest)
    typedef typename RecGeom<MODE>::E E;
    constexpr int es = (int)sizeof(E), KBLK = RecGeom<MODE>::KBLK, VEC = RecGeom<MODE>::VEC;
    constexpr int NB = FewBlocks<MODE, MT == 2>::bwd, UH = 16 * MT, ROW = few_row(UH), GRP = NB < 8 ? NB : 8;
    typedef FewStage<NB> S;
    constexpr unsigned NOWHERE = 0xFFFFFFF0u;
    constexpr int STORES = 4;   // per unit and wave, behind the loads of the next unit
    __shared__ int s_fail_many;
    RecBwdArgs a = *(const RecBwdArgs*)few_scalar(args);
    few_global(a.batch_sizes); few_global(a.t_off); few_global(a.gates); few_global(a.c); few_global(a.dh_above); few_global(a.c0); few_away(a.err);
    few_global(a.dc_state);
    a.whhT = (const void*)(__attribute__((address_space(1))) const void*)a.whhT;
    const int H = a.H, K = 4 * H, X = ps.X, x = ps.x;
    const int lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = tid / UH, u = tid % UH, j = rank * UH + u;
    float* part = reinterpret_cast<float*>(smem);
    unsigned char* stage = smem + (size_t)few_part_floats(UH) * sizeof(float) + (size_t)wave * few_stage_bytes(NB);
    if (tid == 0) s_fail_many = 0;
    bar_lds();   // (LDS of the other form has been read)
    few_clear_part<UH>(part);
    const int blocks = K / KBLK, n_slices = (blocks + NB - 1) / NB;
    const int slice = n_slices == REC_WAVES ? (wave + rank) % REC_WAVES : wave;
    const int n_blk = min(NB, blocks - slice * NB);
    const bool polls = slice < n_slices;
    f32x4_t w[MT * NB];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const E* wrow = static_cast<const E*>(a.whhT) + ((size_t)rank * UH + i * 16 + lr) * K + (slice * NB * 4 + lk * n_blk) * VEC;
#pragma unroll
        for (int b = 0; b < NB; ++b)
            w[i * NB + b] = b < n_blk ? *reinterpret_cast<const f32x4_t*>(wrow + b * VEC) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < MT * NB; ++i) asm volatile("" : "+v"(w[i]));
    constexpr int WHOLE = (int)0x80000000u;
    const unsigned slot = (unsigned)a.many_rows * (unsigned)(K * es);
    const __amdgpu_buffer_rsrc_t rs_ring = __builtin_amdgcn_make_buffer_rsrc(static_cast<unsigned char*>(a.ring_many) + ps.id * (size_t)FEW_RING * slot, 0,
                                                                             (int)(FEW_RING * slot), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_g = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.gates), 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_c = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.c), 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.dh_above), 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_dc = __builtin_amdgcn_make_buffer_rsrc(a.dc_state, 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_dz = __builtin_amdgcn_make_buffer_rsrc(a.dz, 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_c0 = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.c0), 0, a.c0 ? (int)min((size_t)a.seq_cap * H * 4, (size_t)0x7fffffff) : 0, 0x00020000);
    typedef unsigned wv_t __attribute__((ext_vector_type(MODE == MODE_BF16 ? 2 : 4)));
    auto to_ring = [&](wv_t v, unsigned off, unsigned so) __attribute__((always_inline)) {
        if constexpr (MODE == MODE_BF16) __builtin_amdgcn_raw_buffer_store_b64(v, rs_ring, off, so, 0);
        else __builtin_amdgcn_raw_buffer_store_b128(v, rs_ring, off, so, 0);
    };
    const unsigned slice_off = (unsigned)(slice * NB) * 64u;
    FewWindow<-1> win;
    win.init(a.batch_sizes, T, t_few - 1);
    few_touch(win.cur);
    few_touch(win.other);
    // The unit (t, q) ends with the gate gradients of timestep t-1.  all*, bs*: alive pieces of all groups and of this one at t, t-1, t-2.
    int t = t_few, q = 0;
    int all = t < T ? a.batch_sizes[t] : 0, all_1 = win.at(t - 1), all_2 = win.at(t - 2);
    all = __builtin_amdgcn_readfirstlane(all);
    int bs = grp_count(all, ps), bs_1 = grp_count(all_1, ps), bs_2 = grp_count(all_2, ps);
    int base_1 = __builtin_amdgcn_readfirstlane(a.t_off[t - 1]);   // first row of timestep t-1
    auto wait_chunk = [&](int k) -> bool {   // consumer: the input of timestep k
        if (PIPE & PIPE_CONSUMER)
            while (c_wait > 0 && k >= 0 && k < c_wait * pl.ct) {
                --c_wait;
                if (!pipe_wait_chunk(pl, c_wait, a.err)) return false;
            }
        return true;
    };
    // requests the dz rows of timestep rt, tile rq, rbs pieces of which are alive
    auto request = [&](int rt, int rq, int rbs) __attribute__((always_inline)) {
        const unsigned so = (unsigned)(rt & (FEW_RING - 1)) * slot;
#pragma unroll
        for (int i = 0; i < S::LOADS; ++i) {
            const int r = S::row(i);   // (a row beyond the last: the last one again)
            const unsigned off = (unsigned)min(rq * 16 + r, rbs - 1) * (unsigned)(K * es) + slice_off + S::src(r, n_blk);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_ring, (lds_ptr_t)(stage + i * 1024), 16, off, so, 0, 17);
        }
    };
    // what the gate gradients of timestep k, tile rq, need: n_k pieces alive, n_up of them at k+1 too
    auto fetch = [&](ManySaved& s, int k, int rq, int n_k, int n_up, int rbase, int rbase_prev) __attribute__((always_inline)) {
        const int mm = rq * 16 + m;
        const unsigned col = (unsigned)((mm * X + x) * H + j), so = (unsigned)rbase * (unsigned)H;
        const bool live = m < 16 && mm < n_k;
        s.g = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs_g, live ? col * 16u : NOWHERE, so * 16u, 0));
        s.c = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_c, live ? col * 4u : NOWHERE, so * 4u, 0));
        s.dh_above = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_a, live ? col * 4u : NOWHERE, so * 4u, 0));
        s.c_prev = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(k == 0 ? rs_c0 : rs_c, live ? col * 4u : NOWHERE, k == 0 ? 0u : (unsigned)rbase_prev * (unsigned)H * 4u, 0));
        s.dc = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_dc, live && mm < n_up ? col * 4u : NOWHERE, 0u, 0));
    };
    // gate gradients of timestep k, tile kq; dh: carried to it
    auto gradients = [&](const ManySaved& s, float dh_sum, int k, int kq, int n_k, int rbase) __attribute__((always_inline)) {
        const int mm = kq * 16 + m;
        const bool live = m < 16 && mm < n_k;
        const float gi = s.g[0], gf = s.g[1], gg = s.g[2], go = s.g[3], tc = tanhf_(s.c);
        const float dh = s.dh_above + dh_sum, dc = s.dc + dh * go * (1.f - tc * tc);
        const float dzi = dc * gg * gi * (1.f - gi), dzf = dc * s.c_prev * gf * (1.f - gf), dzg = dc * gi * (1.f - gg * gg), dzo = dh * tc * go * (1.f - go);
        wv_t word;
        if constexpr (MODE == MODE_BF16) {
            word[0] = few_word((unsigned)to_bf16_finite(dzi) | ((unsigned)to_bf16_finite(dzf) << 16));
            word[1] = few_word((unsigned)to_bf16_finite(dzg) | ((unsigned)to_bf16_finite(dzo) << 16));
        } else {
            word[0] = few_word(__float_as_uint(dzi)); word[1] = few_word(__float_as_uint(dzf));
            word[2] = few_word(__float_as_uint(dzg)); word[3] = few_word(__float_as_uint(dzo));
        }
        const unsigned in_ring = live && k > 0 ? (unsigned)(mm * K + j * 4) * es : NOWHERE;
        to_ring(word, in_ring, (unsigned)(k & (FEW_RING - 1)) * slot);
        to_ring(wv_t(FEW_EMPTY), in_ring, (unsigned)((k + 2) & (FEW_RING - 1)) * slot);
        const unsigned col = (unsigned)((mm * X + x) * H + j);
        const unsigned in_dz = live ? col * 4u * es : NOWHERE, so_dz = (unsigned)rbase * (unsigned)(K * es);
        many_dz<E, (PIPE & PIPE_PRODUCER) ? 17 : 0>(rs_dz, word, in_dz, so_dz);   // (two layers: the rows are also read on other XCDs)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dc * gf), rs_dc, live ? col * 4u : NOWHERE, 0u, 0);
        if (live) { db[0] += dzi; db[1] += dzf; db[2] += dzg; db[3] += dzo; }
    };
    ManySaved s0, s1;
    bar_lds();   // (the partial sums are clear)
    if (!wait_chunk(t - 1) || !wait_chunk(t - 2)) return false;
    // timestep t_few - 1, whose dh comes from the other form
    for (int k = 0; k * 16 < bs_1; ++k) {
        fetch(s0, t - 1, k, bs_1, 0, base_1, base_1 - all_2);
        const bool carried = k == 0 && m < bs;
        if (carried) s0.dc = dc_few;
        gradients(s0, carried ? dh_few : 0.f, t - 1, k, bs_1, base_1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    bool alive = true, more = true;
    auto down = [&] {   // to the timestep below
        all = all_1; bs = bs_1;
        all_1 = all_2; bs_1 = bs_2;
        --t;
        base_1 -= all_1;
        all_2 = win.at(t - 2);
        bs_2 = grp_count(all_2, ps);
    };
    down();
    if (t > 0) {
        if (polls) request(t, 0, bs);
        fetch(s0, t - 1, 0, bs_1, bs, base_1, base_1 - all_2);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (no stores behind these: the count below holds from the second unit on)
    }
    // false: that was the last unit, or a wait was abandoned
    auto unit = [&](ManySaved& s, ManySaved& s_next) __attribute__((always_inline)) -> bool {
        const bool step = (q + 1) * 16 >= bs_1;   // the timestep's last unit
        more = !step || t - 1 > 0;
        if (q == 0) win.advance(t - 3);
        if (step && !wait_chunk(t - 2)) {   // (what timestep t-2 needs is fetched in this unit)
            alive = false;
            return false;
        }
        // this unit's loads have completed (issued in the unit before, in front of its stores)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(STORES) : "memory");
        const int rows = min(max(bs - q * 16, 0), 16);
        if (polls && rows > 0) {
            const unsigned char* row = stage + lr * (S::C * 16);
            const int key = S::key(lr);
            int spins = 0;
            f32x4_t acc[MT];
            for (;;) {
                unsigned worst = 0;
#pragma unroll
                for (int i = 0; i < MT; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int b0 = 0; b0 < NB; b0 += GRP) {
                    if (!few_always_whole<MODE, MT>() && b0 >= n_blk) break;
                    f32x4_t op[GRP];
#pragma unroll
                    for (int b = 0; b < GRP; ++b) {
                        op[b] = *reinterpret_cast<const f32x4_t*>(row + (((lk * n_blk + b0 + b) ^ key) << 4));
                        const u32x4_t v = __builtin_bit_cast(u32x4_t, op[b]);
                        worst = max(max(worst, max(v[0], v[1])), max(v[2], v[3]));
                    }
#pragma unroll
                    for (int b = 0; b < GRP; ++b)
#pragma unroll
                        for (int i = 0; i < MT; ++i) acc[i] = mfma_block<MODE>(w[i * NB + b0 + b], op[b], acc[i]);
                }
                if (__all(worst != FEW_EMPTY)) break;
                ++spins;
                if ((spins & 1023) == 0 && (spins > REC_SPIN_LIMIT || __builtin_amdgcn_readfirstlane(ld_agent(a.err)) != 0)) {
                    st_agent(a.err, 1);
                    s_fail_many = 1;
                    break;
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                request(t, q, bs);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            few_stage_write<MT>(acc, rows, part + slice * (16 * ROW));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (the staging area has been read)
        if (more) {   // the next unit's loads, see the forward loop
            const int rt = step ? t - 1 : t, rq = step ? 0 : q + 1, rbs = step ? bs_1 : bs;
            if (polls && rq * 16 < rbs) request(rt, rq, rbs);
            fetch(s_next, rt - 1, rq, step ? bs_2 : bs_1, rbs, step ? base_1 - all_2 : base_1, step ? base_1 - all_2 - win.at(t - 3) : base_1 - all_2);
        }
        bar_lds();
        const int failed = s_fail_many;
        // Every workgroup has published this tile's rows of timestep t, at least two units after its stores for timestep t+1.
        if ((PIPE & PIPE_PRODUCER) && rank == 0 && tid == REC_THREADS - 1 && q == 1 && t + 1 < T) st_agent(pl.progress, T - (t + 1));
        float dh = 0.f;
        {
            float o[REC_WAVES];
            const float* p = part + (m & 15) * ROW + u;
#pragma unroll
            for (int k = 0; k < REC_WAVES; ++k) o[k] = p[k * (16 * ROW)];
#pragma unroll
            for (int k = 0; k < REC_WAVES; ++k) dh += o[k];
        }
        gradients(s, m < rows ? dh : 0.f, t - 1, q, bs_1, base_1);
        bar_lds();   // (the partial sums have been read)
        if (__builtin_amdgcn_readfirstlane(failed)) {
            alive = false;
            return false;
        }
        if (!more) return false;
        if (step) {
            down();
            q = 0;
        } else {
            ++q;
        }
        return true;
    };
    // (two units per iteration: what was requested is used where it was loaded)
    while (t > 0) {
        if (!unit(s0, s1)) break;
        few_touch(win.cur);
        few_touch(win.other);
        if (!unit(s1, s0)) break;
        few_touch(win.cur);
        few_touch(win.other);
    }
    if (!alive) return false;
    if (PIPE & PIPE_PRODUCER) {   // the last rows are complete once every flag says so
        rec_publish(flags, rank, T + 1);
        if (rank == 0) {
            if (!rec_wait(flags, a.G, T + 1, a.err)) return false;
            if (tid == 0) st_agent(pl.progress, T);
        }
    }
    return true;
}

}  // namespace ver
