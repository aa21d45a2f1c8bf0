// The forward time loop while a group has more than 16 alive pieces (included by lstm_few.h, whose exchange it uses).  gfx950 only.
//
// The alive pieces of a timestep are worked through 16 at a time.  Such a unit, (timestep, tile of 16 pieces), depends on the same tile
// of the timestep before, which is at least one unit back, so that no unit has to wait for the exchange: a unit's rows, its
// input projections and its cell states are requested while the unit before is worked on.  The rows go from the ring straight into
// LDS (two areas per wave in turn); an operand that is still empty when it is read (lstm_few.h) is requested again.
// Memory operations of a wave complete in order, and a unit issues the same number of them whatever its pieces (those without
// one go beyond the buffers), so that the wait for a unit's rows leaves the stores of the unit before and the next unit's loads in
// flight.
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
// Not fp32 up to 128 units, where one or two waves hold all of the contraction, 2 us of MFMAs per unit (the flag form shares them): 64 units 3.5 /
// 3.6 / 6.8 -> 3.9 / 3.9 / 7.6, 128 3.8 / 3.9 / 7.6 -> 3.9 / 3.9 / 7.8.
template <int MODE> __host__ __device__ constexpr bool many_pays(int H) { return MODE == MODE_BF16 || H > 128; }
inline __host__ __device__ int many_rows(int M) { return M < MANY_MAX ? (M + 15) / 16 * 16 : MANY_MAX; }
inline __host__ __device__ size_t many_ring_bytes(int mode, int H, int rows) { return (size_t)FEW_RING * rows * H * (mode == MODE_BF16 ? 2 : 4); }
inline __host__ __device__ size_t many_lds_bytes(int cols, int nb) { return (size_t)few_part_floats(cols) * sizeof(float) + (size_t)2 * REC_WAVES * few_stage_bytes(nb); }

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
    few_global(a.batch_sizes); few_global(a.t_off); few_global(a.gates); few_global(a.c); few_global(a.hout); few_global(a.c0); few_global(a.err);
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
        if (q == 0) {   // a new timestep
            win.advance(t + 2);
            if ((PIPE & PIPE_CONSUMER) && t + 1 == edge) {   // (its input is fetched in this timestep's last unit)
                if (!pipe_wait_chunk(pl, c_wait, a.err)) {
                    alive = false;
                    return false;
                }
                ++c_wait;
                edge = c_wait * pl.ct < T ? c_wait * pl.ct : 0x7fffffff;
            }
        }
        const bool step = (q + 1) * 16 >= bs;   // the timestep's last unit
        const bool more = !step || t + 1 < t_hi;
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
        if ((PIPE & PIPE_PRODUCER) && rank == 0 && tid == REC_THREADS - 1 && step && t - 1 > t_lo) st_agent(pl.progress, t - 1);
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

}  // namespace ver
