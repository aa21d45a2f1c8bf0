// The time loops while a group has up to four alive pieces (included by lstm_few.h, whose exchange they use).  gfx950 only.
//
// Here four neighbouring lanes own a (piece, unit), one lane per gate, and a wave owns (part of) one piece: which piece,
// and whether it is alive, is a scalar.  What bounds these timesteps is the chain of instructions that one wave walks
// from the arrival of the exchanged values to the publication of the next ones, at 4 to 5 cycles per instruction and more per
// branch.  So:
//  * a lane adds the partial sums of one gate and applies one non-linearity (one exponential and one reciprocal behind another
//    where a thread per unit needs three of each), and the four gates meet through DPP;
//  * the poll is requested right behind the wave's own publication (but see LATE), and what the next timestep needs is made while it is on its way:
//    where its rows begin, who is alive, whether a chunk has to be waited for, and backward the factors of the gate gradients that
//    only depend on what the forward pass saved.  Between the arrival of the values and the publication there is
//    what depends on them, and the memory operations of the owner wave, behind the MFMAs;
//  * scalar registers are as scarce as time (see few_fwd): one copy of a loop's body, comparisons of lane numbers made anew.
// Instructions from barrier to barrier, backward with one piece at 512 units: 640 -> 320.  lstm_few.h has the times.
// (Backward loads of the saved activations through pointers instead of buffers: two scalar registers each instead of four, but
// 1.32 us per timestep instead of 1.15.  One loop for one to four pieces instead of two: 1.53 instead of 1.28 in fp32.)
#pragma once

namespace ver {

// The value of lane I of every quad, in all four.
template <int I> __device__ __forceinline__ float quad_get(float v) { return __uint_as_float(few_dpp<I * 0x55>(__float_as_uint(v))); }
// The sum over the quad, the same bits in all four lanes.
__device__ __forceinline__ float quad_sum(float v) {
    v += __uint_as_float(few_dpp<0xb1>(__float_as_uint(v)));   // (quad_perm 1,0,3,2)
    return v + __uint_as_float(few_dpp<0x4e>(__float_as_uint(v)));   // (quad_perm 2,3,0,1)
}
// Scalars that are wanted in registers here and not where they are used.
__device__ __forceinline__ void quad_now(unsigned& a) {
    a = __builtin_amdgcn_readfirstlane(a);
    asm volatile("" : "+s"(a));
}

// A poll in two halves: the loads are requested as soon as the wave has published its own words, and what has to be done for the
// next timestep is done while they are on their way.  Lanes without words of their own ask beyond the buffer, for zeros.
constexpr unsigned QUAD_NOWHERE = 0xFFFFFFF0u;
template <int L>
__device__ __forceinline__ void quad_request(__amdgpu_buffer_rsrc_t rs, const unsigned (&off)[L], unsigned slot, u32x4_t (&raw)[L]) {
#pragma unroll
    for (int j = 0; j < L; ++j) raw[j] = __builtin_amdgcn_raw_buffer_load_b128(rs, off[j], slot, 17);   // (sc0 sc1: not from the CU's L1)
}
// Until no requested word is empty.  False: the wait was abandoned (time-out here or in another workgroup).
template <int L>
__device__ __forceinline__ bool quad_arrived(__amdgpu_buffer_rsrc_t rs, const unsigned (&off)[L], unsigned slot, u32x4_t (&raw)[L], int* err) {
    int spins = 0;
    for (;;) {
        unsigned m = 0;
#pragma unroll
        for (int j = 0; j < L; ++j) m = max(max(m, max(raw[j][0], raw[j][1])), max(raw[j][2], raw[j][3]));
        if (__all(m != FEW_EMPTY)) return true;
        ++spins;
        if ((spins & 1023) == 0 && (spins > REC_SPIN_LIMIT || __builtin_amdgcn_readfirstlane(ld_agent(err)) != 0)) {
            st_agent(err, 1);
            return false;
        }
        quad_request<L>(rs, off, slot, raw);
    }
}
// Offsets of the L loads of a lane inside a slot: operand blocks blk, blk + BPL, ... of its piece, as far as there are any.
template <int L, int BPL>
__device__ __forceinline__ void quad_offsets(unsigned (&off)[L], unsigned first, bool any, int blk, int n_blk) {
#pragma unroll
    for (int j = 0; j < L; ++j) off[j] = any && blk + j * BPL < n_blk ? first + j * BPL * 16 : QUAD_NOWHERE;
}

// The lane of a quad, to be compared anew: a comparison made once and kept takes two scalar registers.
__device__ __forceinline__ void quad_again(int& q) { asm volatile("" : "+v"(q)); }

// Product of the polled rows and the wave's partial sums, with `between` behind the MFMAs.
template <int MODE, int MT, int NB, int P, int L, typename F>
__device__ __forceinline__ void quad_product(const f32x4_t (&w)[MT * NB], const u32x4_t (&raw)[L], int bs, int n_blk, float* s, bool polls, F&& between) {
    f32x4_t acc[MT];
    if (polls) {
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        few_product<MODE, MT, NB, P, L>(w, raw, bs, n_blk, acc);
    }
    between();
    if (polls) few_write<MODE, MT, P>(acc, bs, s);
}

// ---- forward ------------------------------------------------------------------------------------------------
// Timesteps [t, T), at most QUAD_FWD alive pieces.  False: a wait was abandoned.
template <int MODE, int MT, int NB, int PIPE>
__device__ __forceinline__ bool quad_fwd(FewFwd<MODE, MT, NB>& s, const RecFwdArgs& a, const PieceSet& ps, int rank, int* flags,
                                         unsigned char* ring, const PipeLink& pl, int& t, int T) {
    typedef typename RecGeom<MODE>::E E;
    constexpr int es = (int)sizeof(E), P = QUAD_FWD<MT>;
    constexpr int UH = 4 * MT, COLS = 16 * MT, ROW = few_row(COLS), PART = P * ROW;
    constexpr int BPL = 16 / P, L = (NB + BPL - 1) / BPL;
    const int X = ps.X, x = ps.x, H = a.H;
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = wave * 64 / COLS;                                  // this wave's piece
    const int col = tid % COLS, u = col >> 2, j0 = rank * UH, n = m * X + x;
    int q = tid & 3;
    const int piece = lr / BPL, blk = lr % BPL;
    const unsigned slice_off = (unsigned)(s.slice * NB) * 64u;
    const unsigned k_off = slice_off + (unsigned)(lk * s.n_blk + blk) * 16u;
    const unsigned slot = (unsigned)few_slot_bytes(MODE, H);
    const bool polls = s.slice < s.n_slices;
    // from a thread per (piece, unit) to a lane per gate
    float z2 = 0.f, s_c = 0.f;   // input projection of the next timestep, cell state
    bar_lds();   // (the partial sums of the phase before have been read)
    if (tid < P * UH) {
        *reinterpret_cast<f32x4_t*>(s.part + tid * 4) = s.z;
        s.part[P * COLS + tid] = s.c;
    }
    bar_lds();
    if (m < P) {
        z2 = s.part[tid];
        s_c = s.part[P * COLS + m * UH + u];
    }
    bar_lds();
    few_clear_part<COLS>(s.part);
    bar_lds();
    constexpr int WHOLE = (int)0x80000000u;
    const __amdgpu_buffer_rsrc_t rs_g = __builtin_amdgcn_make_buffer_rsrc(a.gates, 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_hc = __builtin_amdgcn_make_buffer_rsrc(a.hcopy, 0, (PIPE & PIPE_PRODUCER) ? WHOLE : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_ring = __builtin_amdgcn_make_buffer_rsrc(ring, 0, (int)(FEW_RING * slot), 0x00020000);
    const unsigned g_off = (unsigned)(n * 4 * H + j0 * 4 + col) * 4u;   // bytes inside a timestep's gates rows
    const unsigned h_off = (unsigned)(n * H + j0 + u);                  // elements inside those of an [M, H] array
    const bool word_lane = q == 0 && (MODE == MODE_F32 || (u & 1) == 0);   // publishes: a value, or a bf16 pair
    const unsigned w_off = (unsigned)(m * H + j0 + u) * es;             // inside a slot
    // lane 0 of a quad stores the cell state, 1 h, 2 the words of hprev: one instruction
    unsigned char* const to_c = reinterpret_cast<unsigned char*>(a.c), * const to_h = reinterpret_cast<unsigned char*>(a.hout), * const to_hp = static_cast<unsigned char*>(a.hprev);
    unsigned char* const side = (q == 0 ? to_c : q == 1 ? to_h : to_hp) + h_off * (q == 2 ? (unsigned)es : 4u);
    const bool side_ch = q == 0 || (q == 1 && !(PIPE & PIPE_PRODUCER)), side_hp = q == 2 && (MODE == MODE_F32 || (u & 1) == 0);
    // the non-linearity of this lane's gate: e = 2^(k x), value = ga / (1 + e) + gb (sigmoid, or tanh for gate 2)
    const float k_exp = q == 2 ? 2.8853900817779268f : -1.4426950408889634f, ga = q == 2 ? -2.f : 1.f, gb = q == 2 ? 1.f : 0.f;
    float s_g = 0.f, s_h = 0.f;               // with s_c: results of the timestep before, not yet stored
    unsigned s_w = 0;
    int bs_prev = 0;                          // pieces they belong to
    int edge = (PIPE & PIPE_CONSUMER) && s.c_wait * pl.ct < T ? s.c_wait * pl.ct : 0x7fffffff;   // first timestep of the chunk to wait for
    int off_bs = grp_count(s.bs_a, ps);
    unsigned off[L];
    quad_offsets<L, BPL>(off, (unsigned)(piece * H) * es + k_off, piece < off_bs, blk, s.n_blk);
    u32x4_t raw[L];
#pragma unroll
    for (int j = 0; j < L; ++j) raw[j] = u32x4_t{0u, 0u, 0u, 0u};
    if (polls && t != s.t0) quad_request<L>(rs_ring, off, (unsigned)((t - 1) & (FEW_RING - 1)) * slot, raw);
    auto store_results = [&](int bs, unsigned so_g, unsigned so_c, unsigned so_hp, unsigned so_hc) __attribute__((always_inline)) {
        // (copies first: a choice between variables, and not between their values, would keep them in memory)
        const unsigned vc = __float_as_uint(s_c), vh = __float_as_uint(s_h), vw = s_w;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s_g), rs_g, g_off, so_g, 0);
        if (side_ch || (side_hp && m < bs)) {
            *reinterpret_cast<unsigned*>(side + (q == 2 ? so_hp : so_c)) = q == 0 ? vc : q == 1 ? vh : vw;
        }
        if ((PIPE & PIPE_PRODUCER) && word_lane)   // written through: input of the workers' product
            __builtin_amdgcn_raw_buffer_store_b32(s_w, rs_hc, h_off * es, so_hc, 17);
    };

    // One copy of the loop's body, values that arrive for the next timestep moved after the poll (two copies that swap roles cost 60 to
    // 90 moves where they leave the loop and meet again).
    int bs = grp_count(s.bs_a, ps);
    bool alive = true;
    for (;;) {
        quad_again(q);
        const int bs_next = grp_count(s.bs_b, ps);   // (0 beyond T)
        const int base_next = s.base + s.bs_a;
        s.win.advance(t + 2);
        int to_edge = 0x7fffffff;   // consumer: timesteps until the next chunk has to be there
        if (PIPE & PIPE_CONSUMER) {
            if (t + 1 == edge) {
                if (!s.ready && !pipe_wait_chunk(pl, s.c_wait, a.err)) {
                    alive = false;
                    break;
                }
                ++s.c_wait;
                s.ready = false;
                edge = s.c_wait * pl.ct < T ? s.c_wait * pl.ct : 0x7fffffff;
            }
            to_edge = edge - (t + 1);
        }
        unsigned so_gnext = (unsigned)base_next * (unsigned)H * 16u, so_g = (unsigned)s.base_prev * (unsigned)H * 16u;
        unsigned so_hp = (unsigned)s.base * (unsigned)(H * es), so_w = (unsigned)(t & (FEW_RING - 1)) * slot, so_e = (unsigned)((t + 2) & (FEW_RING - 1)) * slot;
        quad_now(so_gnext); quad_now(so_g); quad_now(so_hp); quad_now(so_w); quad_now(so_e);
        bool ok = true;
        if (t == s.t0) {
            // the rows were written under the flag protocol (initial states, or the timestep before with more pieces)
            if (!rec_wait(flags, a.G, t + 1, a.err)) {
                alive = false;
                break;
            }
            if ((PIPE & PIPE_PRODUCER) && rank == 0 && tid == 0 && t > 0) st_agent(pl.progress, t);
            if (polls) {
                const unsigned char* rows = reinterpret_cast<const unsigned char*>(static_cast<const E*>(a.hprev) + (size_t)(s.base + x) * H);
                unsigned first[L];
                few_offsets<L, BPL>(first, (unsigned)(piece * X * H) * es + k_off, blk, s.n_blk);
                few_read<L>(rows, first, piece < bs && blk < s.n_blk, false, raw, a.err);
            }
        } else if (polls) {
            ok = quad_arrived<L>(rs_ring, off, (unsigned)((t - 1) & (FEW_RING - 1)) * slot, raw, a.err);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (also: this wave's stores of two timesteps ago have completed)
        few_touch(z2);
        few_touch(s.win.cur);
        few_touch(s.win.other);
        if (PIPE & PIPE_CONSUMER) few_touch(s.have);
        if (!ok) *s.fail = 1;
        const float z = z2;
        float* part = s.part + (t & 1) * (REC_WAVES * PART);
        quad_product<MODE, MT, NB, P, L>(s.w, raw, bs, s.n_blk, part + s.slice * PART, polls, [&]() __attribute__((always_inline)) {
            // the input projection of the next timestep, the results of the one before
            if (m < bs_next) z2 = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_g, g_off, so_gnext, 0));
            if (m < bs_prev) store_results(bs, so_g, so_g >> 2, so_hp, (so_g >> 4) * es);
        });
        // A look at the chunk that the next timestep asks for: usually finished, which saves that wait its round trip.  Its
        // counter is requested a timestep earlier.
        if ((PIPE & PIPE_CONSUMER) && to_edge <= 2) {
            if (to_edge == 1) {
                if (tid == REC_THREADS - 1) s.fail[1] = s.have;
                s.have = 0;
            } else if (tid == REC_THREADS - 1) {
                s.have = ld_agent(&pl.done[s.c_wait]);
            }
        }
        bar_lds();
        const int failed = *s.fail;   // (looked at after the publication: its read is not waited for by itself)
        // Every workgroup has published the rows of timestep t-1, which it did after its stores for timestep t-3 had
        // completed (they are issued in timestep t-2 and waited for in timestep t-1).
        if ((PIPE & PIPE_PRODUCER) && rank == 0 && tid == REC_THREADS - 1 && t - 2 > s.t0) st_agent(pl.progress, t - 2);
        if (m < bs) {
            float o[REC_WAVES];
            const float* p = part + m * ROW + col;
#pragma unroll
            for (int k = 0; k < REC_WAVES; ++k) o[k] = p[k * PART];
            const float zz = z + (((o[0] + o[1]) + (o[2] + o[3])) + ((o[4] + o[5]) + (o[6] + o[7])));
            s_g = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(zz * k_exp)) * ga + gb;
            s_c = quad_get<1>(s_g) * s_c + quad_get<0>(s_g) * quad_get<2>(s_g);
            s_h = quad_get<3>(s_g) * tanhf_(s_c);
            if constexpr (MODE == MODE_BF16) {
                const unsigned w = to_bf16_finite(s_h);
                s_w = few_word(w | (few_dpp<0x104>(w) << 16));   // (row_shl:4, the next unit's; used where u is even)
            } else {
                s_w = few_word(__float_as_uint(s_h));
            }
            if (m < bs_next && word_lane) {
                __builtin_amdgcn_raw_buffer_store_b32(s_w, rs_ring, w_off, so_w, 0);
                __builtin_amdgcn_raw_buffer_store_b32(FEW_EMPTY, rs_ring, w_off, so_e, 0);
            }
        }
        if (bs_next != off_bs) {
            off_bs = bs_next;
            quad_offsets<L, BPL>(off, (unsigned)(piece * H) * es + k_off, piece < bs_next, blk, s.n_blk);
        }
        if (polls) quad_request<L>(rs_ring, off, so_w, raw);   // (after the last timestep: nothing, from beyond the buffer)
        __builtin_amdgcn_sched_barrier(0);
        if ((PIPE & PIPE_CONSUMER) && to_edge == 1) s.ready = __builtin_amdgcn_readfirstlane(s.fail[1]) >= few_scalar(pl.need);
        if (__builtin_amdgcn_readfirstlane(failed)) {
            alive = false;
            break;
        }
        bs_prev = bs;
        bs = bs_next;
        s.base_prev = s.base;
        s.base = base_next;
        s.bs_a = s.bs_b;
        s.bs_b = s.win.at(t + 2);
        if (++t >= T) break;
    }
    if (!alive) return false;
    if (m < bs_prev) {
        const unsigned so_g = (unsigned)s.base_prev * (unsigned)H * 16u;
        store_results(0, so_g, so_g >> 2, 0u, (so_g >> 4) * es);
    }
    return true;
}

// ---- backward -----------------------------------------------------------------------------------------------
// What the forward pass saved for this lane's gate at one timestep.
struct QuadSaved {
    float g, c_prev, dh_above;
    float c;                   // only loaded for a piece whose last timestep this is
};
// What of a timestep's gate gradients does not depend on the gradient that is carried to it.
struct QuadFactor {
    float dz;      // of dh (output gate) or dc (the others)
    float dc;      // of dh in dc
    float gf, dh_above;
};
// Timesteps t, t-1, ... >= t_stop while at most QUAD_MAX pieces are alive (t = T-1 at the call).  Leaves the carried gradients and
// the cell state as a thread per (piece, unit) holds them, and adds to the sums of the gate gradients.
template <int MODE, int MT, int NB, int PIPE>
struct QuadBwd {
    typedef typename RecGeom<MODE>::E E;
    static constexpr int es = (int)sizeof(E);
    static constexpr int UH = 16 * MT, COLS = 4 * UH, ROW = few_row(UH), PART = QUAD_MAX * ROW;
    float dh, dc, db;           // gradients carried to timestep t, sum of the gate gradients
    float c, c_prev;            // cell state of timesteps t, t - 1
    QuadSaved r0, r1;           // saved for timesteps t-1 and t-2
    QuadFactor f;               // of timestep t
    int bs_m3;                  // alive pieces at t-3
};

// Requests the saved activations of timestep k (rows from base_k, of timestep k-1 from base_k1) for a live piece m.
__device__ __forceinline__ float quad_load(const float* array, unsigned rows, unsigned H, unsigned byte) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(array), 0, (int)0x80000000u, 0x00020000);
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, byte, rows * H * 4u, 0));
}
__device__ __forceinline__ void quad_load_saved(QuadSaved& r, const RecBwdArgs& a, int m, int n, unsigned g_col, unsigned h_col, int k, int bs_up, int base_k,
                                                int base_k1) {
    const unsigned H = (unsigned)a.H;
    r.g = quad_load(a.gates, (unsigned)base_k * 4u, H, g_col);
    r.dh_above = quad_load(a.dh_above, (unsigned)base_k, H, h_col);
    if (k > 0) r.c_prev = quad_load(a.c, (unsigned)base_k1, H, h_col);
    else r.c_prev = (a.c0 && n < a.seq_cap) ? a.c0[h_col >> 2] : 0.f;
    if (m >= bs_up) r.c = quad_load(a.c, (unsigned)base_k, H, h_col);
}
__device__ __forceinline__ void quad_touch(QuadSaved& r) { few_touch(r.g); few_touch(r.c_prev); few_touch(r.dh_above); few_touch(r.c); }
// c: the cell state of the timestep.
__device__ __forceinline__ QuadFactor quad_factor(const QuadSaved& r, float c, int q) {
    const float g = r.g, gi_gg = __uint_as_float(few_dpp<0xc6>(__float_as_uint(g)));   // (quad_perm 2,1,0,3)
    const float tc = tanhf_(c);
    QuadFactor f;
    const float own = q == 2 ? 1.f - g * g : g * (1.f - g);
    f.dz = own * (q == 1 ? r.c_prev : q == 3 ? tc : gi_gg);
    f.dc = quad_get<3>(g) * (1.f - tc * tc);
    f.gf = quad_get<1>(g);
    f.dh_above = r.dh_above;
    return f;
}

template <int MODE, int MT, int NB, int P, int PIPE>
__device__ __forceinline__ bool quad_bwd_loop(QuadBwd<MODE, MT, NB, PIPE>& d, FewBwd<MODE, MT, NB>& s, const RecBwdArgs& a, const PieceSet& ps, int rank,
                                               unsigned char* ring, const PipeLink& pl, int& t, int T, int t_stop) {
    typedef QuadBwd<MODE, MT, NB, PIPE> D;
    constexpr int es = D::es, UH = D::UH, COLS = D::COLS, ROW = D::ROW, PART = D::PART;
    constexpr int BPL = 16 / P, L = (NB + BPL - 1) / BPL;
    // A poll here is four loads per lane in 32 workgroups, and right behind the publication it comes too early to be the only one (judged by the times, not
    // counted): it is requested behind the factors.  us per timestep of two layers with 2 / 3 / 4 pieces per group, right behind the publication -> behind
    // the factors: 1024 units 1.72 / 2.08 / 2.30 -> 1.61 / 1.90 / 2.01, 576 (2 / 4) 1.58 / 1.83 -> 1.50 / 1.67; one layer, 1024 1.61 / 1.95 / 2.08 -> 1.49 / 1.71 / 1.78.
    constexpr bool LATE = MT == 2 && P > 2;
    const int X = ps.X, x = ps.x, H = a.H, K = 4 * H;
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = wave * 64 / COLS;
    const int col = tid % COLS, u = col >> 2, j0 = rank * UH, n = m * X + x;
    int q = tid & 3;
    const int piece = lr / BPL, blk = lr % BPL;
    const unsigned k_off = (unsigned)(s.slice * NB) * 64u + (unsigned)(lk * s.n_blk + blk) * 16u;
    const unsigned slot = (unsigned)few_slot_bytes(MODE, K);
    const bool polls = s.slice < s.n_slices;
    const unsigned w_off = (unsigned)(m * K + j0 * 4 + col) * es;       // inside a slot
    const unsigned dz_off = (unsigned)(n * K + j0 * 4 + col) * es;      // inside a timestep's dz rows
    const unsigned g_col = (unsigned)(n * K + j0 * 4 + col) * 4u, h_col = (unsigned)(n * H + j0 + u) * 4u;
    constexpr int WHOLE = (int)0x80000000u;
    const __amdgpu_buffer_rsrc_t rs_dz = __builtin_amdgcn_make_buffer_rsrc(a.dz, 0, WHOLE, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_ring = __builtin_amdgcn_make_buffer_rsrc(ring, 0, (int)(FEW_RING * slot), 0x00020000);
    int edge = s.c_wait * pl.ct;   // consumer: first timestep of the lowest chunk waited for
    unsigned so_w = (unsigned)(t & (FEW_RING - 1)) * slot;
    int off_bs = -1;
    unsigned off[L];
    u32x4_t raw[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
        raw[i] = u32x4_t{0u, 0u, 0u, 0u};
        off[i] = QUAD_NOWHERE;
    }
    bar_lds();   // (the partial sums of the phase before have been read)
    few_clear_part<UH>(s.part);
    bar_lds();

    int bs = grp_count(s.bs_t, ps), bs_up = grp_count(s.bs_up, ps), bs_1 = grp_count(s.bs_m1, ps), bs_2 = grp_count(s.bs_m2, ps);
    bool alive = true;
    for (;;) {   // (see the forward loop)
        quad_again(q);
        unsigned word = 0;
        // A. gate gradients
        if (m < bs) {
            const bool carried = m < bs_up;
            const float dh = d.f.dh_above + (carried ? d.dh : 0.f);
            const float dc = dh * d.f.dc + (carried ? d.dc : 0.f);
            const float dz = (q == 3 ? dh : dc) * d.f.dz;
            if constexpr (MODE == MODE_BF16) {
                const unsigned w = to_bf16_finite(dz);
                word = few_word(w | (few_dpp<0xb1>(w) << 16));   // (quad_perm 1,0,3,2; used by even lanes)
            } else {
                word = few_word(__float_as_uint(dz));
            }
            if (t > 0 && (MODE == MODE_F32 || (q & 1) == 0)) __builtin_amdgcn_raw_buffer_store_b32(word, rs_ring, w_off, so_w, 0);
            d.db += dz;
            d.dc = dc * d.f.gf;
        }
        if (bs != off_bs) {
            off_bs = bs;
            quad_offsets<L, BPL>(off, (unsigned)(piece * K) * es + k_off, piece < bs, blk, s.n_blk);
        }
        if (!LATE && polls && t > 0) quad_request<L>(rs_ring, off, so_w, raw);
        __builtin_amdgcn_sched_barrier(0);
        unsigned so_dz = (unsigned)s.base * (unsigned)(K * es);
        if (t == 0) {   // nothing is carried before the first timestep
            if (m < bs && (MODE == MODE_F32 || (q & 1) == 0)) __builtin_amdgcn_raw_buffer_store_b32(word, rs_dz, dz_off, so_dz, (PIPE & PIPE_PRODUCER) ? 17 : 0);
            --t;
            break;
        }
        const int bs_3 = grp_count(d.bs_m3, ps);
        s.win.advance(t - 4);
        int to_edge = 0x7fffffff;   // consumer: timesteps until the chunk below has to be there
        if (PIPE & PIPE_CONSUMER) {
            if (t - 3 < edge && t >= 3) {
                --s.c_wait;
                if (!s.ready && !pipe_wait_chunk(pl, s.c_wait, a.err)) {
                    alive = false;
                    break;
                }
                s.ready = false;
                edge -= pl.ct;
            }
            if (edge > 0) to_edge = t - 2 - edge;
        }
        // what of timestep t-1 is known
        if (m < min(bs_1, QUAD_MAX)) {
            d.c = m < bs ? d.c_prev : d.r0.c;
            d.f = quad_factor(d.r0, d.c, q);
            d.c_prev = d.r0.c_prev;
        }
        unsigned base_3 = (unsigned)(s.base - s.bs_m1 - s.bs_m2 - d.bs_m3);
        unsigned so_e = (unsigned)((t + 1) & (FEW_RING - 1)) * slot;
        quad_now(base_3); quad_now(so_dz); quad_now(so_e);
        // B. dh carried to t-1: dh[piece][k] = sum_q dz[piece][q] * W_hh[q][k] for this workgroup's columns k
        bool ok = true;
        if (LATE) {
            __builtin_amdgcn_sched_barrier(0);
            if (polls) quad_request<L>(rs_ring, off, so_w, raw);
        }
        if (polls) ok = quad_arrived<L>(rs_ring, off, so_w, raw, a.err);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (also: this wave's dz rows of timestep t+1 have completed)
        quad_touch(d.r1);
        few_touch(s.win.cur);
        few_touch(s.win.other);
        if (PIPE & PIPE_CONSUMER) few_touch(s.have);
        if (!ok) *s.fail = 1;
        const int bs_m4 = s.win.at(t - 4);
        d.r0 = d.r1;
        float* part = s.part + (t & 1) * (REC_WAVES * PART);
        quad_product<MODE, MT, NB, P, L>(s.w, raw, bs, s.n_blk, part + s.slice * PART, polls, [&]() __attribute__((always_inline)) {
            // the dz rows of this timestep, the saved activations of timestep t-3
            if (m < bs_3 && m < QUAD_MAX) quad_load_saved(d.r1, a, m, n, g_col, h_col, t - 3, bs_2, (int)base_3, (int)base_3 - bs_m4);
            if (m < bs && (MODE == MODE_F32 || (q & 1) == 0)) __builtin_amdgcn_raw_buffer_store_b32(word, rs_dz, dz_off, so_dz, (PIPE & PIPE_PRODUCER) ? 17 : 0);
        });
        // a look at the chunk that the next timestep asks for, see the forward loop
        if ((PIPE & PIPE_CONSUMER) && to_edge <= 2) {
            if (to_edge == 1) {
                if (tid == REC_THREADS - 1) s.fail[1] = s.have;
                s.have = 0;
            } else if (tid == REC_THREADS - 1) {
                s.have = ld_agent(&pl.done[s.c_wait - 1]);
            }
        }
        bar_lds();
        const int failed = *s.fail;
        // Every workgroup has published the rows of timestep t, which it did after its dz rows of timestep t+2 had
        // completed (they are stored in that timestep and waited for in timestep t+1).
        if ((PIPE & PIPE_PRODUCER) && rank == 0 && tid == REC_THREADS - 1 && t + 2 < T) st_agent(pl.progress, T - (t + 2));
        if (m < bs) {
            const float* p = part + m * ROW + u + 2 * q * PART;   // (a lane adds two of the eight)
            d.dh = quad_sum(p[0] + p[PART]);
            if (MODE == MODE_F32 || (q & 1) == 0) __builtin_amdgcn_raw_buffer_store_b32(FEW_EMPTY, rs_ring, w_off, so_e, 0);
        }
        if ((PIPE & PIPE_CONSUMER) && to_edge == 1) s.ready = __builtin_amdgcn_readfirstlane(s.fail[1]) >= few_scalar(pl.need);
        if (__builtin_amdgcn_readfirstlane(failed)) {
            alive = false;
            break;
        }
        s.base -= s.bs_m1;
        s.bs_up = s.bs_t;
        s.bs_t = s.bs_m1;
        s.bs_m1 = s.bs_m2;
        s.bs_m2 = d.bs_m3;
        d.bs_m3 = bs_m4;
        bs_up = bs;
        bs = bs_1;
        bs_1 = bs_2;
        bs_2 = bs_3;
        so_w = (unsigned)((t - 1) & (FEW_RING - 1)) * slot;
        if (--t < t_stop || bs > P) break;
    }
    return alive;
}

// Timesteps from t = T-1 down to t_stop while at most QUAD_MAX pieces are alive; s as few_bwd sets it up, without what is saved.
template <int MODE, int MT, int NB, int PIPE>
__device__ __forceinline__ bool quad_bwd(FewBwd<MODE, MT, NB>& s, const RecBwdArgs& a, const PieceSet& ps, int rank, unsigned char* ring, const PipeLink& pl,
                                         int& t, int T, int t_stop) {
    typedef QuadBwd<MODE, MT, NB, PIPE> D;
    constexpr int UH = D::UH, COLS = D::COLS;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = wave * 64 / COLS, col = tid % COLS, q = tid & 3, u = col >> 2, j0 = rank * UH, n = m * ps.X + ps.x, H = a.H, K = 4 * H;
    const unsigned g_col = (unsigned)(n * K + j0 * 4 + col) * 4u, h_col = (unsigned)(n * H + j0 + u) * 4u;
    if (grp_count(s.bs_t, ps) > QUAD_MAX) return true;
    D d;
    d.dh = d.dc = d.c = d.db = 0.f;
    d.r0.g = d.r0.c_prev = d.r0.dh_above = d.r0.c = 0.f;
    d.r1 = d.r0;
    d.bs_m3 = s.win.at(t - 3);
    if (PIPE & PIPE_CONSUMER)   // saved gradients of timesteps down to t-2 are read here
        while (s.c_wait > 0 && t - 2 < s.c_wait * pl.ct) {
            --s.c_wait;
            if (!pipe_wait_chunk(pl, s.c_wait, a.err)) return false;
        }
    QuadSaved r = d.r0;
    const int base_1 = s.base - s.bs_m1, base_2 = base_1 - s.bs_m2, base_3 = base_2 - d.bs_m3;
    // (pieces alive: 0 before the first timestep)
    const int bs = grp_count(s.bs_t, ps), bs_1 = grp_count(s.bs_m1, ps), bs_2 = grp_count(s.bs_m2, ps);
    if (m < bs) quad_load_saved(r, a, m, n, g_col, h_col, t, 0, s.base, base_1);
    if (m < bs_1 && m < QUAD_MAX) quad_load_saved(d.r0, a, m, n, g_col, h_col, t - 1, bs, base_1, base_2);
    if (m < bs_2 && m < QUAD_MAX) quad_load_saved(d.r1, a, m, n, g_col, h_col, t - 2, bs_1, base_2, base_3);
    quad_touch(d.r0);   // (the loads are complete before the loop)
    quad_touch(d.r1);
    d.f = quad_factor(r, r.c, q);
    d.c = r.c;
    d.c_prev = r.c_prev;
    // (as few loads per poll as hold the pieces: one of one or two pieces, up to four of four)
    constexpr int LOW = 16 / NB;
    if (bs <= LOW && !quad_bwd_loop<MODE, MT, NB, LOW, PIPE>(d, s, a, ps, rank, ring, pl, t, T, t_stop)) return false;
    if (LOW < QUAD_MAX && t >= t_stop && grp_count(s.bs_t, ps) <= QUAD_MAX &&
        !quad_bwd_loop<MODE, MT, NB, QUAD_MAX, PIPE>(d, s, a, ps, rank, ring, pl, t, T, t_stop)) return false;
    // to a thread per (piece, unit)
    bar_lds();
    float* const p = s.part;
    if (m < QUAD_MAX) {
        p[tid] = d.db;
        if (q == 0) {
            p[QUAD_MAX * COLS + m * UH + u] = d.dh;
            p[QUAD_MAX * (COLS + UH) + m * UH + u] = d.dc;
            p[QUAD_MAX * (COLS + 2 * UH) + m * UH + u] = d.c;
        }
    }
    bar_lds();
    if (tid < QUAD_MAX * UH) {
        const f32x4_t db = *reinterpret_cast<const f32x4_t*>(p + tid * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) s.db[i] += db[i];
        s.dh = p[QUAD_MAX * COLS + tid];
        s.dc = p[QUAD_MAX * (COLS + UH) + tid];
        s.c = p[QUAD_MAX * (COLS + 2 * UH) + tid];
    }
    return true;
}

}  // namespace ver
