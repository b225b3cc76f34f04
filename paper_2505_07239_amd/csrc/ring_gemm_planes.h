// The int8 matrix-core kernel of the share calls whose weight-side operands arrive as digit planes
// (COMET_WEIGHT_PLANES; see ring_gemm.hip for the formulation and wplanes.hip for the format).
//
// Both operands are stored in matrix-instruction operand order: a 16-byte unit holds one digit of
// sixteen contraction words of one row (activations) or one column (weights), and a lane of
// v_mfma_i32_16x16x64_i8 takes exactly one unit per operand.  A work unit is a PAIR of contraction
// steps (2 x 32 words, the 64 of the instruction); the stacked contraction has 2 KS steps, so a tile has
// KS pairs, and the pair in the middle may take its two steps from different halves.
//
// What bounds it is power.  Secret shares are uniformly random words, and on random operands the chip
// lowers its clock: in a register-resident loop (comet_probe_mfma_i8) 32x32x32 sustains 3.3 POP/s and
// 16x16x64 sustains 3.8 POP/s (32x32x32 on constants: 4.2 to 4.8), so the smaller instruction is used
// although it reads its operands from registers twice as often.  The second lever is the data movement
// beside the multipliers:
//   * activation units go from memory (L2, for the most part) straight into the registers of the
//     wavefront that multiplies them.  The digit pairs are walked with the activation digit
//     descending, so a digit's fragments are used in one run of instructions and then dead: its
//     registers take the same digit of the NEXT pair at once, and the load has a whole pair of steps
//     (about 2.3 us) to arrive.  Nothing is staged twice, and LDS sees a third of the traffic it would
//     carry with both operands in it;
//   * weight units pass through LDS (two stages), because two (128 x 64 tile) wavefronts need them, by
//     LDS-DMA: no registers, no LDS store instructions.  The fragments of a pair are read once and
//     stay in registers to its end;
//   * one barrier per pair, in its middle: barrier b_n publishes the weight stage of pair n + 1
//     (requested behind b_(n-1), a whole pair earlier) and retires the stage of pair n, all of whose
//     reads are older; the transfers for pair n + 2 then overwrite it.  No instruction waits for
//     something requested shortly before.
// Measured against 32x32x32 with both operands staged in LDS (three stages, one barrier per 32 words):
// 512 x 11008 x 4096 dense 1213 -> 1057 us (3.1 POP/s, matrix pipe busy 81 % of the cycles at 1.87 GHz:
// profiles/bench_c5_d100_mfma_counters.md), four products of 256 x 4096 x 1664 in one launch 413 -> 365
// us, one of them 128 -> 111 us a call.  The order of the digit pairs and of the two operands does not
// matter to the power (twelve orders in a register-resident loop agree within 3 %).
#pragma once

#include "ring_gemm_kernel.h"

namespace comet_gemm {

// Output tile of WAVES_M x WAVES_N wavefronts (four, one per SIMD), each with MT x NT sub-tiles of
// 16 x 16 outputs in eight digit planes: 4 x 2 sub-tiles fill the 256 accumulator registers.  The tile with
// 2 x 2 of them, 64 x 64, is for small products: a pair of steps takes 1.1 us there and 2.2 us on the others,
// and that is the least a workgroup can do (see planes_narrow_bn in ring_gemm.hip for where the line lies).
template <int WAVES_M, int WAVES_N, int MT_, int NT_>
struct PlaneTile {
    static constexpr int MT = MT_, NT = NT_;
    static constexpr int BM = 16 * MT * WAVES_M;
    static constexpr int BN = 16 * NT * WAVES_N;
    static constexpr int CHUNKS = BN / 64;                 // column chunks of the weight planes per tile
    static constexpr int WSTAGE = BN * KPAIR * 8;          // bytes of a weight stage
    static constexpr int RUNS = 8 * CHUNKS;                // LDS-DMA transfers per wavefront and stage
    static_assert(WAVES_M * WAVES_N * 64 == GT, "four wavefronts per workgroup");
    static_assert(BN % 64 == 0, "a wavefront's transfer is one run of 64 columns");
};

// Positions inside a pair, counted in matrix instructions.  Group gi (0 .. 7) multiplies activation
// digit 7 - gi with the weight digits 0 .. gi.
template <class T>
struct PairMap {
    static constexpr int Q = T::MT * T::NT;
    static constexpr int NM = 36 * Q;
    static constexpr int group_begin(int gi) { return gi * (gi + 1) / 2 * Q; }
    static constexpr int group_of(int m) {
        int g = 0;
        while (m >= group_begin(g + 1)) ++g;
        return g;
    }
    static constexpr int t_of(int m) { return 7 - group_of(m); }
    static constexpr int u_of(int m) { return (m - group_begin(group_of(m))) / Q; }
    static constexpr int i_of(int m) { return (m % Q) / T::NT; }
    static constexpr int j_of(int m) { return m % T::NT; }
    // The registers of weight digit u are free from the end of its last use (group 7) on, and its
    // first use is at the end of group u.  Digits 0 and 1 are read from the next pair's stage near the end of
    // a pair, the others at the start of their own: all reads of a stage are behind it at BARRIER.
    static constexpr bool read_ahead(int u) { return u < 2; }
    static constexpr int read_slot(int u) {
        return read_ahead(u) ? NM - (2 - u) * (Q < 4 ? Q : Q / 2 + Q / 4) - Q : (u - 2) * 2 * Q;
    }
    static constexpr int BARRIER = group_begin(5) + Q;     // (digits of groups 0 .. 4 are reloaded before it)
    // activation digit t is requested again, sub-tile by sub-tile, behind its group
    static constexpr int reload_slot(int t) { return group_begin(8 - t) % NM; }
    static_assert(read_slot(7) + 2 * Q <= BARRIER, "a stage is read before the barrier that retires it");
    static_assert(read_slot(0) > BARRIER && read_slot(0) >= group_begin(7) + Q, "the next stage is published, the registers free");
    static_assert(read_slot(1) >= group_begin(7) + 2 * Q && read_slot(1) < NM, "the registers are free");
    // vector-memory loads issued behind the last LDS-DMA transfer of a stage and ahead of the next
    // barrier: at least this many (activation digits 1, 0, 7, 6, 5, 4)
    static constexpr int YOUNGER = 6 * T::MT;
};

template <class T, int KIND, int GMODE, bool LISTED>
struct PlaneStage {
    typedef __attribute__((address_space(1))) const char* gptr;
    unsigned pcb[T::CHUNKS], pcf[T::CHUNKS];   // lane's byte offset of its column in a contraction step: B_i, F
    gptr ap;                                   // this lane's activation unit of the digit requested next
    size_t adig;                               // bytes from one activation digit to the next
    u32 astep;                                 // bytes of one contraction step of the activation planes
    gptr abase;                                // this lane's unit of step 0, digit 0
    gptr wb;                                   // weight planes of the stage being requested: this wavefront's run of digit 0
    unsigned wcol[T::CHUNKS];
    const int* tab;                            // LDS: per position of the segment {x step, first row of k-half 0, of k-half 1, half}
    const int* steps;                          // listed contraction steps of this row tile, or null

    __device__ __forceinline__ void setup(const GemmParams& p, int row0, int tn, int n_eff) {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int c = 0; c < T::CHUNKS; ++c) {
            int col = tn * T::BN + c * 64 + lane;
            col = col < n_eff ? col : n_eff - 1;
            long bcol = col;
            if (KIND == KIND_SOMM && p.b_full) {
                const int blk = col / p.bs;
                const long st = block_start(p, blk);
                bcol = (st < 0 ? 0 : st) + (col - blk * p.bs);
            }
            // chunk of 64 columns, then the column inside it (columns stay below 2^24: host check)
            pcb[c] = ((unsigned)bcol >> 6) * 16384u + ((unsigned)bcol & 63u) * 16u;
            pcf[c] = ((unsigned)col >> 6) * 16384u + ((unsigned)col & 63u) * 16u;
        }
        adig = (size_t)p.mpad * 32;
        astep = (u32)p.mpad * 256u;            // (rows stay below 2^22: host check)
        // a lane's k-group of the 64: two 16-word halves of two steps
        abase = (gptr)p.xp + ((size_t)((lane >> 4) & 1) * p.mpad + row0 + (lane & 15)) * 16;
    }

    // Table of the segment: positions 2 q0 .. 2 (q0 + L) of the stacked contraction (all threads;
    // the caller synchronises).  Rows past the end of the contraction keep a valid address: their
    // activation digits are zero.
    __device__ __forceinline__ void build_table(const GemmParams& p, int* table, int q0, int L, int KS, int kc) {
        for (int q = threadIdx.x; q < 2 * L; q += GT) {
            const int ks = 2 * q0 + q;
            const int h = ks >= KS ? 1 : 0;
            int s = ks - h * KS;
            if constexpr (LISTED) s = steps[s];
            int n0[2];
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int k0 = s * KSTEP + 16 * g;
                n0[g] = k0;
                if (GMODE == W_PLANES_GATHER && h == 0) {
                    // bs is a multiple of 16 (host check), so a half lies inside one block
                    const int kb = k0 <= kc - 16 ? k0 : kc - 16;
                    const int blk = kb / p.bs;
                    const long st = block_start(p, blk);
                    n0[g] = (int)(st < 0 ? 0 : st) + (kb - blk * p.bs);
                }
            }
            *reinterpret_cast<v4i*>(table + 4 * q) = v4i{(h ? p.xstep[1] : p.xstep[0]) + s, n0[0], n0[1], h};
        }
        tab = table;
    }

    // activation units of pair q: each lane looks up the step its k-group belongs to
    __device__ __forceinline__ int a_step(int q) const {
        return tab[4 * (2 * q + (int)((threadIdx.x & 63) >> 5))];
    }
    __device__ __forceinline__ void a_begin(int x) { ap = abase + (size_t)(u32)x * astep + 7 * adig; }
    __device__ __forceinline__ v4i a_load(int i) const {
        return *reinterpret_cast<__attribute__((address_space(1))) const v4i*>(ap + i * 256);
    }

    // Weight stage of pair q: wavefront w moves the runs of k-group w (step w / 2 of the pair,
    // k-half w % 2), digit by digit.
    __device__ __forceinline__ v4i w_entry(int q) const {
        return *reinterpret_cast<const v4i*>(tab + 4 * (2 * q + (int)(threadIdx.x >> 7)));
    }
    __device__ __forceinline__ void w_begin(const GemmParams& p, v4i e) {
        const int r0 = __builtin_amdgcn_readfirstlane((threadIdx.x & 64) ? e.z : e.y);
        const int h = __builtin_amdgcn_readfirstlane(e.w);
        const size_t prow = (size_t)(((h ? p.ldf : p.ldb) + 63) >> 6) * 16384u;
        wb = (gptr)(h ? p.F : p.B) + (size_t)(r0 >> 5) * prow + (size_t)((r0 >> 4) & 1) * 1024u;
#pragma unroll
        for (int c = 0; c < T::CHUNKS; ++c) wcol[c] = pcb[c] + ((pcf[c] - pcb[c]) & (0u - (unsigned)h));
    }
    // Issued as plain text so that the compiler's own wait-count bookkeeping does not treat every
    // later LDS read as dependent on this transfer; what orders it is the explicit wait at the
    // barrier.  M0 carries the wavefront's LDS address.
    template <int J>
    __device__ __forceinline__ void w_piece(unsigned lds_stage) {
        constexpr int u = J / T::CHUNKS, c = J % T::CHUNKS;
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const unsigned lds = __builtin_amdgcn_readfirstlane(lds_stage + ((u * 4 + wave) * T::BN + c * 64) * 16);
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(lds), "v"(wcol[c]), "s"(wb + u * 2048)
                     : "memory", "m0");
    }
    template <int... Js>
    __device__ __forceinline__ void w_stage(std::integer_sequence<int, Js...>, unsigned lds_stage) {
        (w_piece<Js>(lds_stage), ...);
    }
};

// acc += a b.  Written out so that the accumulators stay where they are, in the 256 accumulation
// registers: from the builtin the compiler builds a three-address form, permutes the accumulators
// around the loop and spills fragments.  (The same accumulator is not used again for at least four
// instructions, and mfma_done() ends the pair: the compiler does not know that these are matrix instructions and adds no
// wait of its own before another use of their results.)
__device__ __forceinline__ void mfma_acc(v4i& acc, const v4i& a, const v4i& b) {
    asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// Wait states from the last matrix instruction to any other access to its result: eight (four passes), BETWEEN of them
// taken by instructions that follow it. They stand at the end of the loop body and not behind the loop, where a
// register copy, which is no memory access, could still be placed ahead of them; the matrix pipe is busy meanwhile.
template <int BETWEEN>
__device__ __forceinline__ void mfma_done() {
    asm volatile("s_nop %0" ::"n"(7 - BETWEEN) : "memory");
}

template <class T, int KIND, int GMODE, bool LISTED, int... Ms>
__device__ __forceinline__ void plane_pair(std::integer_sequence<int, Ms...>, const GemmParams& p,
                                           PlaneStage<T, KIND, GMODE, LISTED>& st, v4i (&acc)[T::MT][T::NT][8],
                                           v4i (&a)[8][T::MT], v4i (&b)[8][T::NT], const unsigned char* rd,
                                           const unsigned char* rd_next, unsigned fill, int q_next, int q_fill) {
    using PM = PairMap<T>;
    int x_next = 0;
    v4i w_next = {0, 0, 0, 0};
    (
        [&] {
            constexpr int M = Ms;
            if constexpr (M == 0) x_next = st.a_step(q_next);
            if constexpr (M == PM::BARRIER - PM::Q) w_next = st.w_entry(q_fill);
            if constexpr (M == PM::BARRIER) {
                wait_and_barrier<PM::YOUNGER>();
                st.w_begin(p, w_next);
            }
            constexpr int t = PM::t_of(M), u = PM::u_of(M), i = PM::i_of(M), j = PM::j_of(M);
            mfma_acc(acc[i][j][t + u], a[t][i], b[u][j]);
            // weight fragments
            [&]<int... Us>(std::integer_sequence<int, Us...>) {
                ([&] {
                    constexpr int off = M - PM::read_slot(Us);
                    if constexpr (off >= 0 && off < T::NT)
                        b[Us][off] = lds_frag((PM::read_ahead(Us) ? rd_next : rd) + (Us * 4 * T::BN + off * 16) * 16);
                }(), ...);
            }(std::make_integer_sequence<int, 8>{});
            // activation fragments of the next pair
            [&]<int... Ts>(std::integer_sequence<int, Ts...>) {
                ([&] {
                    constexpr int off = M - PM::reload_slot(Ts);
                    if constexpr (Ts > 0 && off >= 0 && off < T::MT) {
                        if constexpr (Ts == 7 && off == 0) st.a_begin(x_next);
                        a[Ts][off] = st.a_load(off);
                        if constexpr (off == T::MT - 1) st.ap -= st.adig;
                    }
                }(), ...);
            }(std::make_integer_sequence<int, 8>{});
            if constexpr (M > PM::BARRIER) {
                constexpr int gap = 2, n = M - PM::BARRIER - 1;
                if constexpr (n % gap == 0 && n / gap < T::RUNS) st.template w_piece<n / gap>(fill);
            }
            __builtin_amdgcn_sched_barrier(0);
        }(),
        ...);
    // digit 0 of the next pair, behind the last group
#pragma unroll
    for (int i = 0; i < T::MT; ++i) a[0][i] = st.a_load(i);
    __builtin_amdgcn_sched_barrier(0);
    mfma_done<T::MT>();
}

// One workgroup's share of a product: segment by segment, the main loop and the write-out of the
// partial sum.
template <class T, int WAVES_M, int KIND, int GMODE, bool LISTED>
__device__ __forceinline__ void plane_sweep(const GemmParams& p, const Geometry& q, UnitWalk<LISTED>& walk,
                                            const bool own, unsigned char* wsm, int* steptab) {
    using PM = PairMap<T>;
    constexpr int MT = T::MT, NT = T::NT;
    const int n_eff = q.n_eff, kc = q.kc, m_eff = q.m_eff;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wm = wave % WAVES_M, wn = wave / WAVES_M;
    const int g = lane >> 4, r = lane & 15;
    // this lane's weight fragment of digit 0 inside a stage
    const unsigned char* rd0 = wsm + (g * T::BN + wn * NT * 16 + r) * 16;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)wsm;

    PlaneStage<T, KIND, GMODE, LISTED> st;
    Segment sg;
    while (walk.next(sg)) {
        const int L = sg.L;
        const int row0 = sg.tm * T::BM + wm * MT * 16;
        st.setup(p, row0, sg.tn, n_eff);
        st.steps = sg.steps;
        // (the stages and the table of the previous segment are no longer read: every wavefront
        // has passed that segment's last barrier)
        st.build_table(p, steptab, sg.k0, L, sg.KS, kc);
        __syncthreads();

        v4i acc[MT][NT][8];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int s = 0; s < 8; ++s) acc[i][j][s] = v4i{0, 0, 0, 0};

        // prologue: the weight stages of pairs 0 and 1, the activation fragments of pair 0, digit 7 first
        st.w_begin(p, st.w_entry(0));
        st.w_stage(std::make_integer_sequence<int, T::RUNS>{}, lds0);
        st.w_begin(p, st.w_entry(1 < L ? 1 : L - 1));
        st.w_stage(std::make_integer_sequence<int, T::RUNS>{}, lds0 + T::WSTAGE);
        v4i a[8][MT], b[8][NT];
        st.a_begin(st.a_step(0));
#pragma unroll
        for (int t = 7; t >= 0; --t) {
#pragma unroll
            for (int i = 0; i < MT; ++i) a[t][i] = st.a_load(i);
            st.ap -= st.adig;
        }
        __builtin_amdgcn_sched_barrier(0);
        wait_and_barrier<8 * MT>();
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < NT; ++j) b[u][j] = lds_frag(rd0 + (u * 4 * T::BN + j * 16) * 16);

        // pair n reads stage n % 2; behind its barrier pair n + 2 is requested into that stage
        for (int n = 0; n < L; ++n) {
            const int odd = n & 1;
            plane_pair<T, KIND, GMODE, LISTED>(std::make_integer_sequence<int, PM::NM>{}, p, st, acc, a, b,
                                               rd0 + odd * T::WSTAGE, rd0 + (odd ^ 1) * T::WSTAGE,
                                               lds0 + odd * T::WSTAGE, n + 1 < L ? n + 1 : L - 1,
                                               n + 2 < L ? n + 2 : L - 1);
        }
        // the transfers requested for pairs beyond the last are redundant; let them land before the
        // stages are reused
        wait_and_barrier<0>();

        // The only writer of a tile (own) stores Z = C + sum (Z += sum for a later segment of a long
        // contraction: this lane's own earlier store, complete since the barrier above); the loads of
        // a sub-tile go out together, ahead of the arithmetic.  Slices of a shared tile meet in Z,
        // which started out as C, through atomic adds.
        const u64* src = sg.k0 == 0 ? p.C : p.Z;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int col = sg.tn * T::BN + (wn * NT + j) * 16 + r;
            const int ccomp = (p.row_comp && col < n_eff) ? p.blk_comp[col / p.bs] : 0;
            u64 prev[MT][4];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = row0 + i * 16 + 4 * g + e;
                    prev[i][e] = 0;
                    if (own && row < m_eff && col < n_eff) prev[i][e] = src[(size_t)row * p.ldz + col];
                }
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = row0 + i * 16 + 4 * g + e;
                    const v4i (&s)[8] = acc[i][j];
                    const u64 z = recombine(s[0][e], s[1][e], s[2][e], s[3][e], s[4][e], s[5][e], s[6][e], s[7][e]);
                    bool live = row < m_eff && col < n_eff;
                    if (live && p.row_comp) live = p.row_comp[row] == ccomp;   // on a result block
                    if (live) {
                        if (own) p.Z[(size_t)row * p.ldz + col] = prev[i][e] + z;
                        else atomicAdd(p.Z + (size_t)row * p.ldz + col, z);
                    }
                }
        }
    }
}

#define COMET_PLANES_LDS(T)                                          \
    __shared__ __align__(16) unsigned char wsm[2 * T::WSTAGE];       \
    __shared__ __align__(16) int steptab[MAX_SEG * 4]

// OWN: see ring_gemm_kernel
template <int WAVES_M, int WAVES_N, int MT, int NT, int KIND, int GMODE, bool LISTED, bool OWN>
__global__ __launch_bounds__(GT, 1) void ring_planes_kernel(GemmParams p) {
    using T = PlaneTile<WAVES_M, WAVES_N, MT, NT>;
    COMET_PLANES_LDS(T);
    if (p.tile_sel && *p.tile_sel != p.tile_sel_want) return;   // the other tile shape was chosen
    const Geometry q = gemm_geometry<T::BM, T::BN, KIND, LISTED>(p);
    if (q.units == 0) return;
    const int G = gridDim.x;
    const int b = xcd_contiguous(blockIdx.x, G);
    bool own = false;
    if constexpr (OWN) own = owns_tiles(p, q.m_eff, q.n_eff, q.kc);
    UnitWalk<LISTED> walk(p, q, b, G, own);
    plane_sweep<T, WAVES_M, KIND, GMODE, LISTED>(p, q, walk, own, wsm, steptab);
}

// Several products of one shape and one index list (so: one geometry) in one launch: the work
// units of the members follow each other, tile by tile inside a member, and the workgroups share
// out the whole sequence.  A workgroup's range may run across members.
template <int WAVES_M, int WAVES_N, int MT, int NT, int KIND, int GMODE, bool OWN>
__global__ __launch_bounds__(GT, 1) void ring_planes_group_kernel(GemmGroup grp) {
    using T = PlaneTile<WAVES_M, WAVES_N, MT, NT>;
    COMET_PLANES_LDS(T);
    const Geometry q = gemm_geometry<T::BM, T::BN, KIND, false>(grp.p[0]);
    if (q.units == 0) return;
    const int G = gridDim.x;
    const int b = xcd_contiguous(blockIdx.x, G);
    // Teams: when the row tiles divide the grid, tiles_m consecutive workgroups (same XCD) form a
    // team that walks one sequence of (column tile, contraction unit) pairs, each member for its
    // own row tile: the weight planes of a unit are fetched once for all row tiles, in lockstep.
    const bool team = grp.p[0].team && q.tiles_m > 1 && G % q.tiles_m == 0;
    const long units = team ? q.units / q.tiles_m : q.units;        // of one member
    const int parts = team ? G / q.tiles_m : G, part = team ? b / q.tiles_m : b;
    const long total = units * grp.n;
    long u = total * part / parts;
    const long u_end = total * (part + 1) / parts;
    bool own = false;
    if constexpr (OWN) own = owns_tiles(grp.p[0], q.m_eff, q.n_eff, q.kc);
#pragma nounroll
    for (int j = (int)(u / units); u < u_end; ++j) {
        const long base = (long)j * units;
        const long hi = u_end - base < units ? u_end - base : units;
        UnitWalk<false> walk(grp.p[j], q, u - base, hi, team ? b % q.tiles_m : -1);
        plane_sweep<T, WAVES_M, KIND, GMODE, false>(grp.p[j], q, walk, own, wsm, steptab);
        u = base + units;
    }
}

// The kernel variant for a call, instantiated explicitly in translation units of their own
// (ring_gemm_planes_*.hip, ring_gemm_group_*.hip).  The 128 x 64 tile has no variants for step lists
// (the dispatch picks 64 or 32 rows for them), the others none for owned tiles.
template <int WAVES_M, int WAVES_N, int MT, int NT, bool LISTED, bool OWN>
GemmKernel planes_kernel_for(const GemmParams& p) {
    if (p.kind == KIND_SIMM) {
        if (p.b_full) return ring_planes_kernel<WAVES_M, WAVES_N, MT, NT, KIND_SIMM, W_PLANES_GATHER, LISTED, OWN>;
        return ring_planes_kernel<WAVES_M, WAVES_N, MT, NT, KIND_SIMM, W_PLANES, LISTED, OWN>;
    }
    if constexpr (LISTED) return nullptr;      // step lists belong to Protocol 3
    else return ring_planes_kernel<WAVES_M, WAVES_N, MT, NT, KIND_SOMM, W_PLANES, false, OWN>;
}
extern template GemmKernel planes_kernel_for<2, 2, 4, 2, false, false>(const GemmParams&);
extern template GemmKernel planes_kernel_for<2, 2, 4, 2, false, true>(const GemmParams&);
extern template GemmKernel planes_kernel_for<1, 4, 4, 2, false, false>(const GemmParams&);
extern template GemmKernel planes_kernel_for<2, 2, 2, 2, false, false>(const GemmParams&);
extern template GemmKernel planes_kernel_for<2, 2, 2, 2, true, false>(const GemmParams&);
extern template GemmKernel planes_kernel_for<1, 4, 4, 2, true, false>(const GemmParams&);
extern template GemmKernel planes_kernel_for<1, 4, 2, 2, false, false>(const GemmParams&);
extern template GemmKernel planes_kernel_for<1, 4, 2, 2, true, false>(const GemmParams&);

template <int WAVES_M, int WAVES_N, int MT, int NT>
int launch_planes(comet_ctx* ctx, const char* what, const GemmParams& p) {
    using T = PlaneTile<WAVES_M, WAVES_N, MT, NT>;
    GemmKernel kern = nullptr;
    if constexpr (T::BM == 128) {
        if (!p.step_list)
            kern = p.own_try ? planes_kernel_for<WAVES_M, WAVES_N, MT, NT, false, true>(p)
                             : planes_kernel_for<WAVES_M, WAVES_N, MT, NT, false, false>(p);
    } else {
        if (!p.own_try)
            kern = p.step_list ? planes_kernel_for<WAVES_M, WAVES_N, MT, NT, true, false>(p)
                               : planes_kernel_for<WAVES_M, WAVES_N, MT, NT, false, false>(p);
    }
    if (!kern || !p.w_planes) return comet_fail(ctx, COMET_EINVAL, "%s: no kernel variant for this call", what);
    if (p.tile_bm != T::BM || p.tile_bn != T::BN || p.grid < 1)
        return comet_fail(ctx, COMET_EINVAL, "%s: launch plan does not match the kernel", what);
    return launch_share_kernel(ctx, what, kern, dim3((unsigned)p.grid), p);
}

template <int WAVES_M, int WAVES_N, int MT, int NT, bool OWN>
GemmGroupKernel planes_group_kernel_for(const GemmParams& p) {
    if (p.kind == KIND_SIMM) {
        if (p.b_full) return ring_planes_group_kernel<WAVES_M, WAVES_N, MT, NT, KIND_SIMM, W_PLANES_GATHER, OWN>;
        return ring_planes_group_kernel<WAVES_M, WAVES_N, MT, NT, KIND_SIMM, W_PLANES, OWN>;
    }
    return ring_planes_group_kernel<WAVES_M, WAVES_N, MT, NT, KIND_SOMM, W_PLANES, OWN>;
}
extern template GemmGroupKernel planes_group_kernel_for<2, 2, 4, 2, false>(const GemmParams&);
extern template GemmGroupKernel planes_group_kernel_for<2, 2, 4, 2, true>(const GemmParams&);

template <int WAVES_M, int WAVES_N, int MT, int NT>
int launch_planes_group(comet_ctx* ctx, const char* what, const GemmGroup& grp) {
    using T = PlaneTile<WAVES_M, WAVES_N, MT, NT>;
    const GemmParams& p = grp.p[0];
    if (grp.n < 1 || grp.n > GROUP_MAX || !p.w_planes || p.tile_bm != T::BM || p.tile_bn != T::BN || p.grid < 1)
        return comet_fail(ctx, COMET_EINVAL, "%s: launch plan does not match the grouped kernel", what);
    return launch_share_kernel(ctx, what, p.own_try ? planes_group_kernel_for<WAVES_M, WAVES_N, MT, NT, true>(p)
                                                    : planes_group_kernel_for<WAVES_M, WAVES_N, MT, NT, false>(p),
                               dim3((unsigned)p.grid), grp);
}

}  // namespace comet_gemm
