// The int8 matrix-core kernel on weight WORDS whose wavefronts load, split, stage and multiply in one instruction stream
// (see ring_gemm.hip for the formulation), with two output tiles: 32 x 256 up to 32 rows, where the product is bound by
// reading the weights and 2 KB of every weight row in one piece count for more than the matrix instructions; 64 x 64, two
// workgroups per compute unit, for products of few steps (takes_staged_tile() in ring_gemm.hip).  The loader that stages
// both operands, one contraction step, the stream-K kernel and its launcher.  More rows: ring_words.h, the smallest
// products: ring_fewrow.hip.
#pragma once

#include "ring_gemm_kernel.h"

namespace comet_gemm {

// how the weight-side rows of B_i are addressed (SIMM with a full-size B_i only)
constexpr int GATHER_NONE = 0;   // rows are the compact contraction index
constexpr int GATHER_POW2 = 1;   // block gather, bs a power of two >= 8
constexpr int GATHER_ANY = 2;    // block gather, any bs
// SOMM with neuron-major weights: B_i and F hold one row of k contiguous words per output column
constexpr int WEIGHTS_TR = 3;
template <int WAVES_M, int WAVES_N, int WM, int WN>
struct Tile {
    static constexpr int BM = 32 * WM * WAVES_M;
    static constexpr int BN = 32 * WN * WAVES_N;
    static constexpr int XBYTES = BM * 256;          // 8 digits x 2 k-halves x BM rows x 16 bytes
    static constexpr int WBYTES = BN * 256;
    static constexpr int XSTAGES = 3;                // written by LDS-DMA two steps ahead
    static constexpr int WSTAGES = 2;                // written from registers one step ahead
    static constexpr int WBASE = XSTAGES * XBYTES;
    static constexpr int SMEM = XSTAGES * XBYTES + WSTAGES * WBYTES;
    // four wavefronts, one per SIMD
    static constexpr int THREADS = GT;
    static_assert(WAVES_M * WAVES_N * 64 == GT, "four wavefronts per workgroup");
    static constexpr int XVEC = XBYTES / 16 / THREADS;    // 16-byte units per thread per stage
    static constexpr int WTASK = BN * 4 / GT;        // (column, octet) tasks per thread per stage
    // vector-memory loads a thread issues per step: the LDS-DMA units plus, per weight task,
    // eight 8-byte loads (or four 16-byte loads when the weights are neuron-major)
    // and one load of a block id with the power-of-two row gather
    static constexpr int vm_per_step(int gmode) {
        return XVEC + (gmode == WEIGHTS_TR ? 4 : 8) * WTASK + (gmode == GATHER_POW2 ? WTASK : 0);
    }
    // two workgroups share a compute unit when one needs at most half of its registers and LDS
    static constexpr int WG_PER_CU = (WM * WN == 1 && SMEM <= 80 * 1024) ? 2 : 1;
    static_assert(XVEC >= 1 && WTASK >= 1, "tile too small for the loader");
    static_assert(vm_per_step(GATHER_POW2) < 63, "outstanding-load counter has 6 bits");
    static_assert(SMEM <= 160 * 1024, "LDS of one CDNA4 compute unit");
};

// Loads and staging of the operands, cut into small pieces.
//
// A contraction step issues 36 * WM * WN matrix instructions.  Everything else
// a step has to do -- start the LDS-DMA of the activation planes two steps
// ahead, request the weight words of the step after next, turn the weight
// words of the next step (requested a step ago) into digit planes and store
// them to LDS -- is cut into pieces of a handful of instructions, and
// gemm_step() places a piece behind every second or third matrix instruction
// so that they execute in its shadow.
//
// Activation side: the packed digit planes go from global memory straight into
// LDS (global_load_lds_dwordx4: every lane supplies its own global address, the
// wavefront's 64 x 16 bytes land contiguously at a wave-uniform LDS address),
// so they occupy no registers and need no LDS store.
//
// Weight side: raw uint64 words into registers; one step later each word is
// split into digits and its register immediately reused for the next request.
// Every load is unconditional: out-of-range rows and columns are clamped to a
// valid address instead of being predicated off.  That is exact because
// (a) a weight column only feeds its own output column, and columns at or
// beyond the kept width are never written back, and (b) the packed activation
// planes hold zeros beyond the contraction length, so whatever the weight side
// reads there is multiplied by zero.
template <class T, int KIND, int GMODE, bool LISTED, bool NT>
struct Loader {
    static constexpr int W = T::WTASK;
    // Where this task's weight words are.  Without a row gather: pointers to (row 0, the task's
    // column) of B_i (column gather applied for SOMM) and of F; neuron-major weights: to the
    // column's own row of k words.  With a row gather (SIMM, full-size B_i): the byte offset of
    // the column inside a row; the row is wave-uniform, so a load is "scalar row address +
    // 32-bit lane offset" and the compiler has no per-load 64-bit vector addresses to keep
    // (it would form all of a step's addresses ahead of time and run out of registers on the
    // 32 x 256 tile).
    static constexpr bool ROW_GATHER = GMODE == GATHER_POW2 || GMODE == GATHER_ANY;
    unsigned cb[W], cf[W];
    const char* wbase;         // row gather: B_i or F, whichever half the look-ahead step is in
    // GATHER_POW2: the eight rows of a task's octet are consecutive, so a task keeps a running
    // (wave-uniform) row address that moves on by one row pitch per load, and the lane's column
    // offset of the half it is in: a load is two scalar additions and the load itself
    const char* wcur[W];
    size_t wpitch;
    unsigned csel[W];
    const u64* wb[W];
    const u64* wf[W];
    const unsigned char* xsrc; // this thread's first 16-byte unit of step (h = 0, s = 0)
    u64 wn[W][8];              // weight words in flight (requested one step before they are split)
    u64 wa[W][8];              // digits of the weight words being staged for the next step
    u32 pl[W][16];             // transposed digits: [t] = words 0..3, [8 + t] = words 4..7
    // wave-uniform state of the look-ahead step, set by begin()
    int h2, s2;
    int ld2;                   // row pitch of the weight-side source in words
    const unsigned char* xs2;
    size_t xstride;            // bytes between the 16-byte units one thread moves per step
    int g0[W];                 // GATHER_POW2: first gathered row of this task's octet
    int gpend[W];              // GATHER_POW2: block id requested for the step after this one
    const int* steps;          // listed contraction steps of this row tile, or null (all steps)

    static_assert(T::THREADS == GT, "the word loader is written for four wavefronts");
    static constexpr int XGRP_PER_PASS = GT / T::BM;         // groups covered by one pass of the block
    static_assert(GT % T::BM == 0, "tile rows must divide the block");

    // Piece list of one step, in execution order: the DMA issues, then task by task the eight
    // split-and-reload pieces, the four transposes and the eight LDS stores (task-major, so the
    // digits and transposed planes of a task are dead before the next task starts).
    static constexpr int P_DMA = 0;
    static constexpr int P_TASK = P_DMA + T::XVEC;
    static constexpr int PER_TASK = 8 + 4 + 8;
    static constexpr int P_END = P_TASK + PER_TASK * W;
    static constexpr int VM_PER_STEP = T::vm_per_step(GMODE);

    __device__ __forceinline__ void setup(const GemmParams& p, int tm, int tn, int n_eff) {
#pragma unroll
        for (int j = 0; j < W; ++j) {
            const int id = threadIdx.x + GT * j;
            int col = tn * T::BN + id % T::BN;
            col = col < n_eff ? col : n_eff - 1;
            long bcol = col;
            if (KIND == KIND_SOMM && p.b_full) {
                const int blk = col / p.bs;
                const long st = block_start(p, blk);
                bcol = (st < 0 ? 0 : st) + (col - blk * p.bs);
            }
            if (GMODE == WEIGHTS_TR) {
                // the column's own row of k words; the contraction index is then the word offset
                wb[j] = p.B + bcol * p.ldb;
                wf[j] = p.F + (long)col * p.ldf;
            } else if (ROW_GATHER) {
                cb[j] = (unsigned)bcol * 8u;      // columns stay below 2^24 (host check)
                cf[j] = (unsigned)col * 8u;
            } else {
                wb[j] = p.B + bcol;
                wf[j] = p.F + col;
            }
        }
        steps = nullptr;
        const int grp = threadIdx.x / T::BM, within = threadIdx.x % T::BM;
        xsrc = p.xp + ((size_t)grp * p.mpad + (size_t)tm * T::BM + within) * 16;
        xstride = (size_t)XGRP_PER_PASS * p.mpad * 16;
    }

    // block id that holds compact row octet (step ks, task j); GATHER_POW2 only
    // A position ks in [0, 2 KS) of the stacked contraction of this tile -> half h and step s.
    // Without a step list the positions are the steps themselves; with one (per-token row sets)
    // a half has KS listed steps and position q stands for step steps[q].
    __device__ __forceinline__ void resolve(int ks, int KS, int& h, int& s) const {
        h = ks >= KS ? 1 : 0;
        s = ks - h * KS;
        if constexpr (LISTED) s = steps[s];
    }

    __device__ __forceinline__ int gather_id(const GemmParams& p, int ks, int KS, int kc, int j) {
        int h, s;
        resolve(ks, KS, h, s);
        const int oct = __builtin_amdgcn_readfirstlane((int)((threadIdx.x + GT * j) / T::BN));
        const int k0 = s * KSTEP + oct * 8;
        const int kb = k0 <= kc - 8 ? k0 : kc - 8;
        // The index is the same for all lanes, but it is made a vector value on purpose (a zero
        // the compiler cannot see through): the id then arrives through the vector-memory queue,
        // in order with the weight words, instead of through a scalar load, whose counter is
        // shared with the LDS reads -- every fragment read of the step would wait for it.
        int lane_zero = 0;
        asm volatile("" : "+v"(lane_zero));
        return p.blk_idx[((kb >> p.bs_shift) & (h - 1)) + lane_zero];
    }

    // first step of a segment: nothing has been requested ahead yet
    __device__ __forceinline__ void prime(const GemmParams& p, int ks, int KS, int kc) {
        if (GMODE == GATHER_POW2) {
#pragma unroll
            for (int j = 0; j < W; ++j) gpend[j] = gather_id(p, ks, KS, kc, j);
        }
    }

    // Fix the step the following dma / load pieces work on.  Steps are visited in
    // order (ks, then ks + 1 capped at ks_limit), which lets the block id of the
    // next step be requested here, a whole step before it is needed (see gather_id()
    // for why that request is a vector load).
    __device__ __forceinline__ void begin(const GemmParams& p, int ks, int KS, int kc, int ks_limit) {
        resolve(ks, KS, h2, s2);
        h2 = __builtin_amdgcn_readfirstlane(h2);
        s2 = __builtin_amdgcn_readfirstlane(s2);
        ld2 = GMODE == WEIGHTS_TR ? 1 : (int)(h2 ? p.ldf : p.ldb);
        if (ROW_GATHER) {
            // both halves as one expression without control flow (h2 is 0 or 1): a branch inside a
            // step makes the compiler lose track of which loads are still in flight, and it then
            // waits for all of the previous step's at the first use
            // (a select between two pointers keeps their address space; going through integers
            // would turn the loads into flat loads, which also count against the LDS counter)
            wbase = reinterpret_cast<const char*>(h2 ? p.F : p.B);
        }
        xs2 = xsrc + (size_t)(h2 * p.ks_cap + s2) * 16 * p.mpad * 16;
        if (GMODE == GATHER_POW2) {
            const int ksn = ks + 1 < ks_limit ? ks + 1 : ks_limit;
#pragma unroll
            for (int j = 0; j < W; ++j) {
                // consumed here, ahead of the fragment reads (the scheduling fence that follows
                // them keeps this arithmetic from sinking to its first use)
                const int id = __builtin_amdgcn_readfirstlane(gpend[j]);
                const long st = (long)id * p.bs;
                const int oct = __builtin_amdgcn_readfirstlane((int)((threadIdx.x + GT * j) / T::BN));
                const int k0 = s2 * KSTEP + oct * 8;
                const int kb = k0 <= kc - 8 ? k0 : kc - 8;
                const long ok = ((st < 0) | (st + p.bs > p.full_extent)) ? 0l : -1l;
                g0[j] = (int)(st & ok) + (kb & (p.bs - 1));
                // first row of the octet: gathered in the B_i half, compact (kb) in the F half;
                // kc is a multiple of 8 here, so an octet lies inside the contraction as a whole
                // or not at all, and kb keeps the latter in range (its activation digits are zero)
                const int r0 = g0[j] + ((kb - g0[j]) & -h2);
                wpitch = (size_t)ld2 * 8u;
                wcur[j] = wbase + (size_t)r0 * wpitch;
                csel[j] = cb[j] + ((cf[j] - cb[j]) & (0u - (unsigned)h2));
                gpend[j] = gather_id(p, ksn, KS, kc, j);
            }
        }
    }

    // one 16-byte unit per lane of the activation planes -> LDS stage (asynchronous)
    template <int J>
    __device__ __forceinline__ void dma_piece(const GemmParams& p, unsigned char* xstage) {
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)xstage;
        // Issued as plain text so that the compiler's own wait-count bookkeeping does not treat
        // every later LDS read as dependent on this transfer; the waits that order it are the
        // explicit ones in wait_and_barrier().  M0 carries the wave's LDS address.
        const unsigned lds = __builtin_amdgcn_readfirstlane(lds0 + (wave * 64 + GT * J) * 16);
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                     :
                     : "s"(lds), "v"(xs2 + J * xstride)
                     : "memory", "m0");
    }

    // NT: past the caches (words_past_caches() in ring_gemm.hip)
    static __device__ __forceinline__ u64 load_word(const u64* q) {
        if (NT) return __builtin_nontemporal_load(q);
        return *q;
    }

    // Word E of task J: split the word that is in the register into digits
    // (it was requested a step ago), then request the word of the step fixed by
    // begin() into the same register.  The choice between the two halves of the
    // stacked contraction and the row gather are selects on wave-uniform values.
    template <int J, int E, bool SPLIT>
    __device__ __forceinline__ void load_piece(const GemmParams& p, int kc) {
        // The compiler's wait for this word (requested a step ago) does not know about the LDS-DMA
        // transfers issued since, which sit between the two in the in-order load queue, so it also
        // waits for those.  Measured, that costs nothing: the kernel is bound by power, and a
        // hand-written, exact wait (which needs the request in inline assembly, outside the
        // compiler's view of the register) gave the same time per step.
        if (SPLIT) wa[J][E] = to_digits(wn[J][E]);
        // octet index is the same for all lanes of a wavefront
        const int oct = __builtin_amdgcn_readfirstlane((int)((threadIdx.x + GT * J) / T::BN));
        const int k0 = s2 * KSTEP + oct * 8;
        if constexpr (GMODE == WEIGHTS_TR) {
            const u64* src = h2 ? wf[J] : wb[J];
            // Words E - 1 and E of the octet are neighbours in memory: one 16-byte load behind the
            // split of the second (k is even and the rows are 16-byte aligned, host check).  Past
            // the end of the contraction any valid pair will do: its activation digits are zero.
            if constexpr ((E & 1) == 1) {
                typedef u64 u64x2 __attribute__((ext_vector_type(2)));
                const int kp = (k0 + E) < kc ? (k0 + E - 1) : kc - 2;
                const u64x2 v = *reinterpret_cast<const u64x2*>(src + kp);
                wn[J][E - 1] = v.x;
                wn[J][E] = v.y;
            }
            return;
        }
        if constexpr (GMODE == GATHER_POW2) {
            const char* rowp = wcur[J];
            wcur[J] += wpitch;
            wn[J][E] = load_word(reinterpret_cast<const u64*>(rowp + csel[J]));
            return;
        }
        const int kk = (k0 + E) < kc ? (k0 + E) : kc - 1;
        int row = kk;
        if (GMODE == GATHER_ANY) {
            const int blk = kk / p.bs;
            const long st = block_start(p, blk);
            row = h2 ? kk : (int)(st < 0 ? 0 : st) + (kk - blk * p.bs);
        }
        if constexpr (ROW_GATHER) {
            // wave-uniform start of the row, then this lane's column
            const char* rowp = wbase + (size_t)row * (size_t)ld2 * 8u;
            const unsigned c = cb[J] + ((cf[J] - cb[J]) & (0u - (unsigned)h2));
            wn[J][E] = *reinterpret_cast<const u64*>(rowp + c);
        } else {
            // every operand holds fewer than 2^31 words (host check), so the word offset fits 32 bits
            const u64* src = h2 ? wf[J] : wb[J];
            const unsigned off = (unsigned)row * (unsigned)ld2;
            wn[J][E] = load_word(src + off);
        }
    }

    // quarter Q of the byte transpose of task J: Q = 0: low digits of words 0..3,
    // 1: high digits of words 0..3, 2: low digits of words 4..7, 3: high digits of words 4..7
    template <int J, int Q>
    __device__ __forceinline__ void transpose_piece() {
        constexpr int e0 = (Q >> 1) * 4, d0 = (Q & 1) * 4, o = (Q >> 1) * 8 + d0;
        u32 x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = (Q & 1) ? (u32)(wa[J][e0 + i] >> 32) : (u32)wa[J][e0 + i];
        transpose4(x[0], x[1], x[2], x[3], pl[J][o], pl[J][o + 1], pl[J][o + 2], pl[J][o + 3]);
    }

    // digit plane Tt of task J -> LDS.  Weight stage layout: 16-byte fragments ordered
    // (digit, k-half, column); an octet is one 8-byte half of a fragment, so a matrix-instruction
    // operand is a single 16-byte LDS read.
    template <int J, int Tt>
    __device__ __forceinline__ void write_piece(unsigned char* wstage) {
        const int id = threadIdx.x + GT * J;
        const int c = id % T::BN, oct = id / T::BN;
        const u64 v = (u64)pl[J][Tt] | ((u64)pl[J][8 + Tt] << 32);
        *reinterpret_cast<u64*>(wstage + ((size_t)(Tt * 2 + (oct >> 1)) * T::BN + c) * 16 + (oct & 1) * 8) = v;
    }

    // SPLIT = false: first visit of a segment, nothing to split or store yet, loads only
    template <int P, bool SPLIT>
    __device__ __forceinline__ void piece(const GemmParams& p, int kc, unsigned char* xstage,
                                          unsigned char* wstage) {
        if constexpr (P < P_TASK) {
            dma_piece<P - P_DMA>(p, xstage);
        } else if constexpr (P < P_END) {
            constexpr int J = (P - P_TASK) / PER_TASK, R = (P - P_TASK) % PER_TASK;
            if constexpr (R < 8) load_piece<J, R, SPLIT>(p, kc);
            else if constexpr (R < 12) { if (SPLIT) transpose_piece<J, R - 8>(); }
            else { if (SPLIT) write_piece<J, R - 12>(wstage); }
        }
    }

    template <int P0, bool SPLIT, int... Ps>
    __device__ __forceinline__ void pieces(std::integer_sequence<int, Ps...>, const GemmParams& p,
                                           int kc, unsigned char* xstage, unsigned char* wstage) {
        (piece<P0 + Ps, SPLIT>(p, kc, xstage, wstage), ...);
    }

};


// Position of matrix instruction M inside a step: activation digit t, weight digit uu, wave
// sub-tiles (ii, j); the accumulator plane is t + uu <= 7.  The 36 digit pairs are walked with
// the digit of the side that has MORE fragments per digit in the outer loop, so that this side's
// fragments are live for one group of instructions only and the other side's are held for the
// step: activation digit outermost for WM >= WN, weight digit outermost for WN > WM (measured on
// the 32 x 256 tile with a row gather: 262 against 330 us on a 938 MB weight side).
template <int WM, int WN>
struct SlotMap {
    static constexpr bool W_OUTER = WN > WM;
    static constexpr int per_outer(int o) { return (8 - o) * WM * WN; }
    static constexpr int outer_of(int m) {
        int o = 0;
        while (m >= per_outer(o)) { m -= per_outer(o); ++o; }
        return o;
    }
    static constexpr int in_outer(int m) {
        int o = 0;
        while (m >= per_outer(o)) { m -= per_outer(o); ++o; }
        return m;
    }
    static constexpr int inner_of(int m) { return in_outer(m) / (WM * WN); }
    static constexpr int t_of(int m) { return W_OUTER ? inner_of(m) : outer_of(m); }
    static constexpr int u_of(int m) { return W_OUTER ? outer_of(m) : inner_of(m); }
    static constexpr int i_of(int m) { return (in_outer(m) / WN) % WM; }
    static constexpr int j_of(int m) { return in_outer(m) % WN; }
};

// Fragment reads of a step: read R < 8 WM is activation fragment a[R / WM][R % WM], the others
// are weight fragments bf[j][uu] with (uu, j) = ((R - 8 WM) / WN, (R - 8 WM) % WN).  slot(R) is
// the matrix instruction after which read R is issued, READ_LEAD instructions ahead of the
// first one that uses it; -1 for the reads issued before the first instruction.
template <int WM, int WN>
struct ReadMap {
    using SM = SlotMap<WM, WN>;
    static constexpr int NR = 8 * (WM + WN);
    static constexpr int NM = 36 * WM * WN;
    static constexpr int READ_LEAD = 8;
    static constexpr bool is_a(int r) { return r < 8 * WM; }
    static constexpr int need(int r) {
        for (int m = 0; m < NM; ++m) {
            if (is_a(r)) {
                if (SM::t_of(m) == r / WM && SM::i_of(m) == r % WM) return m;
            } else {
                if (SM::u_of(m) == (r - 8 * WM) / WN && SM::j_of(m) == (r - 8 * WM) % WN) return m;
            }
        }
        return NM;
    }
    static constexpr int slot(int r) { return need(r) - READ_LEAD < 0 ? -1 : need(r) - READ_LEAD; }
};

// One contraction step of a workgroup: 36 * WM * WN matrix instructions on the
// fragments of activation stage xs and weight stage ws, each followed by its
// share of the look-ahead pieces (see Loader).  The scheduling fences keep the
// compiler from regrouping them.  ks_next2 is clamped by the caller: past the
// end of a segment the look-ahead work is redundant but harmless.
template <class T, class L, int WM, int WN, int... Ms>
__device__ __forceinline__ void gemm_step_impl(std::integer_sequence<int, Ms...>, const GemmParams& p,
                                               L& ld, v16i (&acc)[WM][WN][8],
                                               const unsigned char* xs, const unsigned char* ws,
                                               unsigned char* ws_next, unsigned char* xs_next2,
                                               int a_off, int b_off, int ks_next2, int ks_limit, int KS, int kc) {
    using SM = SlotMap<WM, WN>;
    constexpr int NM = 36 * WM * WN;
    v4i bf[WN][8];
    v4i a[8][WM];
    ld.begin(p, ks_next2, KS, kc, ks_limit);
    // Fragment reads are issued in the order the matrix instructions consume them, each
    // READ_LEAD instructions ahead of its first use: the first instruction of a step then waits
    // for a handful of reads instead of the whole step's, and a fragment of a late digit plane
    // does not hold its registers through the early ones.
    using RM = ReadMap<WM, WN>;
    auto read_frag = [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        if constexpr (RM::is_a(R)) {
            constexpr int t = R / WM, ii = R % WM;
            a[t][ii] = lds_frag(xs + a_off + (t * 2 * T::BM + ii * 32) * 16);
        } else {
            constexpr int uu = (R - 8 * WM) / WN, j = (R - 8 * WM) % WN;
            bf[j][uu] = lds_frag(ws + b_off + (uu * 2 * T::BN + j * 32) * 16);
        }
    };
    auto reads_at = [&](auto slot) {
        constexpr int S = decltype(slot)::value;
        [&]<int... Rs>(std::integer_sequence<int, Rs...>) {
            ([&] { if constexpr (RM::slot(Rs) == S) read_frag(std::integral_constant<int, Rs>{}); }(), ...);
        }(std::make_integer_sequence<int, RM::NR>{});
    };
    reads_at(std::integral_constant<int, -1>{});
    __builtin_amdgcn_sched_barrier(0);
    (
        [&] {
            constexpr int M = Ms;
            constexpr int t = SM::t_of(M), uu = SM::u_of(M), ii = SM::i_of(M), j = SM::j_of(M);
            acc[ii][j][t + uu] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[t][ii], bf[j][uu],
                                                                        acc[ii][j][t + uu], 0, 0, 0);
            reads_at(std::integral_constant<int, M>{});
            constexpr int p0 = (int)((long)M * L::P_END / NM), p1 = (int)((long)(M + 1) * L::P_END / NM);
            ld.template pieces<p0, true>(std::make_integer_sequence<int, p1 - p0>{}, p, kc, xs_next2, ws_next);
            __builtin_amdgcn_sched_barrier(0);
        }(),
        ...);
    // The activation planes of the next step were requested one step ago; only the loads
    // issued during this step may still be in flight past this point.
    wait_and_barrier<L::VM_PER_STEP>();
}

template <class T, class L, int WM, int WN>
__device__ __forceinline__ void gemm_step(const GemmParams& p, L& ld,
                                          v16i (&acc)[WM][WN][8], const unsigned char* xs,
                                          const unsigned char* ws, unsigned char* ws_next,
                                          unsigned char* xs_next2, int a_off, int b_off,
                                          int ks_next2, int ks_limit, int KS, int kc) {
    gemm_step_impl<T, L, WM, WN>(std::make_integer_sequence<int, 36 * WM * WN>{}, p, ld, acc,
                                 xs, ws, ws_next, xs_next2, a_off, b_off, ks_next2, ks_limit, KS, kc);
}

// One workgroup's share of a product: segment by segment, the main loop and the write-out of the
// partial sum.
template <int WAVES_M, int WAVES_N, int WM, int WN, int KIND, int GMODE, bool LISTED, bool NT>
__device__ __forceinline__ void gemm_sweep(const GemmParams& p, const Geometry& q, UnitWalk<LISTED, 1>& walk,
                                           unsigned char* xs0, unsigned char* xs1, unsigned char* xs2,
                                           unsigned char* wsm) {
    using T = Tile<WAVES_M, WAVES_N, WM, WN>;
    using LD = Loader<T, KIND, GMODE, LISTED, NT>;
    const int n_eff = q.n_eff, kc = q.kc, m_eff = q.m_eff;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave % WAVES_M, wn = wave / WAVES_M;
    const int g = lane >> 5, r = lane & 31;
    // this lane's fragment offsets inside a stage (digit 0)
    const int a_off = (g * T::BM + wm * WM * 32 + r) * 16;
    const int b_off = (g * T::BN + wn * WN * 32 + r) * 16;

    LD ld;
    Segment sg;
    while (walk.next(sg)) {
        const int tm = sg.tm, tn = sg.tn, ks0 = sg.k0, L = sg.L, KSt = sg.KS;
        ld.setup(p, tm, tn, n_eff);
        ld.steps = sg.steps;
        v16i acc[WM][WN][8];
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int s = 0; s < 8; ++s)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][j][s][e] = 0;

        // prologue: step ks0 staged, step ks0+1 in flight
        const int ks_last = ks0 + L - 1;
        ld.prime(p, ks0, KSt, kc);
        ld.begin(p, ks0, KSt, kc, ks_last);
        ld.template pieces<LD::P_DMA, false>(std::make_integer_sequence<int, LD::P_END - LD::P_DMA>{}, p, kc, xs0, wsm);
        ld.begin(p, ks0 + 1 < ks_last ? ks0 + 1 : ks_last, KSt, kc, ks_last);
        ld.template pieces<LD::P_DMA, true>(std::make_integer_sequence<int, LD::P_END - LD::P_DMA>{}, p, kc, xs1, wsm);
        wait_and_barrier<0>();

        for (int i = 0; i < L; i += 3) {
            const int k2 = ks0 + i + 2;
            gemm_step<T, LD, WM, WN>(p, ld, acc, xs0, wsm + (i & 1) * T::WBYTES,
                                     wsm + ((i + 1) & 1) * T::WBYTES, xs2, a_off, b_off,
                                     k2 < ks_last ? k2 : ks_last, ks_last, KSt, kc);
            if (i + 1 < L)
                gemm_step<T, LD, WM, WN>(p, ld, acc, xs1, wsm + ((i + 1) & 1) * T::WBYTES,
                                         wsm + (i & 1) * T::WBYTES, xs0, a_off, b_off,
                                         k2 + 1 < ks_last ? k2 + 1 : ks_last, ks_last, KSt, kc);
            if (i + 2 < L)
                gemm_step<T, LD, WM, WN>(p, ld, acc, xs2, wsm + (i & 1) * T::WBYTES,
                                         wsm + ((i + 1) & 1) * T::WBYTES, xs1, a_off, b_off,
                                         k2 + 2 < ks_last ? k2 + 2 : ks_last, ks_last, KSt, kc);
        }
        // the look-ahead transfers of the last steps are redundant; let them land before the
        // stages are reused
        wait_and_barrier<0>();

        // slices of a tile meet in Z, which started out as C, through atomic adds
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                const int col = tn * T::BN + (wn * WN + j) * 32 + r;
                const int ccomp = (p.row_comp && col < n_eff) ? p.blk_comp[col / p.bs] : 0;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = tm * T::BM + (wm * WM + i) * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
                    const u64 z = recombine(acc[i][j][0][e], acc[i][j][1][e], acc[i][j][2][e], acc[i][j][3][e],
                                            acc[i][j][4][e], acc[i][j][5][e], acc[i][j][6][e], acc[i][j][7][e]);
                    bool live = row < m_eff && col < n_eff;
                    if (live && p.row_comp) live = p.row_comp[row] == ccomp;   // on a result block
                    if (live) atomicAdd(p.Z + (size_t)row * p.ldz + col, z);
                }
            }
    }
}

template <int WAVES_M, int WAVES_N, int WM, int WN, int KIND, int GMODE, bool LISTED, bool NT = false>
__global__ __launch_bounds__(GT, (Tile<WAVES_M, WAVES_N, WM, WN>::WG_PER_CU)) void ring_gemm_kernel(GemmParams p) {
    using T = Tile<WAVES_M, WAVES_N, WM, WN>;
    // three activation stages filled by LDS-DMA two steps ahead, as separate arrays so that the
    // compiler can tell a stage being filled from the one being read; two weight stages
    // written from registers one step ahead
    __shared__ __align__(16) unsigned char xs0[T::XBYTES];
    __shared__ __align__(16) unsigned char xs1[T::XBYTES];
    __shared__ __align__(16) unsigned char xs2[T::XBYTES];
    __shared__ __align__(16) unsigned char wsm[T::WSTAGES * T::WBYTES];
    const Geometry q = gemm_geometry<T::BM, T::BN, KIND, LISTED, 1>(p);
    if (q.units == 0) return;
    const int G = gridDim.x;
    const int b = xcd_contiguous(blockIdx.x, G);
    UnitWalk<LISTED, 1> walk(p, q, b, G, false);
    gemm_sweep<WAVES_M, WAVES_N, WM, WN, KIND, GMODE, LISTED, NT>(p, q, walk, xs0, xs1, xs2, wsm);
}

// The kernel variant for a call, instantiated explicitly, one translation unit with and one without step lists.
template <int WAVES_M, int WAVES_N, int WM, int WN, bool LISTED>
GemmKernel gemm_kernel_for(const GemmParams& p) {
    if (p.kind == KIND_SIMM) {
        if (!p.b_full) return p.w_nt ? ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_NONE, LISTED, true>
                                     : ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_NONE, LISTED, false>;
        if (p.bs_shift >= 3) return p.w_nt ? ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_POW2, LISTED, true>
                                     : ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_POW2, LISTED, false>;
        return ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_ANY, LISTED>;
    }
    if constexpr (LISTED) {
        return nullptr;      // step lists belong to Protocol 3
    } else {
        if (p.w_tr) return ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SOMM, WEIGHTS_TR, false>;
        return p.w_nt ? ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SOMM, GATHER_NONE, false, true>
                                     : ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SOMM, GATHER_NONE, false, false>;
    }
}

extern template GemmKernel gemm_kernel_for<2, 2, 1, 1, false>(const GemmParams&);
extern template GemmKernel gemm_kernel_for<2, 2, 1, 1, true>(const GemmParams&);
extern template GemmKernel gemm_kernel_for<1, 4, 1, 2, false>(const GemmParams&);
extern template GemmKernel gemm_kernel_for<1, 4, 1, 2, true>(const GemmParams&);

template <int WAVES_M, int WAVES_N, int WM, int WN>
int launch_gemm(comet_ctx* ctx, const char* what, const GemmParams& p) {
    using T = Tile<WAVES_M, WAVES_N, WM, WN>;
    GemmKernel kern = nullptr;
    if (!p.own_try)
        kern = p.step_list ? gemm_kernel_for<WAVES_M, WAVES_N, WM, WN, true>(p) : gemm_kernel_for<WAVES_M, WAVES_N, WM, WN, false>(p);
    if (!kern || p.w_planes) return comet_fail(ctx, COMET_EINVAL, "%s: no kernel variant for this call", what);
    if (p.tile_bm != T::BM || p.tile_bn != T::BN || p.grid < 1)
        return comet_fail(ctx, COMET_EINVAL, "%s: launch plan does not match the kernel", what);
    return launch_share_kernel(ctx, what, kern, dim3((unsigned)p.grid), p);
}

}  // namespace comet_gemm
