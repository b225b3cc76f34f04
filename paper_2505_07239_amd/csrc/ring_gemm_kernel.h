// The int8 matrix-core kernel behind the share calls on weight WORDS (see ring_gemm.hip for the
// formulation): tile shapes, the loader that stages both operands, one contraction step, the
// stream-K kernel and its launcher; and what it shares with the kernel on weight planes
// (ring_gemm_planes.h): the packed activation format, the walk over the work units, the launch plan.
// The kernel variants are instantiated in translation units of their own (ring_gemm_tile_*.hip),
// so that they compile side by side.
#pragma once

#include "common.h"
#include "digits.h"
#include "gemm_params.h"

#include <type_traits>
#include <utility>

namespace comet_gemm {


typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef u32 u32x4 __attribute__((ext_vector_type(4)));

constexpr int KSTEP = 32;       // ring words contracted per matrix instruction
constexpr int MAX_SEG = 256;    // contraction steps an int32 plane can absorb
constexpr int GT = 256;         // threads per workgroup (4 wavefronts)

// how the weight-side rows of B_i are addressed (SIMM with a full-size B_i only)
constexpr int GATHER_NONE = 0;   // rows are the compact contraction index
constexpr int GATHER_POW2 = 1;   // block gather, bs a power of two >= 8
constexpr int GATHER_ANY = 2;    // block gather, any bs
// SOMM with neuron-major weights: B_i and F hold one row of k contiguous words per output column
constexpr int WEIGHTS_TR = 3;
// B_i and F arrive as digit planes (ring_gemm_planes.h); with W_PLANES_GATHER the rows of a
// full-size B_i are gathered by block (SIMM, bs a multiple of 16)
constexpr int W_PLANES = 4;
constexpr int W_PLANES_GATHER = 5;

// Packed layout of [E | A'] in 16-byte units: group (half h, step s, digit t,
// k-half g) is a run of mpad units, one per row; the 16 bytes of a unit are
// digit t of words k = 32 s + 16 g + 0..15 of that row, which is exactly what
// one lane feeds to v_mfma_i32_32x32x32_i8.  Groups are ordered (h, s, t, g).
__device__ __host__ __forceinline__ size_t xp_group(int h, int s, int t, int g, int ks_cap) {
    return ((((size_t)h * ks_cap + s) * 8 + t) * 2 + g);
}


// ---------------------------------------------------------------------------
// gemm
// ---------------------------------------------------------------------------
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

// Workgroup barrier of the main loop.  Waits until at most N of this
// wavefront's vector-memory loads are still in flight (loads return in order,
// so everything older than the N youngest has landed, including LDS-DMA
// writes) and until all of its LDS accesses are done, then meets the other
// wavefronts.  Written out by hand because the generic barrier would also
// wait for the LDS-DMA loads that were only just issued for a later step.
template <int N>
__device__ __forceinline__ void wait_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

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


__device__ __forceinline__ v4i lds_frag(const unsigned char* p) {
    return *reinterpret_cast<const v4i*>(p);
}

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

// What a launch computes, from the device-resident counts.  PER: contraction steps (of 32 words) in
// a work unit: one with weight words, two with weight planes (ring_gemm_planes.h).
struct Geometry {
    int n_eff, kc, KS, KT, m_eff, tiles_m, tiles_n, tiles;
    long units;     // (tile, contraction unit) pairs; a tile has KT = 2 KS / PER of them
};

template <int BM, int BN, int KIND, bool LISTED, int PER>
__device__ __forceinline__ Geometry gemm_geometry(const GemmParams& p) {
    Geometry q;
    const int nblk = n_blocks(p);
    q.n_eff = KIND == KIND_SOMM ? nblk * p.bs : p.n_cap;
    q.kc = KIND == KIND_SOMM ? p.kc_cap : nblk * p.bs;
    q.KS = (q.kc + KSTEP - 1) / KSTEP;
    q.KT = 2 * q.KS / PER;
    q.m_eff = n_rows(p);
    q.tiles_m = (q.m_eff + BM - 1) / BM;
    q.tiles_n = (q.n_eff + BN - 1) / BN;
    // with result blocks only the listed tiles are computed
    q.tiles = p.row_comp ? p.tile_list[0] : q.tiles_m * q.tiles_n;
    // with per-token row sets only the listed steps of each row tile are computed
    q.units = LISTED ? (long)q.tiles_n * (2 / PER) * p.step_off[q.tiles_m] : (long)q.tiles * q.KT;
    return q;
}

// A run of contraction units of one output tile, what a workgroup computes between two write-outs.
struct Segment {
    int tm, tn;             // output tile
    int k0, L;              // units [k0, k0 + L)
    int KS;                 // contraction steps of one half of the tile's stacked contraction
    const int* steps;       // listed contraction steps of this row tile, or null (all steps)
};

// What a workgroup computes of one product, segment by segment, in one of two ways.
//
// One slice of one tile (the default when there are at least as many workgroups as tiles): the
// contraction of every tile is cut into S = G / tiles slices, a workgroup takes one of them, so it pays
// for filling its pipeline and for writing out its partial sum once.  (An even split of all units
// makes most workgroups straddle two slices: a call with 64 x 4096 x 1664 on weight planes, 6.5
// units each, took 73 us against 56, and one with 20 rows on weight words 56 against 43.)
//
// An even share [u, u_end) of the units: when the slices would leave the longest workgroup more than
// SPLIT_COST units above an even share, with more tiles than workgroups, and where the caller
// fixes the slice length (p.chunk).  Units are ordered chunk-major: all tiles for contraction
// units [0, CH), then all tiles for [CH, 2 CH), ...
//
// Either way, workgroups that run side by side sweep the same slice of the contraction at the same
// time (the activation planes of that slice stay hot in L2) and each XCD ends up with whole
// slices, so a weight word is fetched from HBM by one XCD only.
template <bool LISTED, int PER>
struct UnitWalk {
    static constexpr int SPLIT_COST = 6 / PER;      // units: what a second segment costs a workgroup
    const GemmParams& p;
    const Geometry& q;
    long u_begin, u_end, u;
    const int team_tm, tiles;
    int CH, n_chunks;
    int slice_tile;                                 // tile of this workgroup's slice, or -1: an even share

    // workgroup b of G; own: every workgroup gets whole tiles
    __device__ __forceinline__ UnitWalk(const GemmParams& p_, const Geometry& q_, int b, int G, bool own)
        : p(p_), q(q_), team_tm(-1), tiles(q_.tiles) {
        slice_tile = -1;
        if (!LISTED && !own && p.chunk == 0 && tiles <= G) {
            const int S = G / tiles < q.KT ? G / tiles : q.KT;
            if ((q.KT + S - 1) / S <= q.units / G + SPLIT_COST) {
                slice_tile = b % tiles;
                const int c = b / tiles;
                u_begin = u = c < S ? (long)q.KT * c / S : 0;
                u_end = c < S ? (long)q.KT * (c + 1) / S : 0;
                return;
            }
        }
        u_begin = u = q.units * b / G;
        u_end = q.units * (b + 1) / G;
        CH = p.chunk;
        if (own) CH = q.KT;                    // units tile by tile, all of a tile's contraction in a row
        else if (CH == 0) {
            int slices = (G + tiles / 2) / tiles;      // as many slices as workgroups per tile
            if (slices < 1) slices = 1;
            CH = (q.KT + slices - 1) / slices;
            if (CH > MAX_SEG / PER) CH = MAX_SEG / PER;
            if (CH < 1) CH = 1;
        }
        n_chunks = (q.KT + CH - 1) / CH;
    }

    // The units [u0, u1), tile by tile.  team >= 0: the workgroup computes row tile team only and the
    // units are (column tile, contraction unit) pairs; the workgroups of a team walk the same
    // units side by side.
    __device__ __forceinline__ UnitWalk(const GemmParams& p_, const Geometry& q_, long u0, long u1, int team)
        : p(p_), q(q_), u_begin(u0), u_end(u1), u(u0), team_tm(team), tiles(team >= 0 ? q_.tiles_n : q_.tiles),
          CH(q_.KT), n_chunks(1), slice_tile(-1) {}

    __device__ __forceinline__ bool next(Segment& g) {
        if (u >= u_end) return false;
        long len;
        g.KS = q.KS;
        g.steps = nullptr;
        if constexpr (LISTED) {
            // units are ordered row tile by row tile, inside a row tile column tile by column
            // tile, inside a tile along its listed steps (E B_i half, then A' F half)
            constexpr int F = 2 / PER;         // units per listed step
            int lo = 0, hi = q.tiles_m;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if ((long)q.tiles_n * F * p.step_off[mid] <= u) lo = mid; else hi = mid;
            }
            g.tm = lo;
            g.KS = p.step_cnt[lo];
            const long rem = u - (long)q.tiles_n * F * p.step_off[lo];
            g.tn = (int)(rem / (F * g.KS));
            g.k0 = (int)(rem - (long)g.tn * F * g.KS);
            len = F * g.KS - g.k0;
            g.steps = p.step_list + (size_t)lo * p.ks_cap;
        } else {
            int tile_pos;
            if (slice_tile >= 0) {
                tile_pos = slice_tile;
                g.k0 = (int)u;
                len = u_end - u;
            } else {
                const long full = (long)tiles * CH;
                int c = (int)(u / full);
                if (c > n_chunks - 1) c = n_chunks - 1;
                const long rem = u - (long)c * full;
                const int clen = (c == n_chunks - 1) ? q.KT - c * CH : CH;
                tile_pos = (int)(rem / clen);
                g.k0 = c * CH + (int)(rem - (long)tile_pos * clen);
                len = c * CH + clen - g.k0;
            }
            const int tile = p.row_comp ? p.tile_list[1 + tile_pos] : tile_pos;
            g.tm = tile % q.tiles_m;
            g.tn = tile / q.tiles_m;
            if (team_tm >= 0) { g.tm = team_tm; g.tn = tile; }
        }
        if (len > MAX_SEG / PER) len = MAX_SEG / PER;      // (an owned tile's contraction may be longer than a segment)
        if (len > u_end - u) len = u_end - u;
        g.L = (int)len;
        if (!LISTED && p.k_rotate) {
            // Units tile by tile, a tile cut into parts by the workgroup ranges: the parts take their
            // contraction units in reverse order of their positions (the part [c, d) of a tile gets
            // the units [KT - d, KT - c); any order gives the same sum).  A workgroup that starts
            // in the middle of a tile thus begins at unit 0 like one that starts on a tile, and
            // all workgroups sweep the contraction in two phases only, KT - share apart: the
            // activation planes of a phase are shared through L2 instead of being fetched per tile.
            const long tile_u0 = u - g.k0;
            const long c_lo = u_begin - tile_u0, c_hi = u_end - tile_u0;
            g.k0 += q.KT - (c_lo > 0 ? (int)c_lo : 0) - (c_hi < q.KT ? (int)c_hi : q.KT);
        }
        u += len;
        return true;
    }
};

// sum_s sext64(S_s) << 8s: the four low planes as 32 x 32 -> 64 bit signed multiply-adds, the four
// high planes only reach the upper word
__device__ __forceinline__ u64 recombine(int s0, int s1, int s2, int s3, int s4, int s5, int s6, int s7) {
    long long lo = (long long)s0;
    lo += (long long)s1 * (1 << 8);
    lo += (long long)s2 * (1 << 16);
    lo += (long long)s3 * (1 << 24);
    const u32 hi = (u32)s4 + ((u32)s5 << 8) + ((u32)s6 << 16) + ((u32)s7 << 24);
    return (u64)lo + ((u64)hi << 32);
}

// One workgroup's share of a product: segment by segment, the main loop and the write-out of the
// partial sum.
template <int WAVES_M, int WAVES_N, int WM, int WN, int KIND, int GMODE, bool LISTED, bool NT>
__device__ __forceinline__ void gemm_sweep(const GemmParams& p, const Geometry& q, UnitWalk<LISTED, 1>& walk,
                                           const bool own, unsigned char* xs0, unsigned char* xs1,
                                           unsigned char* xs2, unsigned char* wsm) {
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

        // The only writer of a tile (own) stores Z = C + sum (Z += sum for a later segment of a long
        // contraction: this lane's own earlier store, complete since the barrier above); the loads of
        // a sub-tile go out together, ahead of the arithmetic.  Slices of a shared tile meet in Z,
        // which started out as C, through atomic adds.
        const u64* src = ks0 == 0 ? p.C : p.Z;
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                const int col = tn * T::BN + (wn * WN + j) * 32 + r;
                const int ccomp = (p.row_comp && col < n_eff) ? p.blk_comp[col / p.bs] : 0;
                u64 prev[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = tm * T::BM + (wm * WM + i) * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
                    prev[e] = 0;
                    if (own && row < m_eff && col < n_eff) prev[e] = src[(size_t)row * p.ldz + col];
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = tm * T::BM + (wm * WM + i) * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
                    const u64 z = recombine(acc[i][j][0][e], acc[i][j][1][e], acc[i][j][2][e], acc[i][j][3][e],
                                            acc[i][j][4][e], acc[i][j][5][e], acc[i][j][6][e], acc[i][j][7][e]);
                    bool live = row < m_eff && col < n_eff;
                    if (live && p.row_comp) live = p.row_comp[row] == ccomp;   // on a result block
                    if (live) {
                        if (own) p.Z[(size_t)row * p.ldz + col] = prev[e] + z;
                        else atomicAdd(p.Z + (size_t)row * p.ldz + col, z);
                    }
                }
            }
    }
}

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD one contiguous range of work.
__device__ __forceinline__ int xcd_contiguous(int b, int G) {
    return (G & 7) == 0 ? (b & 7) * (G >> 3) + (b >> 3) : b;
}

// OWN: the variant for launches planned so that every workgroup gets whole output tiles (see
// owns_tiles()); it still checks that on the device, where the counts are, and falls back to the
// shared-tile path.  The other variant never owns: it carries none of that code.
template <int WAVES_M, int WAVES_N, int WM, int WN, int KIND, int GMODE, bool LISTED, bool OWN = false, bool NT = false>
__global__ __launch_bounds__(GT, (Tile<WAVES_M, WAVES_N, WM, WN>::WG_PER_CU)) void ring_gemm_kernel(GemmParams p) {
    using T = Tile<WAVES_M, WAVES_N, WM, WN>;
    // three activation stages filled by LDS-DMA two steps ahead, as separate arrays so that the
    // compiler can tell a stage being filled from the one being read; two weight stages
    // written from registers one step ahead
    __shared__ __align__(16) unsigned char xs0[T::XBYTES];
    __shared__ __align__(16) unsigned char xs1[T::XBYTES];
    __shared__ __align__(16) unsigned char xs2[T::XBYTES];
    __shared__ __align__(16) unsigned char wsm[T::WSTAGES * T::WBYTES];
    if (p.tile_sel && *p.tile_sel != p.tile_sel_want) return;   // the other tile shape was chosen
    const Geometry q = gemm_geometry<T::BM, T::BN, KIND, LISTED, 1>(p);
    if (q.units == 0) return;
    const int G = gridDim.x;
    const int b = xcd_contiguous(blockIdx.x, G);
    bool own = false;
    if constexpr (OWN) own = owns_tiles(p, q.m_eff, q.n_eff, q.kc);
    UnitWalk<LISTED, 1> walk(p, q, b, G, own);
    gemm_sweep<WAVES_M, WAVES_N, WM, WN, KIND, GMODE, LISTED, NT>(p, q, walk, own, xs0, xs1, xs2, wsm);
}

// The kernel variant for a call: the kind of product, how the weight side is addressed, and
// (LISTED) whether a step list is walked.  Instantiated explicitly, one translation unit per
// (tile shape, LISTED), so that the variants compile side by side.
using GemmKernel = void (*)(GemmParams);

// the OWN variants (128 x 64 tile, no step lists): a translation unit of their own
template <int WAVES_M, int WAVES_N, int WM, int WN>
GemmKernel gemm_own_kernel_for(const GemmParams& p) {
    if (p.kind == KIND_SIMM) {
        if (!p.b_full) return p.w_nt ? ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_NONE, false, true, true>
                                     : ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_NONE, false, true, false>;
        if (p.bs_shift >= 3) return p.w_nt ? ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_POW2, false, true, true>
                                     : ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_POW2, false, true, false>;
        return ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_ANY, false, true>;
    }
    if (p.w_tr) return ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SOMM, WEIGHTS_TR, false, true>;
    return p.w_nt ? ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SOMM, GATHER_NONE, false, true, true>
                                     : ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SOMM, GATHER_NONE, false, true, false>;
}
extern template GemmKernel gemm_own_kernel_for<2, 2, 2, 1>(const GemmParams&);

template <int WAVES_M, int WAVES_N, int WM, int WN, bool LISTED>
GemmKernel gemm_kernel_for(const GemmParams& p) {
    if (p.kind == KIND_SIMM) {
        if (!p.b_full) return p.w_nt ? ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_NONE, LISTED, false, true>
                                     : ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_NONE, LISTED, false, false>;
        if (p.bs_shift >= 3) return p.w_nt ? ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_POW2, LISTED, false, true>
                                     : ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_POW2, LISTED, false, false>;
        return ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SIMM, GATHER_ANY, LISTED>;
    }
    if constexpr (LISTED) {
        return nullptr;      // step lists belong to Protocol 3
    } else {
        if (p.w_tr) return ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SOMM, WEIGHTS_TR, false>;
        return p.w_nt ? ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SOMM, GATHER_NONE, false, false, true>
                                     : ring_gemm_kernel<WAVES_M, WAVES_N, WM, WN, KIND_SOMM, GATHER_NONE, false, false, false>;
    }
}

extern template GemmKernel gemm_kernel_for<2, 2, 2, 1, false>(const GemmParams&);
extern template GemmKernel gemm_kernel_for<2, 2, 1, 1, false>(const GemmParams&);
extern template GemmKernel gemm_kernel_for<2, 2, 1, 1, true>(const GemmParams&);
extern template GemmKernel gemm_kernel_for<1, 4, 1, 2, false>(const GemmParams&);
extern template GemmKernel gemm_kernel_for<1, 4, 1, 2, true>(const GemmParams&);

// Launch plan of the matrix-core kernels for an output tile BM x BN: the grid and whether the launch may turn out to own its tiles.  per: contraction steps per work unit (see
// Geometry).  Fixed before the packing kernel is launched, which has to know whether the share
// kernel will initialise Z itself.
inline void plan_gemm(const comet_ctx* ctx, GemmParams& p, int BM, int BN, int wg_per_cu, int per) {
    const long tiles = (long)((p.m + BM - 1) / BM) * ((p.n_cap + BN - 1) / BN);
    const long kt = 2l * p.ks_cap / per;
    const long units_cap = tiles * kt;
    // a chip-sized grid, shrunk when there is too little work to share out
    long grid = (ctx->num_cu / 8) * 8 * wg_per_cu;
    if (grid < 8) grid = 8;
    const long want = (units_cap * per + 1) / 2;      // at least two contraction steps per workgroup
    if (want < grid) grid = want < 8 ? (want < 1 ? 1 : want) : (want / 8) * 8;
    if (ctx->gemm_grid > 0) grid = ctx->gemm_grid;
    // how the contraction is cut is decided on the device (UnitWalk), unless the caller fixes it
    p.chunk = ctx->gemm_chunk > 0 ? (ctx->gemm_chunk + per - 1) / per : 0;
    if (p.chunk > MAX_SEG / per) p.chunk = MAX_SEG / per;
    p.grid = (int)grid;
    p.tile_bm = BM;
    p.tile_bn = BN;
    // Owned tiles: plain product, default slicing, the 128 x 64 tile, and a tile count (at full
    // capacity; the kernel checks the device-resident counts) that the grid divides
    p.own_try = (!p.row_comp && !p.tmask && ctx->gemm_chunk == 0 && BM == 128 && tiles % grid == 0) ? 1 : 0;
}

// Launches a share kernel; when this launch is a timed one the event pair rides on the dispatch
// itself (its start and end timestamps): no marker packets before or after the kernel, so
// timing leaves the stream's schedule as it is.
template <class K, class P>
int launch_share_kernel(comet_ctx* ctx, const char* what, K kern, int grid, const P& p) {
    if (comet_time_this_launch(ctx)) {
        hipExtLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(GT), 0, ctx->stream, ctx->ev[ctx->ev_used],
                              ctx->ev[ctx->ev_used + 1], 0, p);
        ctx->ev_used += 2;
    } else {
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(GT), 0, ctx->stream, p);
    }
    COMET_LAUNCH_CHECK(ctx, what);
    return COMET_OK;
}

template <int WAVES_M, int WAVES_N, int WM, int WN>
int launch_gemm(comet_ctx* ctx, const char* what, const GemmParams& p) {
    using T = Tile<WAVES_M, WAVES_N, WM, WN>;
    GemmKernel kern = nullptr;
    if constexpr (WM * WN == 2 && WAVES_N == 2) {
        // the 128 x 64 tile: no variants for per-token row sets (the dispatch picks 64 rows for them)
        if (p.own_try) kern = gemm_own_kernel_for<WAVES_M, WAVES_N, WM, WN>(p);
        else if (!p.step_list) kern = gemm_kernel_for<WAVES_M, WAVES_N, WM, WN, false>(p);
    } else {
        if (!p.own_try)
            kern = p.step_list ? gemm_kernel_for<WAVES_M, WAVES_N, WM, WN, true>(p)
                               : gemm_kernel_for<WAVES_M, WAVES_N, WM, WN, false>(p);
    }
    if (!kern || p.w_planes) return comet_fail(ctx, COMET_EINVAL, "%s: no kernel variant for this call", what);
    if (p.tile_bm != T::BM || p.tile_bn != T::BN || p.grid < 1)
        return comet_fail(ctx, COMET_EINVAL, "%s: launch plan does not match the kernel", what);
    return launch_share_kernel(ctx, what, kern, p.grid, p);
}

}  // namespace comet_gemm
