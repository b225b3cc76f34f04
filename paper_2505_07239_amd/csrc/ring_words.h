// The int8 matrix-core kernel of the share calls whose weight-side operands are WORDS (see
// ring_gemm.hip for the formulation).
//
// A workgroup is eight wavefronts, two per SIMD: four of them multiply, four feed them.  A work unit
// is a pair of contraction steps (64 words), what v_mfma_i32_16x16x64_i8 contracts.
//   * A feeding wavefront owns sixteen of the 64 contraction words: its lanes hold one output column
//     each, load the column's sixteen words three pairs ahead of
//     their use, split them into signed digits, byte-transpose them in registers (v_perm_b32) and store
//     eight 16-byte units, one per digit, to LDS in matrix-instruction operand order.  All
//     addressing -- the block gather of Protocols 2 and 3, step lists, neuron-major weights, the ends
//     of the operands -- is its business.
//   * A multiplying wavefront owns 16 rows x 64 columns in eight digit planes (128 accumulator
//     registers).  Activation units come straight from memory (L2, for the most part) into
//     registers, a pair ahead: every row belongs to one wavefront of the workgroup, so nothing is read
//     twice.  Weight units are read from LDS digit by digit: the weight digits are walked downwards,
//     so that the first ones feed few products and the last one 32, behind which the next pair's
//     first units arrive.
//   * One barrier per pair.  Two LDS stages: pair n is read from stage n % 2 while pair n + 1 is
//     written to the other; the barrier lies ahead of the last digit's products, when all units of
//     the pair are in registers.
//
// Why two kinds of wavefront: the vector work of the digit split and the waits for memory stay out of
// the instruction stream of the matrix instructions, and the two share the SIMD's issue slots without
// waiting for each other.  Kernels that do both in every wavefront (32x32x32, operands of both sides staged in LDS,
// 64 x 64 and 128 x 64 tiles) take, for 64 rows, k = 4096, n = 11008 (722 MB of words), 220 us, of which 180
// remained when every load hit the cache and 160 when eight of nine matrix instructions were left out.
// What bounds this one, by the counters: with 512 rows the clock falls to 1.74 GHz (1.90 in the row product) at 66 % busy
// matrix units, so power for the most part; with 64 rows the clock holds, the matrix units are busy half of the time, the
// words come at 3.9 TB/s and a third of the wavefronts' cycles is waiting (193 us from a cool chip, 245 in a long run; the
// planes kernel 172 and 220).  Without the digit split it is no faster.
// Against those kernels, whole calls: 192 x 1664 x 4096 106 -> 91 us, 512 x 4096 x 1664 238 -> 212, 512 x 4096 x 11008
// 1486 -> 1361, 64 x 11008 x 4096 235 -> 216; rows gathered in blocks that are no multiple of 16 (256 x 819 x 1001) 50 -> 39.
// The multiplying wavefronts take every register they can have; what does not fit (20 bytes of scratch per lane with step
// lists, 40 to 44 without) is stored and read back around a segment, in its set-up and its write-out: no scratch access lies
// in the loops over the pairs, of either kind of wavefront, in any variant.
// A pair is the least a workgroup can do; where a workgroup has one or two the 64 x 64 tile of ring_tile.h is ahead
// (takes_staged_tile() in ring_gemm.hip).
#pragma once

#include "ring_gemm_kernel.h"

namespace comet_gemm {

constexpr int WORD_THREADS = 2 * GT;      // four multiplying and four feeding wavefronts

constexpr int WORD_BM = 64, WORD_BN = 64;                 // output tile: four wavefronts of 16 x 64 on top of each other
constexpr int WORD_STAGE = WORD_BN * KPAIR * 8;           // bytes of a weight stage
constexpr int WORD_SETS = 3;                              // pairs whose words are on their way: 96 KB per compute unit
constexpr int WORD_LEN = MAX_SEG / 2;                     // longest segment, in pairs

// how a feeding wavefront finds its sixteen contraction rows
constexpr int ROWS_PLAIN = 0;     // consecutive rows of both operands
constexpr int ROWS_GATHER16 = 1;  // SIMM, full-size B_i, bs a multiple of 16: one block per sixteen rows
constexpr int ROWS_GATHER = 2;    // SIMM, full-size B_i, any bs
constexpr int ROWS_TR = 3;        // SOMM, neuron-major weights: a column's contraction words are consecutive

// LDS accesses done, then meet the other wavefronts (loads from memory stay in flight).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ---------------------------------------------------------------------------
// the feeding wavefronts
// ---------------------------------------------------------------------------
template <int KIND, int ROWS, bool LISTED, bool NT>
struct WordSource {
    // Per pair of the segment the first row of this wavefront's group (step lists, gather by sixteen) or all
    // sixteen rows (gather), worked out once per segment.
    static constexpr int TAB = ROWS == ROWS_GATHER ? 16 : (LISTED || ROWS == ROWS_GATHER16) ? 1 : 0;
    typedef u64 u64x2 __attribute__((ext_vector_type(2)));

    const GemmParams& p;
    const int kc, wave, lane;
    int* const tab;
    unsigned cb, cf;               // the lane's column in a row of B_i and of F, in bytes
    const u64* wb;                 // ROWS_TR: the lane's row of k words
    const u64* wf;
    int k0, L, KS;                 // the segment

    __device__ __forceinline__ WordSource(const GemmParams& p_, int kc_, int wave_, int* tab_)
        : p(p_), kc(kc_), wave(wave_), lane((int)(threadIdx.x & 63)), tab(tab_) {}

    __device__ __forceinline__ void setup(const Segment& sg, int n_eff) {
        k0 = sg.k0; L = sg.L; KS = sg.KS;
        int col = sg.tn * WORD_BN + lane;
        col = col < n_eff ? col : n_eff - 1;               // (its products are never written back)
        long bcol = col;
        if (KIND == KIND_SOMM && p.b_full) {
            const int blk = col / p.bs;
            const long st = block_start(p, blk);
            bcol = (st < 0 ? 0 : st) + (col - blk * p.bs);
        }
        if constexpr (ROWS == ROWS_TR) {
            wb = p.B + bcol * p.ldb;
            wf = p.F + (long)col * p.ldf;
        } else {
            cb = (unsigned)bcol * 8u;                      // columns stay below 2^24 (host check)
            cf = (unsigned)col * 8u;
        }
        if constexpr (TAB > 0) {
            for (int i = lane; i < L * TAB; i += 64) {
                const int ks = 2 * (k0 + i / TAB) + (wave >> 1);
                const int h = ks >= KS ? 1 : 0;
                int s = ks - h * KS;
                if constexpr (LISTED) s = sg.steps[s];
                int k = s * KSTEP + 16 * (wave & 1);
                if constexpr (ROWS == ROWS_GATHER) k += i % TAB;
                // Rows past the end of the contraction keep a valid address: their activation digits are zero.
                if constexpr (ROWS == ROWS_GATHER16) k = k <= kc - 16 ? k : kc - 16;
                if constexpr (ROWS == ROWS_GATHER) k = k < kc ? k : kc - 1;
                if ((ROWS == ROWS_GATHER16 || ROWS == ROWS_GATHER) && h == 0) {
                    const int blk = k / p.bs;
                    const long st = block_start(p, blk);
                    k = (int)(st < 0 ? 0 : st) + (k - blk * p.bs);
                }
                tab[i] = k;
            }
        }
    }

    static __device__ __forceinline__ u64 load_word(const char* row, unsigned col) {
        const u64* q = reinterpret_cast<const u64*>(row + col);
        if (NT) return __builtin_nontemporal_load(q);      // past the caches (words_past_caches() in ring_gemm.hip)
        return *q;
    }

    // Request the words of pair q (beyond the segment: one row of its last pair, over and over).
    __device__ __forceinline__ void request(int q, u64 (&w)[16]) const {
        const bool in = q < L;
        const int qq = in ? q : L - 1;
        const int ks = 2 * (k0 + qq) + (wave >> 1);
        const int h = ks >= KS ? 1 : 0;
        const char* op = reinterpret_cast<const char*>(h ? p.F : p.B);
        const u32 pitch = (u32)(h ? p.ldf : p.ldb) * 8u;  // (rows stay below 2^24 words: host check)
        if constexpr (ROWS == ROWS_GATHER) {
            const u64 off = (u64)(u32)tab[qq * 16 + (in ? lane & 15 : 0)] * pitch;
            const u32 lo = (u32)off, hi = (u32)(off >> 32);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const size_t o = (size_t)(u32)__builtin_amdgcn_readlane((int)lo, i) |
                                 ((size_t)(u32)__builtin_amdgcn_readlane((int)hi, i) << 32);
                w[i] = load_word(op + o, h ? cf : cb);
            }
            return;
        }
        int r0 = (ks - h * KS) * KSTEP + 16 * (wave & 1);
        if constexpr (TAB == 1) r0 = __builtin_amdgcn_readfirstlane(tab[qq]);
        if constexpr (ROWS == ROWS_TR) {
            // pairs of contraction words: k is even and the rows are 16-byte aligned (host check)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = r0 + (in ? 2 * j : 0);
                const int kp = k <= kc - 2 ? k : kc - 2;
                const u64x2 v = *reinterpret_cast<const u64x2*>((h ? wf : wb) + kp);
                w[2 * j] = v.x;
                w[2 * j + 1] = v.y;
            }
            return;
        }
        // consecutive rows, the last row of the operand over and over beyond its end
        int more = in ? 15 : 0;
        if constexpr (ROWS == ROWS_PLAIN) {
            r0 = r0 < kc ? r0 : kc - 1;
            more = more < kc - 1 - r0 ? more : kc - 1 - r0;
        }
        const char* row = op + (size_t)r0 * pitch;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            w[i] = load_word(row, h ? cf : cb);
            row += i < more ? pitch : 0u;
        }
    }

    // The words of a pair -> digit units in an LDS stage, ordered (digit, group of sixteen words, column).
    __device__ __forceinline__ void convert(const u64 (&w)[16], unsigned char* stage) const {
        u64 plane[2][8];
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            u64 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = to_digits(w[8 * o + i]);
            digits_to_planes(v, plane[o]);
        }
        u64x2* dst = reinterpret_cast<u64x2*>(stage) + wave * WORD_BN + lane;
#pragma unroll
        for (int t = 0; t < 8; ++t) dst[t * 4 * WORD_BN] = u64x2{plane[0][t], plane[1][t]};
    }
};

template <int KIND, int ROWS, bool LISTED, bool NT>
__device__ __forceinline__ void word_feed(const GemmParams& p, const Geometry& q, UnitWalk<LISTED>& walk, int wave,
                                          unsigned char* wsm, int* tab) {
    constexpr int D = WORD_SETS;
    WordSource<KIND, ROWS, LISTED, NT> src(p, q.kc, wave, tab);
    u64 w[D][16];
    Segment sg;
    while (walk.next(sg)) {
        src.setup(sg, q.n_eff);
        if (sg.L <= 2) {
            // (a product so small that its launch, not its work, takes the time: no look-ahead to fill)
            src.request(0, w[0]);
            if (sg.L == 2) src.request(1, w[1]);
            src.convert(w[0], wsm);
            lds_barrier();
            if (sg.L == 2) src.convert(w[1], wsm + WORD_STAGE);
            lds_barrier();
            if (sg.L == 2) lds_barrier();
            continue;
        }
#pragma unroll
        for (int d = 0; d < D; ++d) src.request(d, w[d]);
        src.convert(w[0], wsm);
        src.request(D, w[0]);
        lds_barrier();
        // behind barrier n pair n + 1 is converted, and pair n + 1 + D requested into its registers
        auto step = [&]<int I>(std::integral_constant<int, I>, int n) -> bool {
            const bool more = n + 1 < sg.L;
            if (more) {
                src.convert(w[(I + 1) % D], wsm + ((I + 1) & 1) * WORD_STAGE);
                src.request(n + 1 + D, w[(I + 1) % D]);
            }
            lds_barrier();
            return more;
        };
        // (leaving by a jump out of the loop: paths with different loads in flight must not join)
        for (int n = 0;; n += 6) {
            if (!step(std::integral_constant<int, 0>{}, n)) break;
            if (!step(std::integral_constant<int, 1>{}, n + 1)) break;
            if (!step(std::integral_constant<int, 2>{}, n + 2)) break;
            if (!step(std::integral_constant<int, 3>{}, n + 3)) break;
            if (!step(std::integral_constant<int, 4>{}, n + 4)) break;
            if (!step(std::integral_constant<int, 5>{}, n + 5)) break;
        }
    }
}

// ---------------------------------------------------------------------------
// the multiplying wavefronts
// ---------------------------------------------------------------------------
// Positions inside a pair, counted in matrix instructions.  Group g (0 .. 7) multiplies weight digit
// 7 - g with the activation digits 0 .. g, four sub-tiles of 16 columns each.
template <int NT>
struct WordMap {
    static constexpr int NM = 36 * NT;
    static constexpr int group_begin(int g) { return g * (g + 1) / 2 * NT; }
    static constexpr int group_of(int m) {
        int g = 0;
        while (m >= group_begin(g + 1)) ++g;
        return g;
    }
    static constexpr int t_of(int m) { return (m - group_begin(group_of(m))) / NT; }
    static constexpr int j_of(int m) { return m % NT; }
    // Three sets of registers hold the weight units of a digit.  The units of groups 0 and 1 are read behind the
    // barrier, in group 7 of the pair before; the others as soon as their registers are free.
    static constexpr int set_of(int g) { return g == 7 ? 2 : g % 3; }
    // Activation digits below TWICE have two sets of registers, the current pair's and the next one's.  The others are used
    // late in a pair only and are requested again behind their last use.
    static constexpr int TWICE = 4;
    static constexpr int BARRIER = group_begin(7);
    static constexpr int read_at(int g) {
        return g == 0 ? BARRIER : g == 1 ? BARRIER + 4 : g == 2 ? 0 : g == 7 ? group_begin(6) : group_begin(g - 2);
    }
    static_assert(set_of(7) != set_of(0) && set_of(7) != set_of(1), "read while group 7 is multiplied");
    static_assert(set_of(7) == set_of(5) && read_at(7) >= group_begin(6), "the registers of group 5 are free");
};

template <bool LISTED>
struct WordRows {
    typedef __attribute__((address_space(1))) const char* gptr;
    gptr abase;                    // the lane's activation unit of step 0, digit 0
    size_t adig;                   // bytes from one activation digit to the next
    u32 astep;                     // bytes of one contraction step
    int k0, L, KS, x0, x1;         // the segment; first steps of the two halves
    const int* steps;

    __device__ __forceinline__ void setup(const GemmParams& p, const Segment& sg, int row0) {
        const int lane = threadIdx.x & 63;
        adig = (size_t)p.mpad * 32;
        astep = (u32)p.mpad * 256u;                        // (rows stay below 2^22: host check)
        // a lane's k-group of the 64: two 16-word halves of two steps
        abase = (gptr)p.xp + ((size_t)((lane >> 4) & 1) * p.mpad + row0 + (lane & 15)) * 16;
        k0 = sg.k0; L = sg.L; KS = sg.KS; steps = sg.steps;
        x0 = p.xstep[0];
        x1 = p.xstep[1];
    }
    // the step of the activation planes that the lane's k-group of pair q belongs to
    __device__ __forceinline__ int at(int q) const {
        const int ks = 2 * (k0 + (q < L ? q : L - 1)) + (int)((threadIdx.x & 63) >> 5);
        const int h = ks >= KS ? 1 : 0;
        int s = ks - h * KS;
        if constexpr (LISTED) s = steps[s];
        return (h ? x1 : x0) + s;
    }
    __device__ __forceinline__ gptr unit(int x) const { return abase + (size_t)(u32)x * astep; }
    static __device__ __forceinline__ v4i load(gptr q) { return *reinterpret_cast<__attribute__((address_space(1))) const v4i*>(q); }
};

__device__ __forceinline__ void word_mfma(v4i& acc, const v4i& a, const v4i& b) {
    acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, acc, 0, 0, 0);
}

// One pair: a and a_high hold its activation units, a_next and a_high take the next pair's; b holds the units of groups 0 and 1.
template <bool LISTED, int... Ms>
__device__ __forceinline__ void word_pair(std::integer_sequence<int, Ms...>, const WordRows<LISTED>& st, v4i (&acc)[4][8],
                                          const v4i (&a)[WordMap<4>::TWICE], v4i (&a_next)[WordMap<4>::TWICE],
                                          v4i (&a_high)[8 - WordMap<4>::TWICE], v4i (&b)[3][4], const unsigned char* rd,
                                          const unsigned char* rd_next, int& x, int q_after) {
    using PM = WordMap<4>;
    typename WordRows<LISTED>::gptr ap = st.unit(x);
    if constexpr (LISTED) x = st.at(q_after);              // (requested a pair ahead of its use)
    (
        [&] {
            constexpr int M = Ms, g = PM::group_of(M), t = PM::t_of(M), j = PM::j_of(M), u = 7 - g;
            if constexpr (M == PM::BARRIER) lds_barrier();
            if constexpr (t < PM::TWICE) word_mfma(acc[j][t + u], a[t], b[PM::set_of(g)][j]);
            else word_mfma(acc[j][t + u], a_high[t - PM::TWICE], b[PM::set_of(g)][j]);
            [&]<int... Gs>(std::integer_sequence<int, Gs...>) {
                ([&] {
                    constexpr int off = M - PM::read_at(Gs);
                    if constexpr (off >= 0 && off < 4)
                        b[PM::set_of(Gs)][off] = lds_frag((Gs < 2 ? rd_next : rd) + ((7 - Gs) * 4 * WORD_BN + off * 16) * 16);
                }(), ...);
            }(std::make_integer_sequence<int, 8>{});
            // the next pair's activation units, digit by digit
            if constexpr (M >= 4 && M < 4 + 4 * PM::TWICE && M % 4 == 0) {
                a_next[M / 4 - 1] = st.load(ap);
                ap += st.adig;
            }
            if constexpr (g == 7 && t >= PM::TWICE && j == 3) {
                a_high[t - PM::TWICE] = st.load(ap);
                if constexpr (t < 7) ap += st.adig;
            }
            __builtin_amdgcn_sched_barrier(0);
        }(),
        ...);
    if constexpr (!LISTED) x = st.at(q_after);
}

template <bool LISTED>
__device__ __forceinline__ void word_multiply(const GemmParams& p, const Geometry& q, UnitWalk<LISTED>& walk, const bool own,
                                              int wave, const unsigned char* wsm) {
    using PM = WordMap<4>;
    const int lane = threadIdx.x & 63;
    const int g = lane >> 4, r = lane & 15;
    const unsigned char* rd0 = wsm + (g * WORD_BN + r) * 16;
    const unsigned char* rd1 = rd0 + WORD_STAGE;
    WordRows<LISTED> st;
    Segment sg;
    while (walk.next(sg)) {
        const int row0 = sg.tm * WORD_BM + wave * 16, L = sg.L;
        st.setup(p, sg, row0);
        v4i acc[4][8];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int s = 0; s < 8; ++s) acc[j][s] = v4i{0, 0, 0, 0};
        v4i a0[PM::TWICE], a1[PM::TWICE], ah[8 - PM::TWICE], b[3][4];
        {
            typename WordRows<LISTED>::gptr ap = st.unit(st.at(0));
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                if (t < PM::TWICE) a0[t] = st.load(ap);
                else ah[t - PM::TWICE] = st.load(ap);
                ap += st.adig;
            }
        }
        int x = st.at(1);
        lds_barrier();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) b[i][j] = lds_frag(rd0 + ((7 - i) * 4 * WORD_BN + j * 16) * 16);
        for (int n = 0;; n += 2) {
            word_pair<LISTED>(std::make_integer_sequence<int, PM::NM>{}, st, acc, a0, a1, ah, b, rd0, rd1, x, n + 2);
            if (n + 1 >= L) break;
            word_pair<LISTED>(std::make_integer_sequence<int, PM::NM>{}, st, acc, a1, a0, ah, b, rd1, rd0, x, n + 3);
            if (n + 2 >= L) break;
        }

        // The only writer of a tile (own) stores Z = C + sum (Z += sum for a later segment of a long
        // contraction: this lane's own earlier store).  Slices of a shared tile meet in Z, which started out
        // as C, through atomic adds.
        const u64* src = sg.k0 == 0 ? p.C : p.Z;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = sg.tn * WORD_BN + j * 16 + r;
            const int ccomp = (p.row_comp && col < q.n_eff) ? p.blk_comp[col / p.bs] : 0;
            u64 prev[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = row0 + 4 * g + e;
                prev[e] = 0;
                if (own && row < q.m_eff && col < q.n_eff) prev[e] = src[(size_t)row * p.ldz + col];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = row0 + 4 * g + e;
                const v4i (&s)[8] = acc[j];
                const u64 z = recombine(s[0][e], s[1][e], s[2][e], s[3][e], s[4][e], s[5][e], s[6][e], s[7][e]);
                bool live = row < q.m_eff && col < q.n_eff;
                if (live && p.row_comp) live = p.row_comp[row] == ccomp;   // on a result block
                if (live) {
                    if (own) p.Z[(size_t)row * p.ldz + col] = prev[e] + z;
                    else atomicAdd(p.Z + (size_t)row * p.ldz + col, z);
                }
            }
        }
    }
}

template <int KIND, int ROWS, bool LISTED, bool NT = false>
__global__ __launch_bounds__(WORD_THREADS, 1) void ring_words_kernel(GemmParams p) {
    __shared__ __align__(16) unsigned char wsm[2 * WORD_STAGE];
    constexpr int TAB = WordSource<KIND, ROWS, LISTED, NT>::TAB;
    __shared__ int tab[TAB > 0 ? 4 : 1][TAB > 0 ? TAB * WORD_LEN : 1];
    const Geometry q = gemm_geometry<WORD_BM, WORD_BN, KIND, LISTED>(p);
    if (q.units == 0) return;
    const int G = gridDim.x;
    const int b = xcd_contiguous(blockIdx.x, G);
    const bool own = owns_tiles(p, q.m_eff, q.n_eff, q.kc);
    UnitWalk<LISTED> walk(p, q, b, G, own);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (wave < 4) word_multiply<LISTED>(p, q, walk, own, wave, wsm);
    else word_feed<KIND, ROWS, LISTED, NT>(p, q, walk, wave - 4, wsm, tab[TAB > 0 ? wave - 4 : 0]);
}

// The kernel variant for a call, instantiated explicitly in translation units of their own (ring_words_*.hip).
template <bool LISTED>
GemmKernel words_kernel_for(const GemmParams& p) {
    if (p.kind == KIND_SIMM) {
        if (!p.b_full) return p.w_nt ? ring_words_kernel<KIND_SIMM, ROWS_PLAIN, LISTED, true>
                                     : ring_words_kernel<KIND_SIMM, ROWS_PLAIN, LISTED, false>;
        if (p.bs % 16 == 0) return p.w_nt ? ring_words_kernel<KIND_SIMM, ROWS_GATHER16, LISTED, true>
                                          : ring_words_kernel<KIND_SIMM, ROWS_GATHER16, LISTED, false>;
        return ring_words_kernel<KIND_SIMM, ROWS_GATHER, LISTED>;
    }
    if constexpr (LISTED) {
        return nullptr;      // step lists belong to Protocol 3
    } else {
        if (p.w_tr) return ring_words_kernel<KIND_SOMM, ROWS_TR, false>;
        return p.w_nt ? ring_words_kernel<KIND_SOMM, ROWS_PLAIN, false, true>
                      : ring_words_kernel<KIND_SOMM, ROWS_PLAIN, false, false>;
    }
}
extern template GemmKernel words_kernel_for<false>(const GemmParams&);
extern template GemmKernel words_kernel_for<true>(const GemmParams&);

inline int launch_words(comet_ctx* ctx, const char* what, const GemmParams& p) {
    const GemmKernel kern = p.step_list ? words_kernel_for<true>(p) : words_kernel_for<false>(p);
    if (!kern || p.w_planes) return comet_fail(ctx, COMET_EINVAL, "%s: no kernel variant for this call", what);
    if (p.tile_bm != WORD_BM || p.tile_bn != WORD_BN || p.grid < 1)
        return comet_fail(ctx, COMET_EINVAL, "%s: launch plan does not match the kernel", what);
    return launch_share_kernel(ctx, what, kern, dim3((unsigned)p.grid), p, WORD_THREADS);
}

}  // namespace comet_gemm
