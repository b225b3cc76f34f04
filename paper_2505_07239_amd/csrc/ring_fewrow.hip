// One party's output share (paper Eq. 1 on the indexed sub-matrices of Protocols 2 and 3)
//
//     [Z]_i = [C]_i + [ E | A' ] . [ B_i ; F ],   A' = A_i + party * E      (mod 2^64)
//
// for at most 32 activation rows (a decoding batch) on weight planes, and for small products of any number
// of rows.  A product of few rows is bound by reading B_i and F once: every weight fragment feeds exactly one
// matrix instruction per digit pair, so staging it in LDS for other wavefronts buys nothing; a small product
// is bound by how soon its few contraction steps are under way and written out, and stages and barriers are
// in the way of that.
// Here every wavefront works on its own, without a barrier anywhere in the kernel:
//   * it owns 32 x 32 outputs and a run of the stacked contraction; per contraction step of 32
//     it loads its weight and activation fragments straight from memory into registers, two steps
//     ahead of their use, and issues the 36 digit-pair instructions (v_mfma_i32_32x32x32_i8) into eight
//     int32 planes.  Both plane formats are stored in matrix-instruction operand order (a fragment is one
//     16-byte load per lane); of weight WORDS a lane loads the sixteen contraction words of its column
//     itself, splits them into digits and byte-transposes them in its registers, which gives its eight
//     fragments;
//   * the four wavefronts of a workgroup take four adjacent column tiles at the same contraction
//     steps, so the workgroup reads 32 KB of consecutive weight planes per step and its
//     activation fragments (the same for all four, a few MB in all) come from the cache;
//   * the (tile, step) units, of all members of a group, are dealt out evenly over the workgroups; a run ends
//     at a tile's last step or after 256 steps (a plane cannot overflow before that), its
//     planes are recombined and added onto Z, which started out as C, with 64-bit atomics:
//     addition mod 2^64 is associative and commutative, so the result is bit-exact for any split.
// The block gather of Protocols 2 and 3 is folded into the addressing: a column offset per lane
// (SOMM with a full-size B_i) or looked-up rows (SIMM).
#include "ring_words.h"

namespace {

using namespace comet_gemm;

constexpr int FT = 256;          // threads per workgroup
constexpr int FW = FT / 64;      // independent wavefronts
constexpr int FCOLS = 32 * FW;   // output columns per workgroup
constexpr int FSEG = 256;        // longest run of steps between two recombinations
constexpr int FST = 3;           // sets of fragment registers: two steps ahead

// A run of contraction steps of one output tile.
struct Run {
    int tm, cg;          // row tile, column group
    int q0, len;         // steps [q0, q0 + len) of the stacked contraction
};

// Weight fragments from digit planes.  GATHER: SIMM with a full-size B_i, whose rows are looked up once per run (a load
// from the index list inside the pipelined loop would have to wait for every weight load issued before it).
template <int KIND, bool GATHER>
struct PlaneFragments {
    static constexpr int TAB = KIND == KIND_SIMM && GATHER ? 2 : 0, SEG = FSEG;   // rows looked up per step, longest run
    struct Set { v4i f[8]; };
    const GemmParams& p;
    const int KS, lane;
    const size_t prow_b, prow_f;
    const int* tab;
    int q0;
    unsigned off_b, off_f;

    __device__ __forceinline__ PlaneFragments(const GemmParams& p_, int KS_, int)
        : p(p_), KS(KS_), lane(threadIdx.x & 63), prow_b((size_t)((p_.ldb + 63) >> 6) * 16384u),
          prow_f((size_t)((p_.ldf + 63) >> 6) * 16384u) {}

    __device__ __forceinline__ void begin(const Run& run, int col, int kc, int* table) {
        const int g = lane >> 5;
        long bcol = col;
        if (KIND == KIND_SOMM && GATHER) {
            const int blk = col / p.bs;
            const long st = block_start(p, blk);
            bcol = (st < 0 ? 0 : st) + (col - blk * p.bs);
        }
        // the lane's byte offset inside a contraction step of each weight operand (columns stay
        // below 2^24: host check), with the k-half it feeds
        off_b = (unsigned)(bcol >> 6) * 16384u + (unsigned)(bcol & 63) * 16u + (unsigned)g * 1024u;
        off_f = (unsigned)(col >> 6) * 16384u + (unsigned)(col & 63) * 16u + (unsigned)g * 1024u;
        q0 = run.q0;
        tab = table;
        if constexpr (TAB > 0) {
            for (int i = lane; i < 2 * run.len; i += 64) {
                const int q = q0 + (i >> 1);
                int row = 0;
                if (q < KS) {
                    // bs is a multiple of 16 (host check), so the sixteen rows lie inside one block;
                    // beyond the contraction the activation digits are zero and any valid rows do
                    int kb = q * KSTEP + 16 * (i & 1);
                    kb = kb <= kc - 16 ? kb : kc - 16;
                    const int blk = p.bs_shift >= 0 ? (kb >> p.bs_shift) : kb / p.bs;
                    const long st = block_start(p, blk);
                    row = (int)(st < 0 ? 0 : st) + (kb - blk * p.bs);
                }
                table[i] = row;
            }
        }
    }

    __device__ __forceinline__ void load(int q, Set& w) const {
        const int h = q >= KS ? 1 : 0;
        const int s = q - h * KS;
        const char* const Bp = reinterpret_cast<const char*>(p.B);
        const char* const Fp = reinterpret_cast<const char*>(p.F);
        if (TAB > 0 && h == 0) {
            // the lane's sixteen rows start at its own row of B_i
            const int g = lane >> 5, row = tab[2 * (q - q0) + g];
            const char* wb = Bp + (size_t)(row >> 5) * prow_b + (size_t)((row >> 4) & 1) * 1024u +
                             (off_b - (unsigned)g * 1024u);
#pragma unroll
            for (int t = 0; t < 8; ++t)
                w.f[t] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(wb + t * 2048));
        } else {
            // rows 32 s + 16 g + 0..15: step s of the operand, the k-half is in the lane's offset
            const char* ws = (h ? Fp : Bp) + (size_t)s * (h ? prow_f : prow_b);
            const unsigned off = h ? off_f : off_b;
#pragma unroll
            for (int t = 0; t < 8; ++t)
                w.f[t] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(ws + t * 2048 + off));
        }
    }
    static __device__ __forceinline__ void finish(const Set& w, v4i (&f)[8]) {
#pragma unroll
        for (int t = 0; t < 8; ++t) f[t] = w.f[t];
    }
};

// Weight fragments from words.  ROWS (ring_words.h): how the sixteen rows are found.
template <int KIND, int ROWS>
struct WordFragments {
    static constexpr int TAB = ROWS == ROWS_GATHER ? 32 : ROWS == ROWS_GATHER16 ? 2 : 0;
    static constexpr int SEG = ROWS == ROWS_GATHER ? 64 : FSEG;
    struct Set { u64 w[16]; };
    typedef u64 u64x2 __attribute__((ext_vector_type(2)));
    const GemmParams& p;
    const int KS, kc, lane;
    const u32 pitch_b, pitch_f;              // (below 2^27 bytes: host check)
    const int* tab;
    int q0;
    u32 off_b, off_f;                        // the lane's first word of a step
    const u64* tr_b;                         // ROWS_TR: the lane's row of k words
    const u64* tr_f;

    __device__ __forceinline__ WordFragments(const GemmParams& p_, int KS_, int kc_)
        : p(p_), KS(KS_), kc(kc_), lane(threadIdx.x & 63), pitch_b((u32)p_.ldb * 8u), pitch_f((u32)p_.ldf * 8u) {}

    __device__ __forceinline__ void begin(const Run& run, int col, int, int* table) {
        long bcol = col;
        if (KIND == KIND_SOMM && p.b_full) {
            const int blk = col / p.bs;
            const long st = block_start(p, blk);
            bcol = (st < 0 ? 0 : st) + (col - blk * p.bs);
        }
        off_b = (u32)bcol * 8u;
        off_f = (u32)col * 8u;
        if constexpr (ROWS == ROWS_TR) {
            tr_b = p.B + bcol * p.ldb;
            tr_f = p.F + (long)col * p.ldf;
        }
        q0 = run.q0;
        tab = table;
        if constexpr (TAB > 0) {
            // rows of B_i in its own numbering, of F as they come; past the end of the contraction any
            // valid row does (its activation digits are zero)
            for (int i = lane; i < TAB * run.len; i += 64) {
                const int q = q0 + i / TAB, h = q >= KS ? 1 : 0;
                int k = (q - h * KS) * KSTEP;
                if constexpr (ROWS == ROWS_GATHER16) {
                    k += 16 * (i & 1);
                    k = k <= kc - 16 ? k : kc - 16;            // (bs is a multiple of 16: the rows lie inside one block)
                } else {
                    k += i % TAB;
                    k = k < kc ? k : kc - 1;
                }
                if (h == 0) {
                    const int blk = k / p.bs;
                    const long st = block_start(p, blk);
                    k = (int)(st < 0 ? 0 : st) + (k - blk * p.bs);
                }
                table[i] = k;
            }
        }
    }

    __device__ __forceinline__ void load(int q, Set& set) const {
        const int h = q >= KS ? 1 : 0, s = q - h * KS, g = lane >> 5;
        u64 (&w)[16] = set.w;
        if constexpr (ROWS == ROWS_TR) {
            // k is even and the rows are 16-byte aligned (host check)
            const u64* src = h ? tr_f : tr_b;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                int k = s * KSTEP + 16 * g + 2 * j;
                k = k <= kc - 2 ? k : kc - 2;
                const u64x2 v = *reinterpret_cast<const u64x2*>(src + k);
                w[2 * j] = v.x;
                w[2 * j + 1] = v.y;
            }
            return;
        }
        const char* const op = reinterpret_cast<const char*>(h ? p.F : p.B);
        const u32 pitch = h ? pitch_f : pitch_b, off = h ? off_f : off_b;
        if constexpr (ROWS == ROWS_GATHER) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                w[i] = *reinterpret_cast<const u64*>(op + (size_t)(u32)tab[TAB * (q - q0) + 16 * g + i] * pitch + off);
        } else if constexpr (ROWS == ROWS_GATHER16) {
            const char* a = op + (size_t)(u32)tab[2 * (q - q0) + g] * pitch + off;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                w[i] = *reinterpret_cast<const u64*>(a);
                a += pitch;
            }
        } else {
            // rows as they come, past the end of the contraction the last one over and over
            const int last = kc - 1 - s * KSTEP;
            const char* const row = op + (size_t)(s * KSTEP) * pitch;
            u32 o = off + (u32)(16 * g < last ? 16 * g : last) * pitch;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                w[i] = *reinterpret_cast<const u64*>(row + o);
                o += 16 * g + i < last ? pitch : 0u;
            }
        }
    }
    static __device__ __forceinline__ void finish(const Set& set, v4i (&f)[8]) {
        u64 plane[2][8];
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            u64 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = to_digits(set.w[8 * o + i]);
            digits_to_planes(v, plane[o]);
        }
#pragma unroll
        for (int t = 0; t < 8; ++t)
            f[t] = v4i{(int)(u32)plane[0][t], (int)(plane[0][t] >> 32), (int)(u32)plane[1][t], (int)(plane[1][t] >> 32)};
    }
};

template <int KIND>
struct FewGeometry {
    int n_eff, kc, m_eff, KS, KT, tiles_m;
    long units;                              // (row tile, column group, step) of one product
    __device__ __forceinline__ explicit FewGeometry(const GemmParams& p) {
        const int nblk = n_blocks(p);
        n_eff = KIND == KIND_SOMM ? nblk * p.bs : p.n_cap;
        kc = KIND == KIND_SOMM ? p.kc_cap : nblk * p.bs;
        m_eff = n_rows(p);
        KS = (kc + KSTEP - 1) / KSTEP;
        KT = 2 * KS;
        tiles_m = (m_eff + 31) / 32;
        units = n_eff <= 0 ? 0 : (long)tiles_m * ((n_eff + FCOLS - 1) / FCOLS) * KT;
    }
};

// The units [u, u_end) of one product.
template <int KIND, class Fragments>
__device__ __forceinline__ void fewrow_sweep(const GemmParams& p, const FewGeometry<KIND>& q, long u, const long u_end, int* tab) {
    const int KS = q.KS, KT = q.KT;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = lane & 31, g = lane >> 5;
    // Activation fragment of (step, digit t): unit xp_group(0, step, t, g) * mpad + row, i.e. a wave-uniform
    // address and a 32-bit offset per lane
    const char* const Xp = reinterpret_cast<const char*>(p.xp);
    const unsigned x_off = (unsigned)((g * p.mpad + r) * 16);
    const size_t x_digit = (size_t)2 * p.mpad * 16;            // bytes from one digit to the next
    Fragments frag(p, KS, q.kc);

    while (u < u_end) {
        Run run;
        const int tile = (int)(u / KT);
        run.q0 = (int)(u - (long)tile * KT);
        run.tm = tile % q.tiles_m;
        run.cg = tile / q.tiles_m;
        run.len = KT - run.q0;
        if (run.len > u_end - u) run.len = (int)(u_end - u);
        if (run.len > Fragments::SEG) run.len = Fragments::SEG;
        u += run.len;
        const int q0 = run.q0, qe = run.q0 + run.len;
        if (run.cg * FCOLS + wave * 32 >= q.n_eff) continue;    // a column tile beyond the last column
        const int out_col = run.cg * FCOLS + wave * 32 + r;
        frag.begin(run, out_col < q.n_eff ? out_col : q.n_eff - 1, q.kc, tab);
        const char* const xrow = Xp + (size_t)run.tm * 32 * 16;

        typename Fragments::Set w[FST];
        v4i xa[FST][8];
        v16i acc[8];
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[s][e] = 0;

        auto issue = [&](int i, v4i (&xf)[8], typename Fragments::Set& wf) {
            const int h = i >= KS ? 1 : 0;
            const char* xs = xrow + xp_group(0, (h ? p.xstep[1] : p.xstep[0]) + i - h * KS, 0, 0, 0) * p.mpad * 16;
#pragma unroll
            for (int t = 0; t < 8; ++t) xf[t] = *reinterpret_cast<const v4i*>(xs + t * x_digit + x_off);
            frag.load(i, wf);
        };
        auto step = [&](const v4i (&af)[8], const typename Fragments::Set& set) {
            v4i wf[8];
            Fragments::finish(set, wf);
#pragma unroll
            for (int t = 0; t < 8; ++t)
#pragma unroll
                for (int uu = 0; uu + t < 8; ++uu)
                    acc[t + uu] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[t], wf[uu], acc[t + uu], 0, 0, 0);
        };

#pragma unroll
        for (int i = 0; i < FST - 1; ++i)
            if (q0 + i < qe) issue(q0 + i, xa[i], w[i]);
        for (int s = q0; s < qe; s += FST) {
#pragma unroll
            for (int i = 0; i < FST; ++i) {
                if (s + i < qe) {
                    if (s + i + FST - 1 < qe)
                        issue(s + i + FST - 1, xa[(i + FST - 1) % FST], w[(i + FST - 1) % FST]);
                    step(xa[i], w[i]);
                }
            }
        }

#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int row = run.tm * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
            const u64 z = recombine(acc[0][e], acc[1][e], acc[2][e], acc[3][e], acc[4][e], acc[5][e], acc[6][e], acc[7][e]);
            if (row < q.m_eff && out_col < q.n_eff) atomicAdd(p.Z + (size_t)row * p.ldz + out_col, z);
        }
    }
}

#define COMET_FEWROW_TAB(Fragments)                                                                     \
    __shared__ __align__(16) int row_tab[Fragments::TAB ? FW : 1][Fragments::TAB ? Fragments::TAB * Fragments::SEG : 1]; \
    int* const tab = row_tab[Fragments::TAB ? threadIdx.x >> 6 : 0]

template <int KIND, class Fragments>
__global__ __launch_bounds__(FT) void ring_fewrow_kernel(GemmParams p) {
    COMET_FEWROW_TAB(Fragments);
    const FewGeometry<KIND> q(p);
    const int G = gridDim.x;
    const int b = xcd_contiguous(blockIdx.x, G);
    fewrow_sweep<KIND, Fragments>(p, q, q.units * b / G, q.units * (b + 1) / G, tab);
}

// The members of a group (one shape): their units follow each other.
template <int KIND, class Fragments>
__global__ __launch_bounds__(FT) void ring_fewrow_group_kernel(GemmGroup grp) {
    COMET_FEWROW_TAB(Fragments);
    const FewGeometry<KIND> q(grp.p[0]);
    if (q.units == 0) return;
    const int G = gridDim.x;
    const int b = xcd_contiguous(blockIdx.x, G);
    const long total = q.units * grp.n, u_end = total * (b + 1) / G;
    long u = total * b / G;
#pragma nounroll
    for (int j = (int)(u / q.units); u < u_end; ++j) {
        const long base = (long)j * q.units, hi = u_end - base < q.units ? u_end - base : q.units;
        fewrow_sweep<KIND, Fragments>(grp.p[j], q, u - base, hi, tab);
        u = base + q.units;
    }
}

// The smallest products: one launch and nothing around it.  A workgroup owns a tile of 32 x 32 outputs; each of its eight
// wavefronts takes one step of the stacked contraction, loads the words of E and A_i itself (sixteen of a row
// per lane, split and transposed like weight words); they meet in LDS and store Z = C + sum: no packed
// activations, no Z := C ahead, no atomics.  What bounds it is the latency of three dependent loads and the rows of E that a
// wavefront reads word by word; against packing and the few-row kernel see takes_direct() in ring_gemm.hip.
constexpr int DT = 512;                      // threads
constexpr int DW = DT / 64;                  // wavefronts, and steps of the stacked contraction at most (host check)

template <int KIND, class Fragments>
__global__ __launch_bounds__(DT) void ring_direct_kernel(GemmParams p) {
    __shared__ __align__(16) u64 red[DW][32 * 32];
    __shared__ __align__(16) int row_tab[Fragments::TAB ? DW : 1][Fragments::TAB ? Fragments::TAB : 1];
    const FewGeometry<KIND> q(p);
    const int KS = q.KS, kc = q.kc;
    const int tiles_m = (p.m + 31) / 32;
    const int tm = (int)(blockIdx.x % (unsigned)tiles_m), tn = (int)(blockIdx.x / (unsigned)tiles_m);
    if (tm * 32 >= q.m_eff || tn * 32 >= q.n_eff) return;      // uniform over the workgroup
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = lane & 31, g = lane >> 5;
    if (wave < q.KT) {
        const Run run = {tm, tn, wave, 1};
        const int out_col = tn * 32 + r, row = tm * 32 + r;
        const size_t arow = (size_t)(row < q.m_eff ? row : q.m_eff - 1);   // (its results are never stored)
        Fragments frag(p, KS, kc);
        frag.begin(run, out_col < q.n_eff ? out_col : q.n_eff - 1, kc, row_tab[Fragments::TAB ? wave : 0]);
        typename Fragments::Set w;
        frag.load(wave, w);
        // words of [E | A'] of the lane's row, zero beyond the contraction (whatever the weight side reads there)
        const int h = wave >= KS ? 1 : 0, k0 = (wave - h * KS) * KSTEP + 16 * g;
        typename WordFragments<KIND, ROWS_PLAIN>::Set x;
        // (sixteen indices lie in one block when bs is a multiple of 16)
        const bool one_block = KIND == KIND_SIMM && p.a_full && p.bs % 16 == 0;
        const int blk0 = one_block ? (k0 < kc ? k0 : kc - 16) / p.bs : 0;
        const long st0 = one_block ? block_start(p, blk0) : 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int k = k0 + j < kc ? k0 + j : kc - 1;
            u64 v = 0;
            if (h == 0 || p.party) v = p.E[arow * p.lde + k];              // party 0's A' is A_i itself
            if (h) {
                long col = k;
                if (one_block) {
                    col = (st0 < 0 ? 0 : st0) + (k - blk0 * p.bs);
                } else if (KIND == KIND_SIMM && p.a_full) {
                    const int blk = k / p.bs;
                    const long st = block_start(p, blk);
                    col = (st < 0 ? 0 : st) + (k - blk * p.bs);
                }
                v += p.A[arow * p.lda + col];
            }
            x.w[j] = k0 + j < kc ? v : 0;
        }
        v4i af[8], wf[8];
        WordFragments<KIND, ROWS_PLAIN>::finish(x, af);
        Fragments::finish(w, wf);
        v16i acc[8];
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[s][e] = 0;
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int uu = 0; uu + t < 8; ++uu)
                acc[t + uu] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[t], wf[uu], acc[t + uu], 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 16; ++e)
            red[wave][(8 * (e >> 2) + 4 * g + (e & 3)) * 32 + r] =
                recombine(acc[0][e], acc[1][e], acc[2][e], acc[3][e], acc[4][e], acc[5][e], acc[6][e], acc[7][e]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 32 * 32 / DT; ++i) {
        const int at = i * DT + threadIdx.x, zr = tm * 32 + (at >> 5), zc = tn * 32 + (at & 31);
        if (zr < q.m_eff && zc < q.n_eff) {
            const size_t o = (size_t)zr * p.ldz + zc;
            u64 z = p.C[o];
            for (int s = 0; s < q.KT; ++s) z += red[s][at];
            p.Z[o] = z;
        }
    }
}

// One workgroup per compute unit: the accumulator planes and the fragments in flight take a wavefront's whole register
// budget, so that is what the chip holds at once.
int fewrow_grid(const comet_ctx* ctx, const GemmParams& p, int members) {
    const long units = (long)((p.m + 31) / 32) * ((p.n_cap + FCOLS - 1) / FCOLS) * 2 * p.ks_cap * members;
    const long grid = ctx->gemm_grid > 0 ? ctx->gemm_grid : ctx->num_cu;
    return (int)(grid < units ? grid : units > 0 ? units : 1);
}

}  // namespace

// The variant of a kernel for a call.
static_assert(DW * KSTEP == 2 * COMET_DIRECT_MAX_K, "a step per wavefront");
#define COMET_FEW_PLANES(kernel, p)                                                                      \
    ((p).kind == KIND_SOMM ? ((p).b_full ? kernel<KIND_SOMM, PlaneFragments<KIND_SOMM, true>>              \
                                         : kernel<KIND_SOMM, PlaneFragments<KIND_SOMM, false>>)            \
                           : ((p).b_full ? kernel<KIND_SIMM, PlaneFragments<KIND_SIMM, true>>              \
                                         : kernel<KIND_SIMM, PlaneFragments<KIND_SIMM, false>>))
#define COMET_FEW_WORDS(kernel, p)                                                                       \
    ((p).kind == KIND_SOMM ? ((p).w_tr ? kernel<KIND_SOMM, WordFragments<KIND_SOMM, ROWS_TR>>              \
                                       : kernel<KIND_SOMM, WordFragments<KIND_SOMM, ROWS_PLAIN>>)          \
     : !(p).b_full         ? kernel<KIND_SIMM, WordFragments<KIND_SIMM, ROWS_PLAIN>>                       \
     : (p).bs % 16 == 0    ? kernel<KIND_SIMM, WordFragments<KIND_SIMM, ROWS_GATHER16>>                    \
                           : kernel<KIND_SIMM, WordFragments<KIND_SIMM, ROWS_GATHER>>)

static bool few_ok(const GemmParams& p) { return p.m >= 1 && !p.row_comp && !p.tmask && !(p.w_planes && p.w_tr); }

int comet_launch_fewrow(comet_ctx* ctx, const char* what, const GemmParams& p) {
    if (!few_ok(p)) return comet_fail(ctx, COMET_EINVAL, "%s: operands outside the few-row matrix-core path", what);
    const GemmKernel kern = p.w_planes ? COMET_FEW_PLANES(ring_fewrow_kernel, p) : COMET_FEW_WORDS(ring_fewrow_kernel, p);
    return launch_share_kernel(ctx, what, kern, dim3((unsigned)fewrow_grid(ctx, p, 1)), p, FT);
}

int comet_launch_fewrow_group(comet_ctx* ctx, const char* what, const GemmGroup& grp) {
    const GemmParams& p = grp.p[0];
    if (grp.n < 1 || grp.n > GROUP_MAX || !p.w_planes || !few_ok(p))
        return comet_fail(ctx, COMET_EINVAL, "%s: operands outside the few-row matrix-core path", what);
    const GemmGroupKernel kern = COMET_FEW_PLANES(ring_fewrow_group_kernel, p);
    return launch_share_kernel(ctx, what, kern, dim3((unsigned)fewrow_grid(ctx, p, grp.n)), grp, FT);
}

int comet_launch_direct(comet_ctx* ctx, const char* what, const GemmParams& p) {
    const long tiles = (long)((p.m + 31) / 32) * ((p.n_cap + 31) / 32);
    if (!few_ok(p) || p.kc_cap > COMET_DIRECT_MAX_K || tiles < 1 || tiles > (1 << 20))
        return comet_fail(ctx, COMET_EINVAL, "%s: operands outside the path of the smallest products", what);
    const GemmKernel kern = p.w_planes ? COMET_FEW_PLANES(ring_direct_kernel, p) : COMET_FEW_WORDS(ring_direct_kernel, p);
    return launch_share_kernel(ctx, what, kern, dim3((unsigned)tiles), p, DT);
}
