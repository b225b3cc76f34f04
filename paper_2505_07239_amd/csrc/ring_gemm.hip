// One party's output share of the Beaver-triple matrix product (paper Eq. 1 in
// matrix form, invoked on the indexed sub-matrices of Protocols 2 and 3):
//
//     [Z]_i = [C]_i + E [B]_i + [A]_i F + party * E F          (mod 2^64)
//
// Formulation used here
//   * E F + [A]_i F = (E + [A]_i) F, so each party needs exactly two products,
//     and they share one accumulator when the contraction axes are stacked:
//         [Z]_i = [C]_i + [ E | A' ] . [ B_i ; F ],   A' = A_i + party * E.
//   * A 64-bit ring product is carried out on the int8 matrix cores.  Every
//     operand word x is rewritten as eight SIGNED base-256 digits,
//         x = sum_t d_t 2^(8t)  (mod 2^64),  d_t in [-128, 127],
//     which costs two 64-bit ALU operations: the bytes of
//     (x + 0x0080808080808080) ^ 0x0080808080808080 are exactly those digits
//     (adding 128 to a byte and flipping its top bit subtracts 128 again, with
//     the borrow already propagated by the addition; the top digit may be
//     read signed because 2^64 = 0).  Then
//         x y = sum_{t+u <= 7} d_t e_u 2^(8(t+u))      (mod 2^64),
//     36 digit products instead of 64, each an int8 x int8 -> int32 GEMM.
//     All digit pairs of equal weight s = t + u share one int32 accumulator:
//     eight accumulator planes per output element, recombined at the end as
//     sum_s sext64(S_s) << 8s.  |d e| <= 2^14 and a plane receives at most
//     8 * 32 products per contraction step, so a plane cannot overflow within
//     MAX_SEG = 256 steps; the schedule below never accumulates more than that
//     before it flushes.
//   * Addition mod 2^64 is associative and commutative, so partial sums may be
//     formed in any order and by any number of workgroups: the (tile, slice of
//     the stacked contraction) work units are dealt out evenly over a fixed,
//     chip-sized grid (a stream-K split) and every run of units inside one
//     tile ends with 64-bit atomic adds onto Z, which starts out as [C]_i.
//     The result is bit-exact whatever the split.  When the grid divides the
//     number of tiles every workgroup owns whole tiles instead: it stores
//     Z = C + sum itself and no atomic add is issued (owns_tiles()).
//   * Several products of one shape (comet_share_group) run as one launch over
//     the concatenation of their work units.
//
// Data flow
//   xpack kernel : E, A_i  -> digit planes of [E | A'] in the workspace, laid
//                  out so that a tile is a linear copy into LDS (small operand).
//   gemm kernel  : weight-side WORDS are loaded once as uint64 (with the block
//                  gather folded into the addressing), split into digits and
//                  byte-transposed in registers, and fed to the matrix
//                  instructions through LDS (ring_words.h, ring_tile.h) or directly
//                  (ring_fewrow.hip); they are never re-written to
//                  memory.  Weight-side PLANES (COMET_WEIGHT_PLANES: F opened in
//                  that format, B_i packed offline, see wplanes.hip) go to LDS
//                  by LDS-DMA, activation planes straight into registers: a step
//                  then holds nothing but matrix instructions and their fragment
//                  reads (ring_gemm_planes.h).
#include "ring_gemm_planes.h"
#include "ring_tile.h"
#include "ring_words.h"

#include <mutex>

// Scratch of comet_somm_share_static, the entry point for callers that cannot allocate: a
// file-scope device array, one copy per GPU for the life of the process.  In host code the
// name `scratch` is only a handle for hipGetSymbolAddress: the address a kernel may use is the
// one that call returns for the current device, kept in scratch_ptr[] and handed to the kernels
// as an argument like any caller-owned workspace.
constexpr size_t STATIC_SCRATCH_BYTES = COMET_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
static void* scratch_ptr[MAX_DEVICES];
static std::mutex scratch_mutex;

int comet_static_scratch(int device, void** ptr, size_t* bytes) {
    if (device < 0 || device >= MAX_DEVICES || !ptr || !bytes) return COMET_EINVAL;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[device]) {
        void* q = nullptr;
        if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) {
            (void)hipGetLastError();
            return COMET_EDEVICE;
        }
        scratch_ptr[device] = q;
    }
    *ptr = scratch_ptr[device];
    *bytes = STATIC_SCRATCH_BYTES;
    return COMET_OK;
}

namespace {

using namespace comet_gemm;

// ---------------------------------------------------------------------------
// xpack: digit planes of the stacked activation-side operand, and Z := C
// ---------------------------------------------------------------------------
// grid: x = chunks of four 16-word groups, y = chunks of 64 rows, z = 0 (E), 1 (A'), 2 (Z := C).
// A workgroup packs a 64-row x 64-word tile: the lanes of a wavefront read along the rows, and write adjacent 16-byte
// units of 64 rows.
// SETS: with per-token row sets (a variant of its own: their code in the other one cost it 0.1 us a call).
template <bool SETS>
__device__ __forceinline__ void xpack_body(const GemmParams& p, const int part, const int xstep) {
    const int nblk = n_blocks(p);
    const int m_eff = n_rows(p);
    if (part == 2) {
        // Z := C on the kept region (the GEMM adds its partial sums onto it); with result blocks
        // (Protocol 2 in general form) Z := C on the blocks and zero between them
        const int n_eff = p.kind == KIND_SOMM ? nblk * p.bs : p.n_cap;
        // (the share kernel writes Z = C + sum itself when every workgroup owns whole tiles)
        if (owns_tiles(p, m_eff, n_eff, p.kind == KIND_SOMM ? p.kc_cap : nblk * p.bs)) return;
        const long stride = (long)gridDim.x * gridDim.y * GT;
        const long t0 = ((long)blockIdx.y * gridDim.x + blockIdx.x) * GT + threadIdx.x;
        if (((n_eff | p.ldz | p.bs) & 1) == 0 || (!p.row_comp && ((n_eff | p.ldz) & 1) == 0)) {
            // 16-byte accesses (the operands are 16-byte aligned, every row starts on a pair, and
            // a pair never straddles two blocks when that matters)
            typedef u64 u64x2 __attribute__((ext_vector_type(2)));
            const int half = n_eff >> 1;
            const long total = (long)m_eff * half;
            for (long i = t0; i < total; i += stride) {
                const long r = i / half, c = (i - r * half) * 2;
                u64x2 v = *reinterpret_cast<const u64x2*>(p.C + r * p.ldz + c);
                if (p.row_comp && p.row_comp[r] != p.blk_comp[c / p.bs]) v = u64x2{0, 0};
                *reinterpret_cast<u64x2*>(p.Z + r * p.ldz + c) = v;
            }
        } else {
            const long total = (long)m_eff * n_eff;
            for (long i = t0; i < total; i += stride) {
                const long r = i / n_eff, c = i - r * n_eff;
                u64 v = p.C[r * p.ldz + c];
                if (p.row_comp && p.row_comp[r] != p.blk_comp[c / p.bs]) v = 0;
                p.Z[r * p.ldz + c] = v;
            }
        }
        return;
    }
    const int kc = p.kind == KIND_SOMM ? p.kc_cap : nblk * p.bs;
    // The loads want the lanes along k (512 bytes of a row per wavefront or half of one), the stores want them along the
    // rows (a digit group is one run of rows), so the tile passes through LDS in between (row sets aside, see below).
    typedef u64 u64x2 __attribute__((ext_vector_type(2)));
    constexpr int PITCH = 33;                                  // 16-byte vectors per tile row (32 + padding)
    __shared__ u64x2 tile[64 * PITCH];
    const int h = part;                                        // 0: E, 1: A'
    const int kw = blockIdx.x * 64;                            // first word of the workgroup's four groups
    if (kw >= p.ks_cap * KSTEP) return;                        // uniform over the workgroup
    const bool e_too = h == 0 || p.party;                      // party 0's A' is A_i itself
    const int live = m_eff - (int)blockIdx.y * 64;             // rows of the tile that exist (the others pack zeros)
    const bool pairs = ((p.lde | p.lda) & 1) == 0;             // rows start on 16 bytes
    // sixteen words of one row -> their units of the eight digits
    auto store = [&](int trow, int half16, const u64x2 (&w)[8]) {
        u64 plane[2][8];
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            u64 v[8];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[2 * j] = to_digits(w[4 * o + j].x);
                v[2 * j + 1] = to_digits(w[4 * o + j].y);
            }
            digits_to_planes(v, plane[o]);
        }
        const int s = half16 >> 1, g = half16 & 1;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            u64x2* dst = reinterpret_cast<u64x2*>(p.xp) + xp_group(0, xstep + s, t, g, 0) * p.mpad + trow;
            *dst = u64x2{plane[0][t], plane[1][t]};
        }
    };
    if (SETS && pairs && p.bs % 16 == 0) {
        // Row sets, sixteen words in one block: a thread packs sixteen words of one row, so that one flag decides about all
        // of them and nothing else is fetched where it is not set (entries a token does not use take no part, and
        // their values are not read).  Against the way over LDS below, with one flag per word and with one per sixteen: 33 rows
        // x 960 words 5.3 and 5.0 us, 4.6 here; 200 rows, 1 % of the flags set, 5.8, 5.5 and 5.0; 256 x 11008, 15 % set,
        // 15.4, 15.3 and 15.9.
        const int r = threadIdx.x >> 2, half16 = blockIdx.x * 4 + (threadIdx.x & 3);
        const int trow = blockIdx.y * 64 + r, k0 = half16 * 16;
        if (trow >= p.mpad || half16 >= p.ks_cap * 2) return;
        u64x2 w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) w[j] = u64x2{0, 0};
        const int blk = k0 / p.bs;
        if (r < live && k0 < kc && token_uses(p, trow, blk)) {
            if (e_too) {
#pragma unroll
                for (int j = 0; j < 8; ++j) w[j] = *reinterpret_cast<const u64x2*>(p.E + (size_t)trow * p.lde + k0 + 2 * j);
            }
            if (h) {
                const long st = p.a_full ? block_start(p, blk) : 0;
                const long col = p.a_full ? (st < 0 ? 0 : st) + (k0 - (long)blk * p.bs) : k0;
#pragma unroll
                for (int j = 0; j < 8; ++j) w[j] += *reinterpret_cast<const u64x2*>(p.A + (size_t)trow * p.lda + col + 2 * j);
            }
        }
        store(trow, half16, w);
        return;
    }
    if (!SETS && pairs && kw + 64 <= kc && (!p.a_full || p.bs % 16 == 0)) {
        // Whole tile on 16 bytes: two words per lane, all eight rows in flight.  Two members of 128 rows x 768 words 8.5 us
        // with a branch and a wait per row, 6.4 with four in flight, 5.8 with eight; 64 rows x 12288 words 9.8 -> 9.0.
        // A row past the last one reads the last one's words and packs zeros; half a tile that lies behind it as a whole reads
        // nothing (150 rows x 4096 words, 256 padded, 11.8 us when it did, 7.1 without).
        // A_i indexed by blocks of 16 or a multiple too: 256 rows x 1664 gathered words 10.0 us word by word, 8.9 here.
        const int kv = threadIdx.x & 31, r0 = threadIdx.x >> 5;
        long col = kw + 2 * kv;
        if (p.a_full && h) {
            const int blk = (int)col / p.bs;
            const long st = block_start(p, blk);
            col = (st < 0 ? 0 : st) + (col - (long)blk * p.bs);
        }
        const u64* const first = e_too ? p.E + kw + 2 * kv : p.A + col;
        const long ld = e_too ? p.lde : p.lda;
        const size_t row0 = (size_t)blockIdx.y * 64;
        u64x2 x[8], a[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = a[i] = u64x2{0, 0};
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (live <= 32 * half) continue;                   // uniform over the workgroup
#pragma unroll
            for (int i = 4 * half; i < 4 * half + 4; ++i) {
                const int r = 8 * i + r0;
                x[i] = *reinterpret_cast<const u64x2*>(first + (row0 + (r < live ? r : live - 1)) * ld);
            }
            if (h && e_too) {
#pragma unroll
                for (int i = 4 * half; i < 4 * half + 4; ++i) {
                    const int r = 8 * i + r0;
                    a[i] = *reinterpret_cast<const u64x2*>(p.A + col + (row0 + (r < live ? r : live - 1)) * p.lda);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) tile[(8 * i + r0) * PITCH + kv] = 8 * i + r0 < live ? x[i] + a[i] : u64x2{0, 0};
    } else {
        // Word by word, a wavefront along 64 words of a row: what bounds it is the latency of these loads, so a lane keeps
        // its contraction index, looks the block it lies in (indexed A_i, row sets) up once and has sixteen rows in flight.
        // Against a thread that packed sixteen words of one row: 77 rows x 1001 words 13.7 -> 6.2 us, x 819 gathered words
        // 16.2 -> 5.6.
        const int kk = kw + (threadIdx.x & 63), r0 = threadIdx.x >> 6;
        const int k = kk < kc ? kk : kc - 1;
        const size_t row0 = (size_t)blockIdx.y * 64;
        long col = k;
        unsigned uses = kk < kc ? 0xffff : 0;                  // of the sixteen rows
        if (kc > 0 && live > 0 && (p.a_full || SETS)) {
            const int blk = k / p.bs;
            const long st = block_start(p, blk);
            if (p.a_full) col = (st < 0 ? 0 : st) + (k - blk * p.bs);
            if (SETS) {
                // The uses of the rows first, all in flight, then their values (entries a token does not use take no part).
                const long flag = p.blk_idx[blk];
                const bool listed = flag >= 0 && flag < p.tmask_nb;    // (see token_uses)
                unsigned char on[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int r = r0 + 4 * i;
                    on[i] = p.tmask[(long)(row0 + (r < live ? r : live - 1)) * p.tmask_nb + (listed ? flag : 0)];
                }
                unsigned set = 0;
#pragma unroll
                for (int i = 0; i < 16; ++i) set |= (on[i] != 0 ? 1u : 0u) << i;
                uses &= listed ? set : 0;
            }
        }
        u64 x[16], a[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = r0 + 4 * i;
            x[i] = a[i] = 0;
            if (r >= live || !(uses >> i & 1)) continue;
            if (e_too) x[i] = p.E[(row0 + r) * p.lde + k];
            if (h) a[i] = p.A[(row0 + r) * p.lda + col];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i)
            reinterpret_cast<u64*>(tile)[(r0 + 4 * i) * 2 * PITCH + (threadIdx.x & 63)] = x[i] + a[i];
    }
    __syncthreads();
    const int r = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int trow = blockIdx.y * 64 + r, half16 = blockIdx.x * 4 + q;
    if (trow >= p.mpad || half16 >= p.ks_cap * 2) return;      // (the few-row kernel packs 32 rows)
    u64x2 w[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = tile[r * PITCH + 8 * q + j];
    store(trow, half16, w);
}

template <bool SETS>
__global__ __launch_bounds__(GT) void xpack_kernel(GemmParams p) {
    xpack_body<SETS>(p, blockIdx.z, blockIdx.z == 1 ? p.ks_cap : 0);
    // The ticket of step_list_kernel.  Behind the packing: ahead of a store the compiler reads the
    // parameters and the counts in one batch of scalar loads, behind one word by word through vector loads
    // (9 rows, 64 x 64 words: 14.9 us a call with this store first, 14.6 with it last).
    if (SETS && (blockIdx.x | blockIdx.y | blockIdx.z | threadIdx.x) == 0) p.tile_list[0] = 0;
}

// the members of a group (one shape): grid.z = 3 * member + part
__global__ __launch_bounds__(GT) void xpack_group_kernel(GemmGroup grp) {
    const GemmParams& p = grp.p[blockIdx.z / 3];
    const int part = blockIdx.z % 3;
    if (part == 0 && p.x_shared) return;                       // packed with an earlier member
    xpack_body<false>(p, part, p.xstep[part == 1]);
}

// ---------------------------------------------------------------------------
// result blocks (Protocol 2 in general form): which output tiles are computed
// ---------------------------------------------------------------------------
// Rows and columns are listed component by component, so a tile touches a result block exactly
// when the component ranges of its rows and of its columns overlap.  One workgroup writes the
// numbers of those tiles, in the order the GEMM enumerates tiles (tile = tn * tiles_m + tm),
// to list[1 ..] and their count to list[0]; the GEMM then deals out work over that list only.
// For tall operands two shapes are listed (128 x 64 and the narrow tile) and the choice between them
// is made here, on the device, from the area each would compute: both GEMM kernels are launched
// and the one that was not chosen returns at once, so the host never waits for the counts.
__device__ int list_tiles(const GemmParams& p, int BM, int BN, int* list) {
    __shared__ int wave_tot[GT / 64];
    const int nblk = n_blocks(p);
    const int m_eff = n_rows(p), n_eff = nblk * p.bs;
    const int tiles_m = (m_eff + BM - 1) / BM, tiles_n = (n_eff + BN - 1) / BN;
    const int tiles = tiles_m * tiles_n;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int base = 0;
    for (int t0 = 0; t0 < tiles; t0 += GT) {
        const int tile = t0 + threadIdx.x;
        bool on = false;
        if (tile < tiles) {
            const int tm = tile % tiles_m, tn = tile / tiles_m;
            const int r_hi = (tm + 1) * BM < m_eff ? (tm + 1) * BM - 1 : m_eff - 1;
            const int c_hi = (tn + 1) * BN < n_eff ? (tn + 1) * BN - 1 : n_eff - 1;
            const int rc0 = p.row_comp[tm * BM], rc1 = p.row_comp[r_hi];
            const int cc0 = p.blk_comp[tn * BN / p.bs], cc1 = p.blk_comp[c_hi / p.bs];
            on = !(rc1 < cc0 || cc1 < rc0);
        }
        const unsigned long long bal = __ballot(on);
        if (lane == 0) wave_tot[wave] = __builtin_popcountll(bal);
        __syncthreads();
        int pos = base + __builtin_popcountll(bal & ((1ull << lane) - 1));
#pragma unroll
        for (int w = 0; w < GT / 64; ++w) {
            const int v = wave_tot[w];
            if (w < wave) pos += v;
            base += v;
        }
        if (on) list[1 + pos] = tile;
        __syncthreads();
    }
    if (threadIdx.x == 0) list[0] = base;
    return base;
}

// One shape, or (list_b) two of them, 128 x 64 in list and the narrow tile BM x BN in list_b.
__global__ __launch_bounds__(GT) void tile_list_kernel(GemmParams p, int BM, int BN, int* list, int* list_b, int* sel,
                                                       int percent) {
    if (!list_b) {
        (void)list_tiles(p, BM, BN, list);
        return;
    }
    const long a = list_tiles(p, 128, 64, list), b = list_tiles(p, BM, BN, list_b);
    // the second shape runs when it computes less than this share of the other's area
    // (smaller tiles follow the block structure more closely but reuse operands less)
    if (threadIdx.x == 0) *sel = 100l * b * BM * BN < (long)percent * a * 128 * 64 ? 1 : 0;
}

// ---------------------------------------------------------------------------
// per-token row sets (Protocol 3 in general form): which contraction steps a row tile computes
// ---------------------------------------------------------------------------
// Protocol 3 multiplies column j of X only on its row set R_j.  At tile granularity: a row tile
// needs contraction step s (32 consecutive kept neurons) only if one of its tokens uses one of
// the blocks the step touches; for all other steps the tile's activation digits are zero.  One
// workgroup per row tile lists its steps in ascending order (grid.x = row tiles), and the last of them to
// finish turns the counts into offsets (step_off[t] = step_cnt[0] + ... + step_cnt[t - 1] for
// t = 0 .. tiles).  The GEMM then deals out work over the listed steps only.
//
// What bounds it is the chain of dependent loads (a block's id, then the tokens' flags), so the flags of
// every (block, group of four tokens) are requested by a thread of its own: first "does some token of the
// tile use block t" for the blocks of a chunk of steps (a byte each in LDS), then the steps from those.
// 256 tokens x 344 blocks, 64-row tiles: 10 us (38 with one thread per step, token after token, and the
// offsets in a launch of their own).
constexpr int SLT = 1024;              // threads per workgroup
constexpr int SL_STEPS = 1024;         // steps per chunk, one per thread
constexpr int SL_ROWS = 4;             // tokens per thread and block
__global__ __launch_bounds__(SLT) void step_list_kernel(GemmParams p, int BM) {
    __shared__ unsigned char used[SL_STEPS * KSTEP + 1];       // (blocks of one neuron: as many as words, and one cut by the start)
    __shared__ int wave_tot[SLT / 64];
    const int nblk = n_blocks(p);
    const int m_eff = n_rows(p);
    const int kc = nblk * p.bs;
    const int KS = (kc + KSTEP - 1) / KSTEP;
    const int tm = blockIdx.x;
    const int r0 = tm * BM, r1 = (tm + 1) * BM < m_eff ? (tm + 1) * BM : m_eff;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int* list = p.step_list + (size_t)tm * p.ks_cap;
    int base = 0;
    const int groups = r0 < r1 ? (r1 - r0 + SL_ROWS - 1) / SL_ROWS : 0;
    for (int s0 = 0; s0 < KS; s0 += SL_STEPS) {
        const int s1 = s0 + SL_STEPS < KS ? s0 + SL_STEPS : KS;
        const int t0 = s0 * KSTEP / p.bs;
        int t1 = (s1 * KSTEP - 1) / p.bs;                      // blocks t0 .. t1 lie in the chunk
        t1 = t1 < nblk - 1 ? t1 : nblk - 1;
        const int nt = t1 - t0 + 1;
        for (int t = threadIdx.x; t < nt; t += SLT) used[t] = 0;
        __syncthreads();
        for (int i = threadIdx.x; i < nt * groups; i += SLT) {
            const int t = i % nt, r = r0 + i / nt * SL_ROWS;
            const long b = p.blk_idx[t0 + t];
            if (b < 0 || b >= p.tmask_nb) continue;            // (see token_uses)
            const unsigned char* flag = p.tmask + (long)r * p.tmask_nb + b;
            unsigned any = 0;
#pragma unroll
            for (int j = 0; j < SL_ROWS; ++j) any |= flag[(r + j < r1 ? j : 0) * p.tmask_nb];
            if (any) used[t] = 1;
        }
        __syncthreads();
        const int st = s0 + threadIdx.x;
        bool on = false;
        if (st < s1) {
            int u1 = (st * KSTEP + KSTEP - 1) / p.bs;
            u1 = u1 < t1 ? u1 : t1;
            for (int t = st * KSTEP / p.bs; t <= u1; ++t) on = on || used[t - t0];
        }
        const unsigned long long bal = __ballot(on);
        if (lane == 0) wave_tot[wave] = __builtin_popcountll(bal);
        __syncthreads();
        int pos = base + __builtin_popcountll(bal & ((1ull << lane) - 1));
#pragma unroll
        for (int w = 0; w < SLT / 64; ++w) {
            const int v = wave_tot[w];
            if (w < wave) pos += v;
            base += v;
        }
        if (on) list[pos] = st;
        __syncthreads();
    }
    // p.tile_list[0] counts the workgroups that are done (set to zero by the packing kernel); the counts pass
    // between the XCDs as device-scope atomics
    __shared__ int last;
    if (threadIdx.x == 0) {
        __hip_atomic_store(p.step_cnt + tm, base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = __hip_atomic_fetch_add(p.tile_list, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    const int tiles = (m_eff + BM - 1) / BM;
    int off = 0;
    for (int t0 = 0; t0 < tiles; t0 += SLT) {
        const int t = t0 + threadIdx.x;
        const int v = t < tiles ? __hip_atomic_load(p.step_cnt + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        int inc = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(inc, d, 64);
            if (lane >= d) inc += o;
        }
        if (lane == 63) wave_tot[wave] = inc;
        __syncthreads();
        int pre = off + inc - v;
#pragma unroll
        for (int w = 0; w < SLT / 64; ++w) {
            const int x = wave_tot[w];
            if (w < wave) pre += x;
            off += x;
        }
        if (t < tiles) p.step_off[t] = pre;
        __syncthreads();
    }
    if (threadIdx.x == 0) p.step_off[tiles] = off;
}

inline int round_up(int64_t v, int64_t to) { return (int)(((v + to - 1) / to) * to); }

// digit planes of [E | A'] (the few-row path keeps its k-major copy there instead)
size_t planes_bytes(int64_t m, int64_t kc_cap) {
    const size_t mpad = (size_t)round_up(m, 128);
    const size_t ks_cap = (size_t)((kc_cap + KSTEP - 1) / KSTEP);
    const size_t bytes = mpad * 2 * ks_cap * 256;
    return bytes ? bytes : 256;
}

// step lists of Protocol 3 with per-token row sets: per row tile of the smallest tile height (32)
// a count, an offset and up to ks_cap listed steps
size_t step_ws_bytes(int64_t m, int64_t kc_cap) {
    const size_t tiles = (size_t)((m + 31) / 32);
    const size_t ks_cap = (size_t)((kc_cap + KSTEP - 1) / KSTEP);
    return ((tiles * (ks_cap + 2) + 1) * sizeof(int) + 255) & ~(size_t)255;
}

// followed by the list of output tiles that touch a result block (general form of Protocol 2):
// a selector, then twice (two tile shapes) one count plus one entry per tile of the smallest
// tile shape, 64 x 64
size_t gemm_ws_bytes(int64_t m, int64_t kc_cap, int64_t n_cap) {
    if (m < 1 || kc_cap < 0 || n_cap < 0 || m > COMET_ROWS_MAX || kc_cap > COMET_DIM_MAX || n_cap > COMET_DIM_MAX)
        return 0;
    const size_t tiles = (size_t)((m + 63) / 64) * (size_t)((n_cap + 63) / 64);
    return planes_bytes(m, kc_cap) + (((2 * (tiles + 1) + 1) * sizeof(int) + 255) & ~(size_t)255) +
           step_ws_bytes(m, kc_cap);
}

// the parts of the workspace and the derived sizes
void place_in_workspace(GemmParams& p, void* ws) {
    p.xp = static_cast<unsigned char*>(ws);
    p.tile_list = reinterpret_cast<int*>(p.xp + planes_bytes(p.m, p.kc_cap));
    p.mpad = round_up(p.m, 128);
    p.ks_cap = (p.kc_cap + KSTEP - 1) / KSTEP;
    p.xstep[0] = 0;
    p.xstep[1] = p.ks_cap;
    p.bs_shift = -1;
    for (int sh = 0; sh < 30; ++sh)
        if (p.bs == (1 << sh)) p.bs_shift = sh;
}

// Columns of the 64-row tile on weight planes: 64, or 128 for large products.  A pair of contraction steps takes a
// workgroup 1.1 us on 64 x 64 and 2.2 us on 64 x 128, which reads half of its operands from LDS less often.  What
// decides is how many 64 x 64 pairs there are per compute unit: below 32 of them the finer pieces fill the chip
// better (128 x 768 x 320 19 -> 16 us, 64 x 1664 x 4096 45 -> 38, 192 x 2560 x 640 40 -> 33), from there on the wider
// tile is ahead (320 x 4096 x 960 101 -> 83, 448 x 4096 x 2560 342 -> 279). Exceptions, as measured: a single row
// tile reads every weight unit once and stays with 64 (64 x 11008 x 1664 97 -> 94); so does a multiple of 64 tiles,
// whose workgroup shares line up with the tiles, up to 256 pairs (192 x 1664 x 4096 96 -> 82, 320 x 1664 x 4096 139
// -> 133).  With step lists the row tiles do not sweep side by side: 128 columns from 32 pairs on (512 tokens x 344
// blocks of 32, n = 1024 334 -> 278), with a single row tile from 24 (33 x 344 of 16, n = 2560 85 -> 75). Result
// blocks leave most tiles out, and the finer tile follows them more closely: 128 columns from 144 pairs, counted over
// all tiles, and 2048 contraction words on only (129 x 400 of 16, k = 4096 209 -> 179, 129 x 563 of 16, k = 4199 572
// -> 333; but 512 x 344 of 32, k = 1024 155 -> 119 and 209 x 100 of 16, k = 4096 71 -> 57 with 64).
int planes_narrow_bn(const comet_ctx* ctx, const GemmParams& p) {
    const long tiles = (long)((p.m + 63) / 64) * ((p.n_cap + 63) / 64);
    const long pairs = tiles * ((p.kc_cap + KSTEP - 1) / KSTEP) / (ctx->num_cu > 0 ? ctx->num_cu : 1);
    if (p.row_comp) return pairs >= 144 && p.kc_cap >= 2048 ? 128 : 64;
    if (p.tmask) return pairs >= (p.m <= 64 ? 24 : 32) ? 128 : 64;
    if (p.m <= 64 || pairs < 32 || (tiles % 64 == 0 && pairs < 256)) return 64;
    return 128;
}

// Are weight words read past the caches?  Words well beyond the 256 MB memory-side cache only push out what is still
// needed there; smaller ones may still lie in it from the call that wrote them.  The line lies at 320 MB of B_i and F
// together: 260 MB took 76 -> 72 us with ordinary loads (k = 4096, 16 rows), 400 MB 107 -> 98 us without (16 rows),
// 115 -> 103 us (32), 147 -> 137 us (64). Several row tiles read the same words and count on the caches between them:
// 722 MB take 583 -> 601 us past the caches (150 rows), 605 -> 618 (192), 1415 -> 1433 (512), 2751 -> 2840 (1024), one
// request of 256 tokens with a step list 697 -> 745. Neuron-major words and blocks that are gathered row by row have
// ordinary loads throughout.
bool words_past_caches(const GemmParams& p) { return p.m <= 64 && 2ll * 8 * p.kc_cap * p.n_cap > (320ll << 20); }

// ---------------------------------------------------------------------------
// which kernel
// ---------------------------------------------------------------------------
// What the few-row kernel deals out: (32-row tile, 128 columns, contraction step) units of all members.
long few_units(const GemmParams& p, int members) {
    return (long)((p.m + 31) / 32) * ((p.n_cap + 127) / 128) * 2 * ((p.kc_cap + KSTEP - 1) / KSTEP) * members;
}

// COMET_TUNE_SKINNY = 1: up to 32 rows go to the tiles
bool rows_to_tiles(const comet_ctx* ctx, const GemmParams& p) { return ctx->skinny_mode == 1 && p.m <= COMET_FEWROW_MAX_ROWS; }

// Does a product take the kernel whose wavefronts stream by themselves (ring_fewrow.hip)?  Up to 32 rows on planes
// always; on words up to 16 units per compute unit (13: 9 and 32 rows, k = 4096, n = 1664 33 and 41 us with the
// 32 x 256 tile, 31 and 36 here; 32 rows, 819 gathered row by row x 1001 46 against 21; but 27: 9 rows, 5120 x 2752 49
// against 53); of more rows the smallest products, up to half a unit (128 x 256 x 256 13.2 against 12.7, 64 x 64 x 64 11.3
// against 8.8; but one unit: 256 x 256 x 256 13.1 against 15.1).
bool takes_few_rows(const comet_ctx* ctx, const GemmParams& p) {
    if (p.row_comp || p.tmask || ctx->gemm_tile >= 2 || ctx->gemm_chunk > 0 || rows_to_tiles(ctx, p)) return false;
    if (p.w_planes && p.m <= COMET_FEWROW_MAX_ROWS) return true;
    return 2 * few_units(p, 1) <= (p.m <= COMET_FEWROW_MAX_ROWS ? 32l : 1l) * ctx->num_cu;
}

// A group on planes there: up to 32 rows always, because the members then share one packing and one share launch; more rows up to
// twenty units per compute unit (two products of 128 x 768 x 320 26.4 -> 21.7 us, four of 256 x 320 x 768 47 -> 36, two of
// 65 x 640 x 2560 44.0 -> 41.7 at 19 units; at 24 units four of 65 x 640 x 1664 50 -> 55).
bool group_takes_few_rows(const comet_ctx* ctx, const GemmParams& p, int members) {
    if (members < 2 || !p.w_planes || p.n_cap < 1 || p.kc_cap < 1 || ctx->group_mode == 2 || ctx->gemm_tile >= 2 ||
        ctx->gemm_chunk > 0 || rows_to_tiles(ctx, p))
        return false;
    if (p.m <= COMET_FEWROW_MAX_ROWS) return true;
    // (the grouped launch of tiles starts at 65 rows)
    if (ctx->group_mode != 0) return p.m <= 64;
    return few_units(p, members) <= 20l * ctx->num_cu;
}

// The smallest products take one launch: up to 100 contraction words and a 32 x 32 tile per compute unit, 2.5 us less of the
// host's time.  On the GPU it is well ahead up to 64 words (few-row kernel with its packing / one launch, words: 64 x 64
// outputs 8.3 / 7.9 us, 256 x 256 9.3 / 8.1, 33 x 3072 9.4 / 8.2) and about even from there to 100, ahead with many tiles,
// behind with few (64 x 64 outputs, 96 words 8.7 / 9.3, 100 words 8.9 / 8.9, 104 words 8.9 / 9.0; 256 x 256 10.3 / 9.8,
// 11.2 / 9.4, 11.3 / 9.5); beyond, up to the 128 words that the kernel holds, it falls behind (112 words 8.9 / 10.3, 128 words
// 8.3 / 10.2; 256 x 256 11.5 / 10.5, 10.9 / 10.8): all eight wavefronts fetch words of 32 rows one by one by then.
// More tiles than units: 128 x 64 x 3072 (384 tiles) 14.6 / 15.7.
bool takes_direct(const comet_ctx* ctx, const GemmParams& p) {
    if (p.row_comp || p.tmask || ctx->gemm_tile >= 2 || ctx->gemm_chunk > 0 || ctx->gemm_grid > 0 || rows_to_tiles(ctx, p)) return false;
    const long tiles = (long)((p.m + 31) / 32) * ((p.n_cap + 31) / 32);
    return p.kc_cap >= 1 && p.kc_cap <= 100 && tiles <= ctx->num_cu;
}

// Products on words of more than 32 rows: the 64 x 64 tile whose four wavefronts load, split, stage and multiply in one
// instruction stream, two workgroups per compute unit (ring_tile.h), or the one with four feeding and four multiplying
// wavefronts (ring_words.h)?  The second is ahead once its workgroups have a few pairs of steps each (512 x 3000 x 2560 254
// -> 227 us, 96 x 384 x 2048 25 -> 18), the first
//   * up to one pair of steps per compute unit, where what counts is how soon the first step is multiplied: 64 x 768 x 320
//     12.4 against 13.4 us, 40 x 160 x 1024 10.9 against 12.4, 129 x 384 x 320 13.2 against 14.7 (but from there on
//     64 x 1024 x 768, 1.5 pairs, 18.6 against 15.9);
//   * where the second has to share the units out evenly, without teams of row tiles (three, five, six of them ..: see
//     UnitWalk), or reads neuron-major weights in such shares, and twice as many workgroups give slices that are hardly longer:
//     400 x 2560 x 640 60 against 67 us, 150 x 4096 x 1664 92 against 101, neuron-major 150 x 4096 x 960 59 against 71.
//     Not where the slices are a tenth longer (400 x 2560 x 1024 91 against 82) or a tile has one to four of them and more
//     than eight pairs each (320 x 1664 x 2048 82 against 77).
// Row sets: up to 64 rows and one pair per unit (33 rows, 60 blocks of 16, n = 96 18.9 against 20.7; more rows are a draw),
// and with a ragged last row tile, which lists fewer steps than the others and so reads the weights at times of its own,
// where the lists are long and the columns few (77 rows, 800 blocks of 16, n = 500 86 against 98, 130 rows 105 against 114,
// 400 rows 256 against 266; but n = 1024 100 rows 110 against 102, 40 blocks of 32 28 against 24).
// Result blocks: up to 64 rows and sixteen pairs per unit (33 rows, 344 blocks of 32, k = 512 36 against 47; 64 rows, 100
// blocks, k = 1024 31 against 34; but 344 blocks, k = 1024, 21 pairs, 71 against 69).
// Rows looked up one by one always take the second (256 rows x 819 x 1001 39 against 50).
bool takes_staged_tile(const comet_ctx* ctx, const GemmParams& p) {
    if (ctx->gemm_tile >= 2) return ctx->gemm_tile == 3;
    if (p.w_planes || ctx->gemm_chunk > 0 || (p.kind == KIND_SIMM && p.b_full && p.bs_shift < 3)) return false;
    const long cu = (ctx->num_cu / 8) * 8, tiles_m = (p.m + 63) / 64, tiles = tiles_m * ((p.n_cap + 63) / 64);
    if (p.row_comp) return p.m <= 64 && tiles * p.ks_cap <= 16 * cu;
    if (p.tmask)
        return (p.m <= 64 && tiles * p.ks_cap <= cu) || (p.m > 64 && p.m % 64 != 0 && p.n_cap <= 512 && p.kc_cap >= 8192);
    if (tiles * p.ks_cap <= cu) return true;
    // the longest run of a workgroup: in pairs when the second kernel shares the units out evenly, in steps when the first
    // cuts a tile into slices (see UnitWalk)
    const long even = (tiles * p.ks_cap + cu - 1) / cu;
    if (tiles <= cu) {
        const long slices = cu / tiles < p.ks_cap ? cu / tiles : p.ks_cap;
        if ((p.ks_cap + slices - 1) / slices <= tiles * p.ks_cap / cu + UnitWalk<false>::SPLIT_COST) return false;
    }
    if (tiles > 2 * cu) return false;
    const long slices = 2 * cu / tiles < 2l * p.ks_cap ? 2 * cu / tiles : 2l * p.ks_cap;
    const long sliced = (2l * p.ks_cap + slices - 1) / slices;
    if (sliced > tiles * p.ks_cap / cu + UnitWalk<false, 1>::SPLIT_COST) return false;
    return p.w_tr || (cu % tiles_m != 0 && 10 * sliced <= 11 * even + 10 && (slices >= 5 || even <= 8));
}

int run_share(comet_ctx* ctx, const char* what, GemmParams p, void* ws, size_t ws_bytes) {
    const size_t need = gemm_ws_bytes(p.m, p.kc_cap, p.n_cap);
    if (!ws || ws_bytes < need)
        return comet_fail(ctx, COMET_EWORKSPACE, "%s: workspace of %zu bytes required", what, need);
    if (reinterpret_cast<uintptr_t>(ws) & 255u)
        return comet_fail(ctx, COMET_EALIGN, "%s: workspace must be 256-byte aligned", what);
    comet_device_guard guard(ctx);
    if (!guard.ok) return comet_fail(ctx, COMET_EDEVICE, "%s: cannot select device", what);

    place_in_workspace(p, ws);

    if (p.n_cap == 0) return COMET_OK;
    if (p.F2 && (p.m > COMET_SKINNY_MAX_ROWS || ctx->skinny_mode == 1 || p.w_tr || p.w_planes || p.row_comp || p.tmask))
        return comet_fail(ctx, COMET_EINVAL, "%s: unopened weight shares are taken by the few-row kernel only "
                          "(m <= %d, row-major words)", what, COMET_SKINNY_MAX_ROWS);
    // (the few-row kernel reads the weights along the output columns: row-major words only)
    if (p.m <= COMET_SKINNY_MAX_ROWS && ctx->skinny_mode != 1 && !p.w_tr && !p.w_planes)
        return comet_launch_skinny(ctx, what, p);
    if (takes_direct(ctx, p)) return comet_launch_direct(ctx, what, p);
    // Tile shape and launch plan first: the packing kernel has to know whether the share kernel
    // will own its tiles (and then initialise Z itself).
    // columns of the 64- and 32-row tiles
    const int narrow_bn = p.w_planes ? planes_narrow_bn(ctx, p) : 64, flat_bn = p.w_planes ? 128 : 256;
    const bool staged = !p.w_planes && takes_staged_tile(ctx, p);
    auto plan = [&](int bm) {
        if (p.w_planes) plan_gemm(ctx, p, bm, bm == 128 ? 64 : bm == 64 ? narrow_bn : flat_bn, bm == 128);
        else if (bm == 32) plan_gemm(ctx, p, 32, flat_bn, false, 1);
        else if (staged) plan_gemm(ctx, p, 64, 64, false, 1, Tile<2, 2, 1, 1>::WG_PER_CU);
        else plan_gemm(ctx, p, 64, 64, true);
    };
    auto launch = [&](int bm) {
        plan(bm);
        if (!p.w_planes && bm == 32) return launch_gemm<1, 4, 1, 2>(ctx, what, p);
        if (!p.w_planes) return staged ? launch_gemm<2, 2, 1, 1>(ctx, what, p) : launch_words(ctx, what, p);
        if (bm == 128) return launch_planes<2, 2, 4, 2>(ctx, what, p);
        if (bm == 64 && narrow_bn == 64) return launch_planes<2, 2, 2, 2>(ctx, what, p);
        if (bm == 64) return launch_planes<1, 4, 4, 2>(ctx, what, p);
        return launch_planes<1, 4, 2, 2>(ctx, what, p);
    };
    // rows per workgroup tile: 128, 64 or 32 (words: 64 or 32)
    int bm = 128;
    const long big_tiles = (long)((p.m + 127) / 128) * ((p.n_cap + 63) / 64);
    if (ctx->gemm_tile >= 2) bm = 64;
    else if (p.m <= 32) bm = 32;
    else if (p.m <= 64 || !p.w_planes) bm = 64;
    // a small product (a handful of 128 x 64 tiles) is bound by the fixed cost per workgroup:
    // 64 rows double the number of independent tiles
    else if (!p.row_comp && big_tiles * 8 <= ctx->num_cu) bm = 64;
    // a ragged last row tile: 64-row tiles when they pad the rows by clearly less (the smaller
    // tile is about 5 % slower per product)
    else if (!p.row_comp && (long)round_up(p.m, 64) * 110 < (long)round_up(p.m, 128) * 100) bm = 64;
    // per-token row sets: 64-row tiles follow the row sets more closely
    else if (p.tmask) bm = 64;
    plan(bm);
    p.w_nt = words_past_caches(p);
    // a decoding batch on weight planes, or a small product: the kernel that streams wavefront by wavefront
    const bool fewrow = takes_few_rows(ctx, p);
    if (fewrow) {
        p.own_try = 0;                                         // Z := C comes from the packing kernel
        if (p.m <= 32) p.mpad = 32;                            // one row tile: a digit group is 512 bytes
    }

    // digit planes of [E | A'] and Z := C, one launch
    {
        unsigned gx = (unsigned)((p.ks_cap * 2 + 3) / 4);
        if (gx < 1) gx = 1;
        // the Z := C slab shares the launch: give it enough workgroups for about four 16-byte
        // accesses per thread (the packing slabs return at once from the extra ones)
        const int slabs = (p.mpad + 63) / 64;
        const long zgx = ((long)p.m * p.n_cap / (2l * 4 * GT) + slabs - 1) / slabs;
        if (zgx > gx) gx = (unsigned)(zgx > 4096 ? 4096 : zgx);
        hipLaunchKernelGGL(p.tmask ? xpack_kernel<true> : xpack_kernel<false>, dim3(gx, (unsigned)slabs, 3), dim3(GT), 0, ctx->stream, p);
        COMET_LAUNCH_CHECK(ctx, what);
    }
    if (p.ks_cap == 0) return COMET_OK;
    if (fewrow) return comet_launch_fewrow(ctx, what, p);
    if (p.row_comp) {
        // result blocks: list the tiles that are computed (see tile_list_kernel)
        int* sel = p.tile_list;
        int* list_a = sel + 1;
        int* list_b = list_a + 1 + (size_t)((p.m + 63) / 64) * (size_t)((p.n_cap + 63) / 64);
        p.tile_list = list_a;
        if (bm != 128) {
            hipLaunchKernelGGL(tile_list_kernel, dim3(1), dim3(GT), 0, ctx->stream, p, bm,
                               bm == 64 ? narrow_bn : flat_bn, list_a, (int*)nullptr, (int*)nullptr, 0);
            COMET_LAUNCH_CHECK(ctx, what);
            return launch(bm);
        }
        // 80 % of the area; less than three quarters, what 129 to 192 rows of one component come to, for 64 x 64 on
        // planes and long contractions (129 rows: k = 4199, 300 blocks of 16 479 -> 317 us on 128 x 64; k = 1024, 344 of 32
        // 131 against 160)
        const int percent = narrow_bn == 64 && p.kc_cap >= 2048 ? 75 : 80;
        hipLaunchKernelGGL(tile_list_kernel, dim3(1), dim3(GT), 0, ctx->stream, p, 64, narrow_bn, list_a, list_b, sel,
                           percent);
        COMET_LAUNCH_CHECK(ctx, what);
        p.tile_sel = sel;
        p.tile_sel_want = 0;
        int rc = launch(128);
        if (rc) return rc;
        p.tile_list = list_b;
        p.tile_sel_want = 1;
        return launch(64);
    }
    if (p.tmask) {
        // list, per row tile, the contraction steps some token of the tile takes part in
        const size_t tiles64 = (size_t)((p.m + 63) / 64) * (size_t)((p.n_cap + 63) / 64);
        const size_t tl_bytes = ((2 * (tiles64 + 1) + 1) * sizeof(int) + 255) & ~(size_t)255;
        const size_t t32 = (size_t)((p.m + 31) / 32);
        int* base = reinterpret_cast<int*>(p.xp + planes_bytes(p.m, p.kc_cap) + tl_bytes);
        p.step_cnt = base;
        p.step_off = base + t32;
        p.step_list = base + 2 * t32 + 1;
        hipLaunchKernelGGL(step_list_kernel, dim3((unsigned)((p.m + bm - 1) / bm)), dim3(SLT), 0, ctx->stream, p, bm);
        COMET_LAUNCH_CHECK(ctx, what);
    }
    return launch(bm);
}

// Several products of one shape, one index list and one operand format.  When they suit the
// grouped kernels (weight planes; few rows or small, or more than 64 rows) they run as one
// packing launch and one share launch over the union of their work units; otherwise one by one.
int run_share_group(comet_ctx* ctx, const char* what, GemmParams* ps, int n, void* ws, size_t ws_bytes) {
    const size_t each = gemm_ws_bytes(ps[0].m, ps[0].kc_cap, ps[0].n_cap);
    if (!ws || each == 0 || ws_bytes / (size_t)n < each)
        return comet_fail(ctx, COMET_EWORKSPACE, "%s: workspace of %zu bytes required", what, each * (size_t)n);
    if (reinterpret_cast<uintptr_t>(ws) & 255u)
        return comet_fail(ctx, COMET_EALIGN, "%s: workspace must be 256-byte aligned", what);
    unsigned char* base = static_cast<unsigned char*>(ws);
    const GemmParams& p0 = ps[0];
    // One launch for all members pays up to 128 contraction steps per workgroup and member.  Short members
    // gain most, because what they cost alone is launches, pipeline fill and write-out: two products of
    // 128 x 768 x 320 39 -> 28 us, four of 65 x 256 x 256 66 -> 22 us, two of 256 x 4096 x 960 142 -> 122 us.
    // Beyond that the fixed cost is amortised already and one long launch only runs at a lower
    // sustained clock than the same work in pieces.
    using T = PlaneTile<2, 2, 4, 2>;
    long grid = (ctx->num_cu / 8) * 8;
    if (grid < 8) grid = 8;
    if (ctx->gemm_grid > 0) grid = ctx->gemm_grid;
    const long tiles = (long)((p0.m + T::BM - 1) / T::BM) * ((p0.n_cap + T::BN - 1) / T::BN);
    const long steps_each = tiles * 2 * ((p0.kc_cap + KSTEP - 1) / KSTEP) / grid;
    const bool few = group_takes_few_rows(ctx, p0, n);
    const bool grouped = few || (n > 1 && p0.w_planes && p0.m > 64 && p0.n_cap > 0 && ctx->gemm_tile < 2 &&
                                 (ctx->group_mode == 1 || ctx->group_mode == 3 ||
                                  (ctx->group_mode == 0 && steps_each <= 128)));
    if (!grouped) {
        for (int j = 0; j < n; ++j) {
            const int rc = run_share(ctx, what, ps[j], base + (size_t)j * each, each);
            if (rc) return rc;
        }
        return COMET_OK;
    }
    comet_device_guard guard(ctx);
    if (!guard.ok) return comet_fail(ctx, COMET_EDEVICE, "%s: cannot select device", what);

    GemmGroup grp = {};
    grp.n = n;
    // The members' activation planes share one buffer, half by half, so that the planes of an E that several
    // members name (both simulated parties of a product) are packed once (LLaMA-7B layer of 256 tokens, six
    // products: 831 -> 826 us).
    int halves = 0;
    for (int j = 0; j < n; ++j) {
        GemmParams& p = grp.p[j];
        p = ps[j];
        place_in_workspace(p, base);
        int same = 0;
        while (same < j && ps[same].E != p.E) ++same;
        p.x_shared = same < j;
        p.xstep[0] = p.x_shared ? grp.p[same].xstep[0] : halves++ * p.ks_cap;
        p.xstep[1] = halves++ * p.ks_cap;
        // (units tile by tile, all of a tile's contraction in a row: a workgroup's share of the whole
        // sequence then covers few tiles, and whole ones when the grid divides their number)
        p.grid = (int)grid;
        p.tile_bm = T::BM;
        p.tile_bn = T::BN;
        p.group_n = n;
        p.own_try = (tiles * n % grid == 0 && !few) ? 1 : 0;          // (few: Z := C comes from the packing kernel)
        if (few && p.m <= 32) p.mpad = 32;
        p.team = ctx->group_mode != 3;      // (3: one launch without teams, for comparison)
    }
    {
        const GemmParams& p = grp.p[0];
        unsigned gx = (unsigned)((p.ks_cap * 2 + 3) / 4);
        if (gx < 1) gx = 1;
        const int slabs = (p.mpad + 63) / 64;
        const long zgx = ((long)p.m * p.n_cap / (2l * 4 * GT) + slabs - 1) / slabs;
        if (zgx > gx) gx = (unsigned)(zgx > 4096 ? 4096 : zgx);
        hipLaunchKernelGGL(xpack_group_kernel, dim3(gx, (unsigned)slabs, 3u * (unsigned)n), dim3(GT), 0, ctx->stream, grp);
        COMET_LAUNCH_CHECK(ctx, what);
    }
    if (few) return comet_launch_fewrow_group(ctx, what, grp);
    return launch_planes_group<2, 2, 4, 2>(ctx, what, grp);
}

int check_common(comet_ctx* ctx, const char* what, int party, int64_t m, int bs, int n_blk_cap,
                 int flags, const void* const* ptrs, int n_ptrs, const int32_t* blk_idx) {
    if (party != 0 && party != 1) return comet_fail(ctx, COMET_EINVAL, "%s: party must be 0 or 1", what);
    if (m < 1 || bs < 1 || n_blk_cap < 0) return comet_fail(ctx, COMET_EINVAL, "%s: bad size", what);
    if (flags & ~(COMET_FULL_A | COMET_FULL_B | COMET_WEIGHTS_NEURON_MAJOR | COMET_WEIGHT_PLANES))
        return comet_fail(ctx, COMET_EINVAL, "%s: unknown flag", what);
    if ((flags & COMET_WEIGHT_PLANES) && (flags & COMET_WEIGHTS_NEURON_MAJOR))
        return comet_fail(ctx, COMET_EINVAL, "%s: weight planes have a layout of their own", what);
    for (int i = 0; i < n_ptrs; ++i) {
        if (!ptrs[i]) return comet_fail(ctx, COMET_EINVAL, "%s: null pointer (operand %d)", what, i);
        if (!comet_aligned16(ptrs[i]))
            return comet_fail(ctx, COMET_EALIGN, "%s: operand %d is not 16-byte aligned", what, i);
    }
    if (!blk_idx && (flags & (COMET_FULL_A | COMET_FULL_B)))
        return comet_fail(ctx, COMET_EINVAL, "%s: blk_idx required for full-size operands", what);
    // rows: the packing kernel walks 64-row slabs of the padded row count on grid.y (< 65536)
    if (m > COMET_ROWS_MAX || (int64_t)n_blk_cap * bs > COMET_DIM_MAX)
        return comet_fail(ctx, COMET_ECAP, "%s: dimension beyond 2^24 (m beyond 2^22 - 128)", what);
    return COMET_OK;
}

int somm_params(comet_ctx* ctx, const char* what, GemmParams& p, int party, int64_t m, int64_t k,
                int64_t n_full, int bs, const int32_t* blk_idx, const int32_t* n_blk_dev, int n_blk_cap,
                int flags, const uint64_t* E, const uint64_t* F, const uint64_t* A_i,
                const uint64_t* B_i, const uint64_t* C_i, uint64_t* Z_i) {
    const void* ptrs[] = {E, F, A_i, B_i, C_i, Z_i};
    int rc = check_common(ctx, what, party, m, bs, n_blk_cap, flags, ptrs, 6, blk_idx);
    if (rc) return rc;
    if (k < 1 || n_full < 0) return comet_fail(ctx, COMET_EINVAL, "%s: bad size", what);
    if (flags & COMET_FULL_A) return comet_fail(ctx, COMET_EINVAL, "%s: A_i is never indexed in SOMM", what);
    if (k > COMET_DIM_MAX || n_full > COMET_DIM_MAX) return comet_fail(ctx, COMET_ECAP, "%s: dimension beyond 2^24", what);
    const int64_t ld = (int64_t)n_blk_cap * bs;
    if ((flags & COMET_FULL_B) && ld > n_full)
        return comet_fail(ctx, COMET_EINVAL, "%s: n_blk_cap * bs exceeds n_full", what);
    if (k * ((flags & COMET_FULL_B) ? n_full : ld) >= (1ll << 31) || k * ld >= (1ll << 31))
        return comet_fail(ctx, COMET_ECAP, "%s: a weight-side operand holds 2^31 words or more", what);
    p.kind = KIND_SOMM; p.party = party; p.m = (int)m; p.kc_cap = (int)k; p.n_cap = (int)ld;
    p.bs = bs; p.n_blk_cap = n_blk_cap; p.blk_idx = blk_idx; p.n_blk_dev = n_blk_dev;
    p.full_extent = (int)n_full;
    p.E = (const u64*)E; p.lde = k;
    p.A = (const u64*)A_i; p.lda = k; p.a_full = 0;
    p.B = (const u64*)B_i; p.b_full = (flags & COMET_FULL_B) ? 1 : 0; p.ldb = p.b_full ? n_full : ld;
    p.F = (const u64*)F; p.ldf = ld;
    if (flags & COMET_WEIGHTS_NEURON_MAJOR) {
        // B_i: n_full x k or ld x k, F: ld x k; the kernel reads pairs of contraction words
        if (k & 1) return comet_fail(ctx, COMET_EINVAL, "%s: neuron-major weights need an even k", what);
        p.w_tr = 1; p.ldb = k; p.ldf = k;
    }
    p.w_planes = (flags & COMET_WEIGHT_PLANES) ? 1 : 0;
    p.C = (const u64*)C_i; p.Z = (u64*)Z_i; p.ldz = ld;
    return COMET_OK;
}

int simm_params(comet_ctx* ctx, const char* what, GemmParams& p, int party, int64_t m, int64_t k_full,
                int64_t n, int bs, const int32_t* blk_idx, const int32_t* n_blk_dev, int n_blk_cap,
                int flags, const uint64_t* E, const uint64_t* F, const uint64_t* A_i,
                const uint64_t* B_i, const uint64_t* C_i, uint64_t* Z_i) {
    const void* ptrs[] = {E, F, A_i, B_i, C_i, Z_i};
    int rc = check_common(ctx, what, party, m, bs, n_blk_cap, flags, ptrs, 6, blk_idx);
    if (rc) return rc;
    if (n < 1 || k_full < 0) return comet_fail(ctx, COMET_EINVAL, "%s: bad size", what);
    if (flags & COMET_WEIGHTS_NEURON_MAJOR)
        return comet_fail(ctx, COMET_EINVAL, "%s: B_i and F of SIMM are neuron-major as they are (one row per neuron)", what);
    if (n > COMET_DIM_MAX || k_full > COMET_DIM_MAX) return comet_fail(ctx, COMET_ECAP, "%s: dimension beyond 2^24", what);
    const int64_t ld = (int64_t)n_blk_cap * bs;
    if ((flags & (COMET_FULL_A | COMET_FULL_B)) && ld > k_full)
        return comet_fail(ctx, COMET_EINVAL, "%s: n_blk_cap * bs exceeds k_full", what);
    if (((flags & COMET_FULL_B) ? k_full : ld) * n >= (1ll << 31))
        return comet_fail(ctx, COMET_ECAP, "%s: a weight-side operand holds 2^31 words or more", what);
    p.kind = KIND_SIMM; p.party = party; p.m = (int)m; p.kc_cap = (int)ld; p.n_cap = (int)n;
    p.bs = bs; p.n_blk_cap = n_blk_cap; p.blk_idx = blk_idx; p.n_blk_dev = n_blk_dev;
    p.full_extent = (int)k_full;
    p.E = (const u64*)E; p.lde = ld;
    p.A = (const u64*)A_i; p.a_full = (flags & COMET_FULL_A) ? 1 : 0; p.lda = p.a_full ? k_full : ld;
    p.B = (const u64*)B_i; p.b_full = (flags & COMET_FULL_B) ? 1 : 0; p.ldb = n;
    p.F = (const u64*)F; p.ldf = n;
    p.w_planes = (flags & COMET_WEIGHT_PLANES) ? 1 : 0;
    // planes of a full-size B_i are gathered in units of sixteen contraction rows
    if (p.w_planes && p.b_full && (bs % 16) != 0)
        return comet_fail(ctx, COMET_EINVAL, "%s: weight planes of a full-size B_i need bs to be a multiple of 16", what);
    p.C = (const u64*)C_i; p.Z = (u64*)Z_i; p.ldz = n;
    return COMET_OK;
}

}  // namespace

size_t comet_gemm_workspace_bytes(int64_t m, int64_t kc_cap, int64_t n_cap) {
    return gemm_ws_bytes(m, kc_cap, n_cap);
}

extern "C" {

int comet_somm_share(comet_ctx* ctx, int party, int64_t m, int64_t k, int64_t n_full, int bs,
                     const int32_t* blk_idx, const int32_t* n_blk_dev, int n_blk_cap, int flags,
                     const uint64_t* E, const uint64_t* F, const uint64_t* A_i,
                     const uint64_t* B_i, const uint64_t* C_i, uint64_t* Z_i, void* ws,
                     size_t ws_bytes) {
    const char* what = "comet_somm_share";
    COMET_CHECK_CTX(ctx);
    GemmParams p = {};
    const int rc = somm_params(ctx, what, p, party, m, k, n_full, bs, blk_idx, n_blk_dev, n_blk_cap, flags,
                               E, F, A_i, B_i, C_i, Z_i);
    if (rc) return rc;
    return run_share(ctx, what, p, ws, ws_bytes);
}

// second masked share of the weights for the *_unopened calls: same layout and checks as F
static int set_unopened(comet_ctx* ctx, const char* what, GemmParams& p, const uint64_t* G_1) {
    if (!G_1) return comet_fail(ctx, COMET_EINVAL, "%s: null pointer", what);
    if (!comet_aligned16(G_1)) return comet_fail(ctx, COMET_EALIGN, "%s: operands must be 16-byte aligned", what);
    p.F2 = (const u64*)G_1;
    return COMET_OK;
}

int comet_somm_share_unopened(comet_ctx* ctx, int party, int64_t m, int64_t k, int64_t n_full, int bs,
                              const int32_t* blk_idx, const int32_t* n_blk_dev, int n_blk_cap, int flags,
                              const uint64_t* E, const uint64_t* G_0, const uint64_t* G_1,
                              const uint64_t* A_i, const uint64_t* B_i, const uint64_t* C_i, uint64_t* Z_i,
                              void* ws, size_t ws_bytes) {
    const char* what = "comet_somm_share_unopened";
    COMET_CHECK_CTX(ctx);
    GemmParams p = {};
    int rc = somm_params(ctx, what, p, party, m, k, n_full, bs, blk_idx, n_blk_dev, n_blk_cap, flags,
                         E, G_0, A_i, B_i, C_i, Z_i);
    if (rc) return rc;
    if ((rc = set_unopened(ctx, what, p, G_1)) != COMET_OK) return rc;
    return run_share(ctx, what, p, ws, ws_bytes);
}

int comet_simm_share_unopened(comet_ctx* ctx, int party, int64_t m, int64_t k_full, int64_t n, int bs,
                              const int32_t* blk_idx, const int32_t* n_blk_dev, int n_blk_cap, int flags,
                              const uint64_t* E, const uint64_t* G_0, const uint64_t* G_1,
                              const uint64_t* A_i, const uint64_t* B_i, const uint64_t* C_i, uint64_t* Z_i,
                              void* ws, size_t ws_bytes) {
    const char* what = "comet_simm_share_unopened";
    COMET_CHECK_CTX(ctx);
    GemmParams p = {};
    int rc = simm_params(ctx, what, p, party, m, k_full, n, bs, blk_idx, n_blk_dev, n_blk_cap, flags,
                         E, G_0, A_i, B_i, C_i, Z_i);
    if (rc) return rc;
    if ((rc = set_unopened(ctx, what, p, G_1)) != COMET_OK) return rc;
    return run_share(ctx, what, p, ws, ws_bytes);
}

int comet_somm_share_static(comet_ctx* ctx, int party, int64_t m, int64_t k, int64_t n_full, int bs,
                            const int32_t* blk_idx, const int32_t* n_blk_dev, int n_blk_cap,
                            int flags, const uint64_t* E, const uint64_t* F, const uint64_t* A_i,
                            const uint64_t* B_i, const uint64_t* C_i, uint64_t* Z_i) {
    const char* what = "comet_somm_share_static";
    COMET_CHECK_CTX(ctx);
    GemmParams p = {};
    const int rc = somm_params(ctx, what, p, party, m, k, n_full, bs, blk_idx, n_blk_dev, n_blk_cap, flags,
                               E, F, A_i, B_i, C_i, Z_i);
    if (rc) return rc;
    const size_t need = gemm_ws_bytes(p.m, p.kc_cap, p.n_cap);
    if (need == 0 || need > STATIC_SCRATCH_BYTES)
        return comet_fail(ctx, COMET_ECAP,
                          "%s: needs %zu bytes of scratch, the static array holds %zu "
                          "(use comet_somm_share with a workspace)", what, need, STATIC_SCRATCH_BYTES);
    if (!ctx->static_ws)
        return comet_fail(ctx, COMET_EDEVICE, "%s: static scratch was not resolved on this device", what);
    // every part of the scratch a call reads it has written before, so nothing needs clearing
    return run_share(ctx, what, p, ctx->static_ws, STATIC_SCRATCH_BYTES);
}

int comet_somm_share_blocks(comet_ctx* ctx, int party, int64_t m_cap, int64_t k, int64_t n_full,
                            int bs, const int32_t* blk_idx, const int32_t* blk_comp,
                            const int32_t* n_blk_dev, int n_blk_cap, const int32_t* row_comp,
                            const int32_t* n_row_dev, int flags, const uint64_t* E,
                            const uint64_t* F, const uint64_t* A_i, const uint64_t* B_i,
                            const uint64_t* C_i, uint64_t* Z_i, void* ws, size_t ws_bytes) {
    const char* what = "comet_somm_share_blocks";
    COMET_CHECK_CTX(ctx);
    if (!blk_idx || !blk_comp || !row_comp)
        return comet_fail(ctx, COMET_EINVAL, "%s: blk_idx, blk_comp and row_comp are required", what);
    GemmParams p = {};
    const int rc = somm_params(ctx, what, p, party, m_cap, k, n_full, bs, blk_idx, n_blk_dev, n_blk_cap,
                               flags, E, F, A_i, B_i, C_i, Z_i);
    if (rc) return rc;
    p.row_comp = row_comp; p.blk_comp = blk_comp; p.n_row_dev = n_row_dev;
    return run_share(ctx, what, p, ws, ws_bytes);
}

int comet_simm_share(comet_ctx* ctx, int party, int64_t m, int64_t k_full, int64_t n, int bs,
                     const int32_t* blk_idx, const int32_t* n_blk_dev, int n_blk_cap, int flags,
                     const uint64_t* E, const uint64_t* F, const uint64_t* A_i,
                     const uint64_t* B_i, const uint64_t* C_i, uint64_t* Z_i, void* ws,
                     size_t ws_bytes) {
    const char* what = "comet_simm_share";
    COMET_CHECK_CTX(ctx);
    GemmParams p = {};
    const int rc = simm_params(ctx, what, p, party, m, k_full, n, bs, blk_idx, n_blk_dev, n_blk_cap, flags,
                               E, F, A_i, B_i, C_i, Z_i);
    if (rc) return rc;
    return run_share(ctx, what, p, ws, ws_bytes);
}

int comet_share_group(comet_ctx* ctx, int op, int n_members, const comet_share_operands* members,
                      int64_t m, int64_t k, int64_t n, int bs, const int32_t* blk_idx,
                      const int32_t* n_blk_dev, int n_blk_cap, int flags, void* ws, size_t ws_bytes) {
    const char* what = "comet_share_group";
    COMET_CHECK_CTX(ctx);
    if (op != COMET_OP_SOMM && op != COMET_OP_SIMM)
        return comet_fail(ctx, COMET_EINVAL, "%s: op must be COMET_OP_SOMM or COMET_OP_SIMM", what);
    if (!members || n_members < 1 || n_members > COMET_SHARE_GROUP_MAX)
        return comet_fail(ctx, COMET_EINVAL, "%s: 1 to %d members", what, (int)COMET_SHARE_GROUP_MAX);
    GemmParams ps[COMET_SHARE_GROUP_MAX] = {};
    for (int j = 0; j < n_members; ++j) {
        const comet_share_operands& o = members[j];
        const int rc = op == COMET_OP_SOMM
            ? somm_params(ctx, what, ps[j], o.party, m, k, n, bs, blk_idx, n_blk_dev, n_blk_cap, flags, o.E, o.F,
                          o.A_i, o.B_i, o.C_i, o.Z_i)
            : simm_params(ctx, what, ps[j], o.party, m, k, n, bs, blk_idx, n_blk_dev, n_blk_cap, flags, o.E, o.F,
                          o.A_i, o.B_i, o.C_i, o.Z_i);
        if (rc) return rc;
    }
    return run_share_group(ctx, what, ps, n_members, ws, ws_bytes);
}

int comet_simm_share_masked(comet_ctx* ctx, int party, int64_t m, int64_t k_full, int64_t n,
                            int bs, const int32_t* blk_idx, const int32_t* n_blk_dev,
                            int n_blk_cap, int flags, const uint8_t* token_mask, int64_t nb,
                            const uint64_t* E, const uint64_t* F, const uint64_t* A_i,
                            const uint64_t* B_i, const uint64_t* C_i, uint64_t* Z_i, void* ws,
                            size_t ws_bytes) {
    const char* what = "comet_simm_share_masked";
    COMET_CHECK_CTX(ctx);
    if (!token_mask || !blk_idx)
        return comet_fail(ctx, COMET_EINVAL, "%s: token_mask and blk_idx are required", what);
    if (nb < 1 || nb > COMET_DIM_MAX) return comet_fail(ctx, COMET_EINVAL, "%s: bad nb", what);
    GemmParams p = {};
    const int rc = simm_params(ctx, what, p, party, m, k_full, n, bs, blk_idx, n_blk_dev, n_blk_cap, flags,
                               E, F, A_i, B_i, C_i, Z_i);
    if (rc) return rc;
    p.tmask = token_mask; p.tmask_nb = nb;
    return run_share(ctx, what, p, ws, ws_bytes);
}

}  // extern "C"
