// What the int8 matrix-core kernels of the share calls have in common (ring_gemm.hip for the formulation; ring_words.h
// and ring_tile.h for weight words, ring_gemm_planes.h for weight planes, ring_fewrow.hip for few rows): the packed
// activation format, the walk over the work units, the launch plan.  The kernel variants are
// instantiated in translation units of their own, so that they compile side by side.
#pragma once

#include "common.h"
#include "digits.h"
#include "gemm_params.h"

#include <type_traits>
#include <utility>

namespace comet_gemm {

using ::GemmGroupKernel;
using ::GemmKernel;

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef u32 u32x4 __attribute__((ext_vector_type(4)));

constexpr int KSTEP = 32;       // ring words contracted per matrix instruction
constexpr int MAX_SEG = 256;    // contraction steps an int32 plane can absorb
constexpr int KPAIR = 2 * KSTEP; // ring words contracted per matrix instruction of 16 x 16 outputs
constexpr int GT = 256;         // threads of the packing and plane kernels' workgroups (4 wavefronts)

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

__device__ __forceinline__ v4i lds_frag(const unsigned char* p) {
    return *reinterpret_cast<const v4i*>(p);
}

// What a launch computes, from the device-resident counts.  PER: contraction steps (of 32 words) in
// a work unit, two but for the 32 x 256 tile on words (ring_tile.h).
struct Geometry {
    int n_eff, kc, KS, KT, m_eff, tiles_m, tiles_n, tiles;
    long units;     // (tile, contraction unit) pairs; a tile has KT = 2 KS / PER of them
};

template <int BM, int BN, int KIND, bool LISTED, int PER = 2>
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
// SPLIT_COST units above an even share, with more tiles than workgroups, with step lists, and where the caller
// fixes the slice length (p.chunk).  With less than a third of a tile per workgroup units are ordered
// chunk-major: all tiles for contraction units [0, CH), then all tiles for [CH, 2 CH), ...  With more, tile by
// tile, the parts of a tile in reverse order of their positions (see next()), and the row tiles of a column
// tile, when their number divides the grid, are walked side by side by as many consecutive workgroups: the weights of a
// unit are fetched once for all of them.  What that saves is the traffic of workgroups that start anywhere in
// the contraction (and the power it takes): planes, 256 x 4096 x 11008 662 -> 594 us, 512 x 4096 x 11008 1300 -> 1135,
// 512 x 2560 x 3000 229 -> 200; but 77 x 4096 x 1664, a fifth of a tile per workgroup, 55 -> 59.  With result blocks
// the same where every tile is listed, one component: words, 512 x 4096 x 11008 1709 -> 1402, 256 rows 830 -> 723, planes
// 256 x 4199 x 4800 307 -> 294.
//
// Either way, workgroups that run side by side sweep the same slice of the contraction at the same
// time (the activation planes of that slice stay hot in L2) and each XCD ends up with whole
// slices, so a weight word is fetched from HBM by one XCD only.
template <bool LISTED, int PER = 2>
struct UnitWalk {
    static constexpr int SPLIT_COST = 6 / PER;      // units: what a second segment costs a workgroup
    const GemmParams& p;
    const Geometry& q;
    long u_begin, u_end, u;
    int team_tm, tiles;
    int CH, n_chunks;
    int slice_tile;                                 // tile of this workgroup's slice, or -1: an even share
    bool rotate;                                    // see next()

    // workgroup b of G; own: every workgroup gets whole tiles
    __device__ __forceinline__ UnitWalk(const GemmParams& p_, const Geometry& q_, int b, int G, bool own)
        : p(p_), q(q_), team_tm(-1), tiles(q_.tiles) {
        slice_tile = -1;
        rotate = false;
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
        CH = p.chunk;
        if (!LISTED && !own && CH == 0 && 3l * tiles > G) {
            // (a list of all tiles is the plain order)
            const bool team = tiles == q.tiles_m * q.tiles_n && q.tiles_m > 1 && G % q.tiles_m == 0;
            const int part = team ? b / q.tiles_m : b, parts = team ? G / q.tiles_m : G;
            if (team) {
                team_tm = b % q.tiles_m;
                tiles = q.tiles_n;
            }
            u_begin = u = (long)tiles * q.KT * part / parts;
            u_end = (long)tiles * q.KT * (part + 1) / parts;
            CH = q.KT;
            n_chunks = 1;
            rotate = true;
            return;
        }
        u_begin = u = q.units * b / G;
        u_end = q.units * (b + 1) / G;
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
          CH(q_.KT), n_chunks(1), slice_tile(-1), rotate(true) {}

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
        if (!LISTED && rotate) {
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

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD one contiguous range of work.
__device__ __forceinline__ int xcd_contiguous(int b, int G) {
    return (G & 7) == 0 ? (b & 7) * (G >> 3) + (b >> 3) : b;
}


// Launch plan of the matrix-core kernels for an output tile BM x BN: the grid and whether the launch may turn out to
// own its tiles (owner: the kernel can).  Fixed before the packing kernel is launched, which has to know whether the
// share kernel will initialise Z itself.
inline void plan_gemm(const comet_ctx* ctx, GemmParams& p, int BM, int BN, bool owner, int per = 2, int wg_per_cu = 1) {
    const long tiles = (long)((p.m + BM - 1) / BM) * ((p.n_cap + BN - 1) / BN);
    const long pairs_cap = tiles * p.ks_cap;
    // as many workgroups as the chip holds, fewer when there are fewer pairs of contraction steps
    long grid = (ctx->num_cu / 8) * 8 * wg_per_cu;
    if (grid < 8) grid = 8;
    if (pairs_cap < grid) grid = pairs_cap < 8 ? (pairs_cap < 1 ? 1 : pairs_cap) : (pairs_cap / 8) * 8;
    if (ctx->gemm_grid > 0) grid = ctx->gemm_grid;
    // how the contraction is cut is decided on the device (UnitWalk), unless the caller fixes it
    p.chunk = ctx->gemm_chunk > 0 ? (ctx->gemm_chunk + per - 1) / per : 0;
    if (p.chunk > MAX_SEG / per) p.chunk = MAX_SEG / per;
    p.grid = (int)grid;
    p.tile_bm = BM;
    p.tile_bn = BN;
    // Owned tiles: plain product, default slicing, a tile count (at full capacity; the kernel checks the
    // device-resident counts) that the grid divides
    p.own_try = (owner && !p.row_comp && !p.tmask && ctx->gemm_chunk == 0 && tiles % grid == 0) ? 1 : 0;
}

// Launches a share kernel; when this launch is a timed one the event pair rides on the dispatch
// itself (its start and end timestamps): no marker packets before or after the kernel, so
// timing leaves the stream's schedule as it is.
template <class K, class P>
int launch_share_kernel(comet_ctx* ctx, const char* what, K kern, dim3 grid, const P& p, int threads = GT) {
    if (comet_time_this_launch(ctx)) {
        hipExtLaunchKernelGGL(kern, grid, dim3((unsigned)threads), 0, ctx->stream, ctx->ev[ctx->ev_used],
                              ctx->ev[ctx->ev_used + 1], 0, p);
        ctx->ev_used += 2;
    } else {
        hipLaunchKernelGGL(kern, grid, dim3((unsigned)threads), 0, ctx->stream, p);
    }
    COMET_LAUNCH_CHECK(ctx, what);
    return COMET_OK;
}

}  // namespace comet_gemm
