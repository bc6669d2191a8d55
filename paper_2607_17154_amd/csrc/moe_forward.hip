// Local MoE execution of one server on gfx950: the (token, slot) pairs that
// the selection assigned to this server are turned into expert rows, run
// through a grouped SwiGLU FFN and combined per token.
//
//   rows_count_kernel    per-block row counts per group (local experts, then
//                        the shared pseudo-expert), duplicates of one token
//                        merged
//   rows_scatter_kernel  each block totals the count table itself (group
//                        offsets, its position in each group), then places its
//                        rows stably (token order inside a group) with the
//                        merged gate weight and the token -> rows map; one more
//                        block makes the work lists of the two GEMMs
//   rows_small_kernel    both row kernels as one block (batches of at most
//                        1024 tokens)
//   ggemm_bf16<.., 0>    gate/up projection, X rows gathered through row_tok,
//                        packed [2f][d] weights, epilogue silu(g) * u -> bf16
//   ggemm_bf16<.., 1>    down projection of the activations, epilogue scales
//                        each row by its gate weight -> bf16 row outputs
//   ggemm_thin<0, 1>     the same two for batches with few rows per expert
//   ggemm_f32<0, 1>      the same two for fp32 storage
//   combine_kernel       y[t] = sum of t's row outputs in slot order (fp32)
// The GEMMs are persistent: each workgroup walks a tile list made on the device
// (row counts are never read by the host).  Tiles of one expert are ordered
// m-fastest so consecutive tiles share a weight tile, and workgroup ids are
// remapped so that each XCD (and its L2) works on a contiguous range of tiles.
// The tiled bf16 GEMMs fit the tile heights to the row counts
// (64 to 256 rows, see TilePlan): whole rounds of tiles, one tile per workgroup
// per round, then the tiles left over, cut along K into pieces at the same
// positions in every tile where that ends the launch sooner; the last workgroup
// to finish a piece of a split tile adds the pieces in a fixed order and runs
// the epilogue.  A shared group with a K at least twice the routed K has its
// tiles cut into up to four K pieces the same way, so that they do not set the
// length of the launch.
#include <hip/hip_runtime.h>

#include <type_traits>

#include <cstdint>

#include "common.hpp"

namespace ordermoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int FT_TB = 256;        // tokens per block in the row kernels
constexpr int MAXG = ORDERMOE_MAX_LOCAL + 1;
constexpr int MAXR = ORDERMOE_MAX_TOPK + 1;   // rows per token (routed + shared)
// bf16 GEMM launches: at most SK_MAX_GRID workgroups.  Every piece of a split
// tile has a slot for its partial tile, every split tile an arrival counter in
// one array of SK_MAX_GRID counters per GEMM (gate/up, down), zeroed by the row
// kernels before every forward.  A tile is cut into at most SK_SPLIT pieces (the
// last arrival reads them all).
constexpr int SK_MAX_GRID = 256;
constexpr int SK_SPLIT = 4;
constexpr int SK_MIN_PIECE_KT = 8;    // K tiles of 64 per piece, at least
// partial tiles of H x 64 rows in the workspace of SK_MAX_GRID whole tiles, whose
// last one's place holds the work lists
__host__ __device__ constexpr int sk_slots(int H) { return 4 * (SK_MAX_GRID - 1) / H; }

// Work list of a bf16 tiled GEMM, written by the row kernels for the launch that
// follows.  A group of R rows is covered by tiles of 64 H rows, H = 1 .. 4 chosen
// for the launch, and one last tile of as many 64-row units as the remainder
// needs.  The shared group comes first, then the routed groups; inside a group
// tiles are m-fastest, so that the tiles that read one weight tile run together.
constexpr int TP_BN = 256;
struct __attribute__((aligned(16))) TileSeg {
    int32_t first;            // the group's first work item
    int32_t mt_hl;            // row tiles * 8 + height of the last one in units of 64 rows
    int32_t off, R;           // first row, rows
};
struct __attribute__((aligned(16))) TilePlan {
    int32_t H;                // tile height in units of 64 rows
    int32_t rounds, items;    // whole rounds of the grid, work items (a shared tile counts once per K piece)
    int32_t sp0, split;       // items from sp0 on are cut along K into `split` pieces
    int32_t spread;           // the last, partial round is shared evenly by the XCDs
    int32_t q, nsh;           // K pieces of a shared tile, shared tiles
    TileSeg seg[ORDERMOE_MAX_LOCAL + 1];   // [g]; n_local: the shared group
};
// what the work list of one GEMM is made from: column tiles and K tiles of the
// routed and shared groups, K pieces of a shared tile wished for, workgroups
struct PlanShape {
    int32_t nt_r, nt_s, kt_r, kt_s, q, grid;
    uint32_t grid_inv;        // 2^32 / grid, rounded up
};
// Time of a tile of h 64-row units over kt K tiles of 64, in hundredths of the
// time of one K tile of a 256-row tile (1.5 us in a full chip): the K loop by
// height, and about five K tiles' time of start and epilogue.  The constants,
// and split_time below, were fitted to both GEMMs of the Mixtral-, Qwen-,
// DeepSeek- and 128-expert-shaped layers at 1000 to 16000 tokens, each timed
// with every height: the height that plan_tiles picks is on average 0.9% slower
// than the fastest of the four.
__host__ __device__ constexpr int tile_time(int h, int kt) {
    return kt * (h == 1 ? 50 : h == 2 ? 56 : h == 3 ? 74 : 100) + 500;
}
// storing and adding up the `pieces` partial tiles of a tile of height h
__host__ __device__ constexpr int split_time(int h, int pieces) { return h * (100 + 150 * pieces); }

struct RowsArgs {
    int64_t T;
    int k, E, n_local, has_shared, server;
    const float* w;
    const int32_t* exec_k;
    const uint8_t* exec_m;
    const uint8_t* loc_in;
    int32_t lidx[ORDERMOE_MAX_EXPERTS];   // expert -> local slot (kernel argument)
    int32_t* blk_rows;        // [nblk][G]
    int32_t* row_offsets;     // [n_local + 2]
    int32_t* row_tok;
    float* row_w;
    int32_t* tok_rows;        // [T][k+1]
    int32_t* tile_info;       // [4]
    int32_t* sk_cnt;          // [2][SK_MAX_GRID] split-tile arrival counters, zeroed here
    int nblk;
    // tile geometry for the tile counts
    int bm_gu, bn_gu, bm_dn, bn_dn;
    int n_gu_r, n_gu_s, n_dn;
    // bf16 tiled GEMMs: work lists of gate/up and down, published by the row kernels (null otherwise)
    TilePlan* plan;           // [2]
    PlanShape shape[2];
    int choose;               // bf16: thin or tiled GEMMs by the row counts (both are launched, one finds no tiles)
};

// One token's slots as read from memory: executing server, expert and gate
// weight per slot, and the token's server.  The reads are issued together
// (unused slots re-read the last slot, in range, and are discarded, so no
// branch separates them); the placement kernels issue them first, so that
// their latency overlaps the reads of the count table.  The arrays are
// indexed only by unrolled constants so that they stay in registers.
struct TokSlots {
    int m[ORDERMOE_MAX_TOPK], ek[ORDERMOE_MAX_TOPK];
    float wv[ORDERMOE_MAX_TOPK];
    int loc;
};
__device__ inline void token_read(const RowsArgs& a, int64_t t, TokSlots& s) {
#pragma unroll
    for (int i = 0; i < ORDERMOE_MAX_TOPK; ++i) {
        const int64_t o = t * a.k + (i < a.k ? i : a.k - 1);
        s.m[i] = a.exec_m[o];
        s.ek[i] = a.exec_k[o];
        s.wv[i] = a.w[o];
    }
    s.loc = a.has_shared ? (int)a.loc_in[t] : -1;
}

// rows of one token: group ids (local slot, or n_local for the shared group)
// and merged gate weights, in slot order of first occurrence
__device__ inline int token_rows(const RowsArgs& a, const int32_t* s_lidx, const TokSlots& ts, int* grp,
                                 float* wsum) {
    int m[ORDERMOE_MAX_TOPK], ek[ORDERMOE_MAX_TOPK];
    float wv[ORDERMOE_MAX_TOPK];
#pragma unroll
    for (int s = 0; s < ORDERMOE_MAX_TOPK; ++s) {
        const bool used = s < a.k;
        m[s] = used ? ts.m[s] : -1;
        ek[s] = used ? ts.ek[s] : -1;
        wv[s] = used ? ts.wv[s] : 0.f;
    }
    const int loc = ts.loc;
#pragma unroll
    for (int q = 0; q < MAXR; ++q) { grp[q] = -1; wsum[q] = 0.f; }
    int n = 0;
#pragma unroll
    for (int s = 0; s < ORDERMOE_MAX_TOPK; ++s) {
        const int e = ek[s];
        const int ls = (m[s] == a.server && e >= 0 && e < a.E) ? s_lidx[e] : -1;
        if (ls >= 0) {
            bool found = false;
#pragma unroll
            for (int q = 0; q < MAXR; ++q)
                if (grp[q] == ls) { wsum[q] = wsum[q] + wv[s]; found = true; }
            if (!found) {
#pragma unroll
                for (int q = 0; q < MAXR; ++q)
                    if (q == n) { grp[q] = ls; wsum[q] = wv[s]; }
                ++n;
            }
        }
    }
    if (loc == a.server) {
#pragma unroll
        for (int q = 0; q < MAXR; ++q)
            if (q == n) { grp[q] = a.n_local; wsum[q] = 1.0f; }
        ++n;
    }
    return n;
}

// Ranks of a wave's rows inside their groups (token order): each lane ORs its
// bit into the 64-bit lane mask of every group it has a row in (LDS atomics),
// then a row's rank is the number of lower lanes in its group's mask.  The
// wave's LDS operations run in program order, so the reads see every OR.  Also
// writes the wave's row count of every group to wcnt[0 .. G).
__device__ inline void wave_group_ranks(unsigned long long* msk, int G, int lane, const int* grp, int n,
                                        int* rank, int32_t* wcnt) {
    for (int g = lane; g < G; g += 64) msk[g] = 0ull;
    const unsigned long long bit = 1ull << lane;
#pragma unroll
    for (int q = 0; q < MAXR; ++q)
        if (q < n) atomicOr(&msk[grp[q]], bit);
#pragma unroll
    for (int q = 0; q < MAXR; ++q) {
        rank[q] = 0;
        if (q < n) rank[q] = __popcll(msk[grp[q]] & (bit - 1ull));
    }
    for (int g = lane; g < G; g += 64) wcnt[g] = __popcll(msk[g]);
}

// Inclusive scans over the 64 lanes of a wave by DPP row shifts and row
// broadcasts (a dozen cycles a step; a step through ds_bpermute waits for LDS,
// and the scans of the row kernels are a serial chain of them).  Lane 63 holds
// the total.  All lanes take part.
template <int CTRL, int ROWS>
__device__ inline int dpp_or0(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false); }
__device__ inline int wave_scan_add(int v) {
    v += dpp_or0<0x111, 0xF>(v);   // row_shr:1
    v += dpp_or0<0x112, 0xF>(v);
    v += dpp_or0<0x114, 0xF>(v);
    v += dpp_or0<0x118, 0xF>(v);
    v += dpp_or0<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    v += dpp_or0<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ inline int wave_max_nonneg(int v) {     // of values >= 0
    int o;
    o = dpp_or0<0x111, 0xF>(v); v = o > v ? o : v;
    o = dpp_or0<0x112, 0xF>(v); v = o > v ? o : v;
    o = dpp_or0<0x114, 0xF>(v); v = o > v ? o : v;
    o = dpp_or0<0x118, 0xF>(v); v = o > v ? o : v;
    o = dpp_or0<0x142, 0xA>(v); v = o > v ? o : v;
    o = dpp_or0<0x143, 0xC>(v); v = o > v ? o : v;
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ inline float wave_sum_f(float v) {
    v += __int_as_float(dpp_or0<0x111, 0xF>(__float_as_int(v)));
    v += __int_as_float(dpp_or0<0x112, 0xF>(__float_as_int(v)));
    v += __int_as_float(dpp_or0<0x114, 0xF>(__float_as_int(v)));
    v += __int_as_float(dpp_or0<0x118, 0xF>(__float_as_int(v)));
    v += __int_as_float(dpp_or0<0x142, 0xA>(__float_as_int(v)));
    v += __int_as_float(dpp_or0<0x143, 0xC>(__float_as_int(v)));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

__global__ void __launch_bounds__(FT_TB) rows_count_kernel(const RowsArgs a) {
    __shared__ int32_t s_lidx[ORDERMOE_MAX_EXPERTS];
    __shared__ int32_t s_h[MAXG];
    const int G = a.n_local + a.has_shared;
    for (int i = threadIdx.x; i < a.E; i += FT_TB) s_lidx[i] = a.lidx[i];
    for (int i = threadIdx.x; i < G; i += FT_TB) s_h[i] = 0;
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * FT_TB + threadIdx.x;
    if (t < a.T) {
        TokSlots ts;
        token_read(a, t, ts);
        int grp[MAXR];
        float ws[MAXR];
        const int n = token_rows(a, s_lidx, ts, grp, ws);
#pragma unroll
        for (int q = 0; q < MAXR; ++q)
            if (q < n) atomicAdd(&s_h[grp[q]], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < G; i += FT_TB) a.blk_rows[(int64_t)blockIdx.x * G + i] = s_h[i];
}

constexpr int SCAN_THREADS = 1024;
constexpr int SCAN_WAVES = SCAN_THREADS / 64;

// One wave: the group offsets (exclusive scan of the group totals tot[0..G),
// local experts then the shared group) into first[], and, when `publish`, the
// row offsets and the tile counts of the two GEMMs into device memory.  Returns
// whether the tiled GEMMs have work (bf16).  Where the row counts choose (a.choose;
// all groups have the same shape), the thin GEMM takes the batch unless its row
// tiles outnumber the groups in use by more than a quarter: 32 of 128 experts of
// d = 4096, f = 1536, thin and tiled us: 320 tokens, 20 rows each 200 and 222; one of
// 320, 31 of 10 rows (1.28) 230 and 233; 16 of 160 rows (5) 352 and 167; 512 tokens,
// 8 of 512 rows 507 and 177.
__device__ inline bool group_layout(const RowsArgs& a, const int32_t* tot, int32_t* first, int lane, bool publish) {
    const int G = a.n_local + a.has_shared;
    int32_t base = 0, tiles_gu = 0, tiles_dn = 0, used = 0, row_tiles = 0;
    for (int g0 = 0; g0 <= a.n_local; g0 += 64) {
        const int g = g0 + lane;
        const int32_t R = g < G ? tot[g] : 0;
        const int32_t inc = wave_scan_add(R);
        if (g <= a.n_local) {
            first[g] = base + inc - R;
            if (publish) a.row_offsets[g] = base + inc - R;
        }
        base += __builtin_amdgcn_readlane(inc, 63);
        // the tile counts of the GEMMs without a work list
        if (publish && (!a.plan || a.choose)) {
            int32_t tg = 0, td = 0;
            if (g < G) {
                const bool sh = g == a.n_local;
                tg = (R + a.bm_gu - 1) / a.bm_gu * ((sh ? a.n_gu_s : a.n_gu_r) / a.bn_gu);
                td = (R + a.bm_dn - 1) / a.bm_dn * (a.n_dn / a.bn_dn);
            }
            tiles_gu += __builtin_amdgcn_readlane(wave_scan_add(tg), 63);
            tiles_dn += __builtin_amdgcn_readlane(wave_scan_add(td), 63);
            if (a.choose) {
                used += __popcll(__builtin_amdgcn_ballot_w64(R > 0));
                row_tiles += __builtin_amdgcn_readlane(wave_scan_add((R + a.bm_gu - 1) / a.bm_gu), 63);
            }
        }
    }
    const bool tiled = a.plan && !(a.choose && 4 * row_tiles <= 5 * used);
    if (publish && lane == 0) {
        a.row_offsets[a.n_local + 1] = base;
        a.tile_info[0] = tiled ? 0 : tiles_gu;
        a.tile_info[1] = tiled ? 0 : tiles_dn;
        a.tile_info[2] = base;
        a.tile_info[3] = 0;
    }
    return tiled;
}

// x / n for x < 2^16 + 4 and n = 1 .. 4
__device__ inline int div4(int x, int n) { return n == 3 ? (int)(((uint32_t)x * 43691u) >> 17) : x >> (n >> 1); }

// The work list of one GEMM with tiles of 64 H rows and the estimated time of the
// launch, by one wave: lane g holds routed group g (R rows; Rs: shared rows).
struct PlanTry {
    float time;
    int first, mt_hl, mts_hls;                     // lane g; shared
    int rounds, items, sp0, split, spread, q, nsh;
};
__device__ inline PlanTry plan_tiles(const PlanShape& c, int R, int Rs, int lane, int H) {
    PlanTry o;
    const int u = (R + 63) >> 6, us = (Rs + 63) >> 6;            // (bf16: fewer than 2^22 rows)
    const int mt = div4(u + H - 1, H), hl = u - (mt - 1) * H;    // (mt = 0: unused)
    const int mts = div4(us + H - 1, H), hls = us - (mts - 1) * H;
    o.mt_hl = mt * 8 + (mt ? hl : 0);
    o.mts_hls = mts * 8 + (mts ? hls : 0);
    const int nsh = mts * c.nt_s, hs = mts > 1 ? H : hls;
    // the routed items: their number, their total time, the tallest one
    int inc = mt * c.nt_r, hmax = mt > 1 ? H : mt == 1 ? hl : 0;
    const int t_h = tile_time(H, c.kt_r);
    float sum_r = mt > 0 ? (float)c.nt_r * ((float)(mt - 1) * (float)t_h + (float)tile_time(hl, c.kt_r)) : 0.f;
    inc = wave_scan_add(inc);
    hmax = wave_max_nonneg(hmax);
    sum_r = wave_sum_f(sum_r);
    const int items_r = __builtin_amdgcn_readlane(inc, 63);
    const int long_r = hmax ? tile_time(hmax, c.kt_r) : 0, h_last = hmax ? hmax : hs;
    // shared tiles with a K of at least twice the routed K may be cut into up to
    // c.q pieces along K, as far as the slots and counters go
    const int qmax = nsh > 0 && nsh <= SK_MAX_GRID ? c.q : 1;
    o.time = 3.0e38f;
    for (int q = 1; q <= qmax && (q == 1 || q * nsh <= sk_slots(H)); ++q) {
        const int kt_q = div4(c.kt_s, q);
        const int sh_items = nsh * q, items = sh_items + items_r;
        float sum = sum_r;
        int longest = long_r;
        if (nsh > 0) {
            const int fix = q > 1 ? split_time(hs, q) : 0, ts = tile_time(hs, kt_q) + fix;
            longest = ts > longest ? ts : longest;
            sum += (float)(c.nt_s * q) *
                   ((float)(mts - 1) * (float)tile_time(H, kt_q) + (float)tile_time(hls, kt_q) + (float)(mts * fix));
        }
        // whole rounds, then the items left over; the routed ones of these are cut
        // along K into `split` pieces when that ends the launch sooner
        // (fewer than 2^21 items, so the multiplication is exact)
        const int rounds = (int)__umulhi((uint32_t)items, c.grid_inv), head = rounds * c.grid, left = items - head;
        const int sp0 = q > 1 && sh_items > head ? sh_items : head, ns = items - sp0, whole = sp0 - head;
        const float mean = items > 0 ? sum * __builtin_amdgcn_rcpf((float)items) : 0.f;
        const bool routed = head >= sh_items && hmax;            // the items left over are routed ones
        const float tail = (float)(routed ? long_r : longest);
        float base = 0.f;
        if (rounds > 0) {
            base = (float)rounds * mean + (tail > mean ? 0.5f * (tail - mean) : 0.f);
            if (base < (float)longest) base = (float)longest;
        }
        float best = base + (left > 0 ? tail : 0.f);
        // after one round, the snake order gives the items left over to the workgroups
        // that ran routed tiles while the others are still at their long shared ones
        if (rounds == 1 && routed && left > 0 && left <= head - sh_items && longest > long_r) {
            best = base - (float)(longest - long_r) + tail;
            if (best < (float)longest) best = (float)longest;
        }
        int split = 1;
        const bool even = nsh == 0 || 2 * kt_q <= 3 * c.kt_r;    // else a long shared tile outlasts the pieces
#pragma unroll
        for (int s = 2; s <= SK_SPLIT; ++s) {
            const int kp = div4(c.kt_r, s);
            const bool can = ns > 0 && even && whole + s * ns <= c.grid && (q > 1 ? sh_items : 0) + s * ns <= sk_slots(H) &&
                             ns + (q > 1 ? nsh : 0) <= SK_MAX_GRID && kp >= SK_MIN_PIECE_KT;
            int t = tile_time(h_last, kp) + split_time(h_last, s);
            if (whole > 0 && t < longest) t = longest;
            if (can && base + (float)t < best) { best = base + (float)t; split = s; }
        }
        if (best < o.time) {
            o.time = best;
            o.first = sh_items + inc - mt * c.nt_r;
            o.rounds = rounds; o.items = items; o.sp0 = sp0; o.split = split; o.q = q; o.nsh = nsh;
            // the last, partial round is spread over the XCDs when every tile has about
            // the same K; otherwise the snake order gives it to the workgroups that just
            // ran short tiles
            o.spread = even;
        }
    }
    return o;
}

// The work lists of both GEMMs: each of PW waves (4 or 8) tries tiles of one
// height, for one GEMM (8) or both (4), and the wave with the least estimate of a
// GEMM publishes (an empty list where the thin GEMMs take the batch).  publish_try,
// a barrier of the block, publish_best.
template <int PW>
__device__ inline void publish_try(const RowsArgs& a, const int32_t* tot, int lane, int wave, float (*s_est)[4], PlanTry* o) {
    const int n = a.n_local;
    const int R = lane < n ? tot[lane] : 0, Rs = a.has_shared ? tot[n] : 0;
#pragma unroll
    for (int i = 0; i < 8 / PW; ++i) {
        const int w = PW == 8 ? wave >> 2 : i;
        o[i] = plan_tiles(a.shape[w], R, Rs, lane, 4 - (wave & 3));
        if (lane == 0) s_est[w][wave & 3] = o[i].time;
    }
}
template <int PW>
__device__ inline void publish_best(const RowsArgs& a, const int32_t* tot, const int32_t* first, int lane, int wave,
                                    const float (*s_est)[4], PlanTry* o, bool tiled) {
    const int n = a.n_local;
#pragma unroll
    for (int i = 0; i < 8 / PW; ++i) {
        const int w = PW == 8 ? wave >> 2 : i;
        int bw = 0;
        float best = s_est[w][0];
#pragma unroll
        for (int j = 1; j < 4; ++j)
            if (s_est[w][j] < best) { best = s_est[w][j]; bw = j; }
        if (bw != (wave & 3)) continue;
        TilePlan* P = a.plan + w;
        if (!tiled) {
            o[i].rounds = o[i].items = o[i].sp0 = o[i].nsh = 0;
            o[i].split = o[i].q = 1;
        }
        if (lane == 0) {
            P->H = 4 - bw; P->rounds = o[i].rounds; P->items = o[i].items; P->sp0 = o[i].sp0; P->split = o[i].split;
            P->spread = o[i].spread; P->q = o[i].q; P->nsh = o[i].nsh;
            P->seg[n] = TileSeg{0, o[i].mts_hls, a.has_shared ? first[n] : 0, a.has_shared ? tot[n] : 0};
        }
        if (lane < n) P->seg[lane] = TileSeg{o[i].first, o[i].mt_hl, first[lane], tot[lane]};
    }
}

// Placement of every row, one block per block of rows_count_kernel, and for the
// bf16 GEMMs one block more that makes their work lists meanwhile.  Each
// block first totals the count table on its own (groups x blocks integers):
// its first row inside each group (the counts of the blocks before it) and the
// group totals, whose exclusive scan gives the group offsets; block 0 also
// publishes the row offsets and tile counts and clears the split-tile arrival
// counters of the GEMMs.  Then every row goes to its group offset + block
// position + its rank in token order.
__global__ void __launch_bounds__(FT_TB) rows_scatter_kernel(const RowsArgs a) {
    __shared__ int32_t s_lidx[ORDERMOE_MAX_EXPERTS];
    __shared__ int32_t s_wcnt[FT_TB / 64][MAXG];
    __shared__ unsigned long long s_msk[FT_TB / 64][MAXG];
    __shared__ int32_t s_lo[MAXG], s_tot[MAXG];
    __shared__ int32_t s_first[MAXG];        // first row of this block in each group
    __shared__ float s_est[2][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = a.n_local + a.has_shared;
    const int b = (int)blockIdx.x;
    const int64_t t = (int64_t)b * FT_TB + tid;
    TokSlots ts;
    if (t < a.T) token_read(a, t, ts);
    for (int i = tid; i < a.E; i += FT_TB) s_lidx[i] = a.lidx[i];
    if (b == 0)
        for (int i = tid; i < 2 * SK_MAX_GRID; i += FT_TB) a.sk_cnt[i] = 0;
    for (int g = wave; g < G; g += FT_TB / 64) {
        int32_t lo = 0, tot = 0;
        for (int i = lane; i < a.nblk; i += 64) {
            const int32_t v = a.blk_rows[(int64_t)i * G + g];
            tot += v;
            lo += i < b ? v : 0;
        }
        for (int off = 32; off >= 1; off >>= 1) {
            lo += __shfl_xor(lo, off);
            tot += __shfl_xor(tot, off);
        }
        if (lane == 0) { s_lo[g] = lo; s_tot[g] = tot; }
    }
    __syncthreads();
    if (b == a.nblk) {
        // the block past the rows: work lists of the GEMMs (t >= T: no rows here)
        if (wave == 0) group_layout(a, s_tot, s_first, lane, false);
        static_assert(FT_TB / 64 == 4, "one wave per tile height");
        PlanTry o[2];
        publish_try<4>(a, s_tot, lane, wave, s_est, o);
        __syncthreads();
        publish_best<4>(a, s_tot, s_first, lane, wave, s_est, o, true);
        return;
    }
    int grp[MAXR], rank[MAXR];
    float ws[MAXR];
    int n = 0;
    if (t < a.T) {
        n = token_rows(a, s_lidx, ts, grp, ws);
    } else {
#pragma unroll
        for (int q = 0; q < MAXR; ++q) { grp[q] = -1; ws[q] = 0.f; }
    }
    wave_group_ranks(s_msk[wave], G, lane, grp, n, rank, s_wcnt[wave]);
    if (wave == 0) {
        group_layout(a, s_tot, s_first, lane, b == 0);
        for (int g = lane; g < G; g += 64) s_first[g] += s_lo[g];
    }
    __syncthreads();
    if (t < a.T) {
        const int stride = a.k + 1;
#pragma unroll
        for (int q = 0; q < MAXR; ++q) {
            if (q < n) {
                const int g = grp[q];
                int32_t pos = s_first[g] + rank[q];
                for (int w = 0; w < wave; ++w) pos += s_wcnt[w][g];
                a.row_tok[pos] = (int32_t)t;
                a.row_w[pos] = ws[q];
                a.tok_rows[t * stride + q] = pos;
            } else if (q < stride) {
                a.tok_rows[t * stride + q] = -1;
            }
        }
    }
}

// Batches of at most SCAN_THREADS tokens (decode): the row kernels as one
// block, one token per thread -- group ranks by wave lane masks, group totals,
// row offsets and tile counts, then the placement (as rows_scatter_kernel).
__global__ void __launch_bounds__(SCAN_THREADS) rows_small_kernel(const RowsArgs a) {
    __shared__ int32_t s_lidx[ORDERMOE_MAX_EXPERTS];
    __shared__ int32_t s_wcnt[SCAN_WAVES][MAXG];
    __shared__ unsigned long long s_msk[SCAN_WAVES][MAXG];
    __shared__ int32_t s_first[MAXG], s_tot[MAXG];
    __shared__ float s_est[2][4];
    __shared__ int s_tiled;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = a.n_local + a.has_shared;
    const int64_t t = tid;
    TokSlots ts;
    if (t < a.T) token_read(a, t, ts);
    for (int i = tid; i < a.E; i += SCAN_THREADS) s_lidx[i] = a.lidx[i];
    for (int i = tid; i < 2 * SK_MAX_GRID; i += SCAN_THREADS) a.sk_cnt[i] = 0;
    __syncthreads();
    int grp[MAXR], rank[MAXR];
    float ws[MAXR];
    int n = 0;
    if (t < a.T) {
        n = token_rows(a, s_lidx, ts, grp, ws);
    } else {
#pragma unroll
        for (int q = 0; q < MAXR; ++q) { grp[q] = -1; ws[q] = 0.f; }
    }
    wave_group_ranks(s_msk[wave], G, lane, grp, n, rank, s_wcnt[wave]);
    __syncthreads();
    if (tid < G) {
        int32_t R = 0;
        for (int w = 0; w < SCAN_WAVES; ++w) R += s_wcnt[w][tid];
        s_tot[tid] = R;
    }
    __syncthreads();
    // the last eight waves, which hold the fewest tokens, make the GEMMs' work lists
    // while wave 0 lays out the groups
    constexpr int PW0 = SCAN_WAVES - 8;
    const bool planner = a.plan && wave >= PW0;
    PlanTry o[1];
    if (wave == 0) {
        const bool tiled = group_layout(a, s_tot, s_first, lane, true);
        if (lane == 0) s_tiled = tiled;
    }
    if (planner) publish_try<8>(a, s_tot, lane, wave - PW0, s_est, o);
    __syncthreads();
    if (planner) publish_best<8>(a, s_tot, s_first, lane, wave - PW0, s_est, o, s_tiled != 0);
    if (t < a.T) {
        const int stride = a.k + 1;
#pragma unroll
        for (int q = 0; q < MAXR; ++q) {
            if (q < n) {
                const int g = grp[q];
                int32_t pos = s_first[g] + rank[q];
                for (int w = 0; w < wave; ++w) pos += s_wcnt[w][g];
                a.row_tok[pos] = (int32_t)t;
                a.row_w[pos] = ws[q];
                a.tok_rows[t * stride + q] = pos;
            } else if (q < stride) {
                a.tok_rows[t * stride + q] = -1;
            }
        }
    }
}

// ---------------------------------------------------------------- weights
// One-time packing (offline).  bf16 weights are stored tile-blocked: a matrix
// [N][K] (N % 256 == 0, K % 64 == 0) becomes [N/256][K/64][256][64], so that
// the 256 weight rows a GEMM tile reads in one 64-deep K step are one 32 KB
// block (and the 64 rows a thin-GEMM workgroup reads per K step 8 KB of it):
// the weight stream leaves DRAM in whole contiguous blocks instead of 128-byte
// slices of rows 8 or 28 KB apart.  fp32 weights keep the row layout.
constexpr int WB_ROWS = 256, WB_K = 64;
__host__ __device__ inline int64_t wblk_elem(int64_t n, int64_t k, int64_t K) {
    return ((n / WB_ROWS) * (K / WB_K) + k / WB_K) * (WB_ROWS * WB_K) + (n % WB_ROWS) * WB_K + k % WB_K;
}

// bf16: a block takes 8 consecutive packed rows (rows [64b, 64b+32) of an expert
// are gate rows [32b, 32b+32), rows [64b+32, 64b+64) the matching up rows, so 8
// packed rows are 8 rows of one source; down rows stay in place).  A wave
// instruction covers one K step of them: lane l reads 16 bytes of row l / 8, whole
// 128-byte lines, and the 64 lanes write 1 KB in a row; PK_U K steps in flight per
// wave.  The stream is bound by HBM and used once, so both sides are
// non-temporal.  Two experts of d = 4096, f = 14336 (1.41 GB read and written),
// gate/up and down together: 236 us (6.0 TB/s); a block per row with ordinary
// loads and 128-byte writes took 265.
constexpr int PK_THREADS = 256, PK_U = 8;
typedef unsigned int pk_u32x4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(PK_THREADS) pack_bf16_kernel(int rows, int K, bool gate_up, const __bf16* a, const __bf16* b,
                                                               __bf16* out) {
    const int64_t r0 = (int64_t)blockIdx.x * 8;       // first packed row, over all experts
    const int64_t ex = r0 / rows;
    const int pr = (int)(r0 % rows);                  // inside the expert
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const __bf16* src = gate_up ? ((pr & 32) ? b : a) + (ex * (rows / 2) + (pr / 64) * 32 + (pr & 31)) * (int64_t)K
                                : a + r0 * K;
    src += (int64_t)(lane >> 3) * K + (lane & 7) * 8;
    __bf16* dst = out + ex * rows * (int64_t)K + wblk_elem(pr, 0, K) + lane * 8;
    const int nks = K / WB_K;
    for (int k0 = wave * PK_U; k0 < nks; k0 += PK_THREADS / 64 * PK_U) {
        pk_u32x4 v[PK_U];
#pragma unroll
        for (int u = 0; u < PK_U; ++u)
            if (k0 + u < nks) v[u] = __builtin_nontemporal_load((const pk_u32x4*)(src + (int64_t)(k0 + u) * WB_K));
#pragma unroll
        for (int u = 0; u < PK_U; ++u)
            if (k0 + u < nks) __builtin_nontemporal_store(v[u], (pk_u32x4*)(dst + (int64_t)(k0 + u) * (WB_ROWS * WB_K)));
    }
}

// fp32: one block per row, copied 16 bytes at a time (K is a multiple of 8)
__global__ void __launch_bounds__(PK_THREADS) pack_f32_kernel(int rows, int K, bool gate_up, const float* a, const float* b,
                                                              float* out) {
    const int64_t r = blockIdx.x, ex = r / rows;
    const int pr = (int)(r % rows);
    const pk_u32x4* src = (const pk_u32x4*)(gate_up ? ((pr & 32) ? b : a) + (ex * (rows / 2) + (pr / 64) * 32 + (pr & 31)) * (int64_t)K
                                                    : a + r * K);
    pk_u32x4* dst = (pk_u32x4*)(out + r * (int64_t)K);
    for (int i = threadIdx.x; i < K / 4; i += PK_THREADS)
        __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// ---------------------------------------------------------------- GEMMs
struct GemmArgs {
    const int32_t* offsets;   // [G + 1] row offsets of the groups (device)
    const int32_t* ntiles;    // device: number of tiles
    int G, n_routed;          // groups; groups >= n_routed are the shared group
    int Nr, Kr, Ns, Ks;       // N, K of routed and shared groups
    const void* Wr;           // [n_routed][Nr][Kr]
    const void* Ws;           // [Ns][Ks]
    const void* X;            // mode 0: token rows [T][ldx]
    const int32_t* row_tok;   // mode 0
    int ldx;
    uint32_t x_bytes;         // mode 0: size of X in bytes
    const void* Ar;           // mode 1: routed activations [*][Kr]
    const void* As;           // mode 1: shared activations [*][Ks]
    void* Or;                 // mode 0: routed activations out; mode 1: row outputs [*][Nr]
    void* Os;                 // mode 0: shared activations out; mode 1: unused
    const float* row_w;       // mode 1
    const TilePlan* plan;     // bf16 tiled: the work list
    int stream;               // bf16: see STREAM_BYTES
    float* sk_part;           // bf16 tiled: [sk_slots(H)][64 H * 256] partial tiles of split tiles
    int32_t* sk_cnt;          // bf16: [2][SK_MAX_GRID] arrival counters (zero at launch)
};

struct TileLoc {
    int g, m0, n0, R, N, K, rowbase;
};

// Tile order: the shared group first (its down projection has the longest K,
// so its tiles start first and the shorter routed tiles fill in around them),
// then the routed groups; inside a group tiles are m-fastest.  Lane g of a wave
// holds routed group g: one read of the row offsets and one scan give every
// group's first tile, and a ballot finds the group of a tile.  (A loop over the
// groups waits for the reads of one group after the other: 4 us of a one-token
// layer of 32 local experts, 3 us of the 8192-token Qwen-shaped layer.)
struct GroupScan {
    int off, R, cum;              // lane g: first row, rows and first tile of routed group g
    int sh_off, sh_R, sh_cnt;     // shared group: first row, rows and tiles
};
template <int BM, int BN>
__device__ inline GroupScan scan_groups(const GemmArgs& p, int lane) {
    static_assert(ORDERMOE_MAX_LOCAL <= 64, "one routed group per lane");
    const int n = p.n_routed;
    GroupScan s;
    const int o1 = p.offsets[lane < n ? lane + 1 : n];
    s.off = p.offsets[lane < n ? lane : n];
    s.R = o1 - s.off;             // lanes past the groups: none
    s.sh_off = s.sh_R = s.sh_cnt = 0;
    if (p.G > n) {
        s.sh_off = p.offsets[n];
        s.sh_R = p.offsets[n + 1] - s.sh_off;
        s.sh_cnt = (s.sh_R + BM - 1) / BM * (p.Ns / BN);
    }
    const int cnt = (s.R + BM - 1) / BM * (p.Nr / BN);
    int inc = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(inc, o);
        if (lane >= o) inc += v;
    }
    s.cum = inc - cnt;
    return s;
}
template <int BM, int BN>
__device__ inline bool find_tile(const GemmArgs& p, const GroupScan& s, int tile, int lane, TileLoc& L) {
    int rem = tile;
    if (tile < s.sh_cnt) {
        L.g = p.n_routed; L.R = s.sh_R; L.N = p.Ns; L.K = p.Ks; L.rowbase = s.sh_off;
    } else {
        rem -= s.sh_cnt;
        const uint64_t m = __builtin_amdgcn_ballot_w64(lane < p.n_routed && s.cum <= rem);
        if (!m) return false;
        // the last group that starts at or before the tile (an empty group starts where the next one does)
        const int g = 63 - __builtin_clzll(m);
        L.g = g; L.N = p.Nr; L.K = p.Kr;
        L.R = __builtin_amdgcn_readlane(s.R, g);
        L.rowbase = __builtin_amdgcn_readlane(s.off, g);
        rem -= __builtin_amdgcn_readlane(s.cum, g);
    }
    const int mt = (L.R + BM - 1) / BM;
    if (rem >= mt * (L.N / BN)) return false;
    L.m0 = (rem % mt) * BM;
    L.n0 = (rem / mt) * BN;
    return true;
}

// Position of workgroup vid in round r of n work items (n <= grid): odd
// rounds mirrored (snake order); with `spread`, a partial round is shared
// evenly by the 8 XCDs (vid / (grid / 8) is the workgroup's XCD), so that no
// XCD sits idle while another runs a full share.  -1: no item for this
// workgroup.
__device__ inline int round_pos(int vid, int r, int n, int grid, bool spread) {
    const int v = (r & 1) ? grid - 1 - vid : vid;
    if (n >= grid || !spread) return v < n ? v : -1;
    const int g8 = grid >> 3, x = v / g8, j = v - x * g8;
    const int lo = x * n / 8, hi = (x + 1) * n / 8;
    return j < hi - lo ? lo + j : -1;
}

// silu(g) = g / (1 + e^-g), with the hardware reciprocal (1 ulp) instead of an
// IEEE divide: the result is rounded to bf16 right after
__device__ inline float silu_f(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// s_waitcnt operand on gfx9-class GPUs: vmcnt (6 bits, split), expcnt (left at
// its maximum), lgkmcnt (4 bits)
constexpr int waitcnt_enc(int vm, int lgkm) { return (vm & 0xF) | ((vm >> 4) << 14) | (7 << 4) | ((lgkm & 0xF) << 8); }

// Workgroup barrier of the K loop.  __syncthreads() (and a workgroup fence on
// LDS alone) waits for every outstanding load into LDS (vmcnt 0), which would
// also drain the loads of a buffer that is read only a tile later; this one
// is the bare s_barrier, and the memory clobber keeps the compiler from moving
// memory accesses across it.  The caller first waits (s_waitcnt vmcnt) for its
// own loads into the buffers read after the barrier, and every LDS read of a
// buffer has returned its data (it fed an MFMA) before the barrier that
// precedes the next load into that buffer.  Nothing waits for LDS writes
// either: __syncthreads() where other waves read them.
__device__ inline void lds_barrier() { asm volatile("s_barrier" ::: "memory"); }

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr int BUF_DWORD3 = 0x00020000;   // raw buffer resource word 3 on gfx9-class GPUs
constexpr int NT = 2;                    // buffer load/store cache bit nt: non-temporal
constexpr int SC1 = 16;                  // buffer load/store cache bit sc1: coherent at agent scope

__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, BUF_DWORD3);
}

template <int AUX = 0>
__device__ inline bf16x8 buf_load16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, AUX);
    return __builtin_bit_cast(bf16x8, v);
}

// Scheduling pattern of one MFMA sub-step: NM MFMAs with NR LDS fragment
// reads and NX other memory instructions (mask XMASK) spread between them,
// reads after even-numbered MFMAs, the others after odd-numbered ones.
template <int Q, int NM, int NR, int NX, int XMASK>
__device__ inline void sched_interleave() {
    if constexpr (Q < NM) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
        constexpr int r = ((Q + 1) * NR + NM - 1) / NM - (Q * NR + NM - 1) / NM;
        if constexpr (r > 0) __builtin_amdgcn_sched_group_barrier(0x100, r, 0);   // LDS read
        constexpr int x = (Q + 1) * NX / NM - Q * NX / NM;
        if constexpr (x > 0) __builtin_amdgcn_sched_group_barrier(XMASK, x, 0);
        sched_interleave<Q + 1, NM, NR, NX, XMASK>();
    }
}

// bf16 grouped GEMM C = A B^T per tile of BM x 256, K step 64, 4 waves (2 x 2),
// each wave a (BM/2) x 128 block of v_mfma_f32_32x32x16_bf16 tiles.  Operands go
// from memory straight into LDS (buffer loads to LDS), two buffers of A and
// three of B, [rows][64] bf16 each; the layout is described at the K loop.  The
// K position travels in the buffer load's scalar offset, and rows past the end
// of a group read as zeros through the buffer range check (their offset is set
// past the buffer).  Byte offsets inside one operand fit in 31 bits (checked by
// the host).  A piece of a split tile stores its fp32 partial tile in its slot,
// and the workgroup whose arrival completes the tile's counter sums the tile's
// pieces in K order (so the result does not depend on who is last) and runs the
// epilogue.  No workgroup waits for another.
// One tile (or K piece of a tile): BM x 256 outputs over the K tiles
// [kt_lo, kt_hi).  nseg > 1: piece of a split tile, its partial sums in slot
// pslot, the tile's pieces in slots pslot0 + i * sstride, arrivals counted in
// counter ctr.
template <int BM, int MODE, int BAUX = 0>
__device__ __attribute__((always_inline)) inline void bf16_tile(const GemmArgs& p, const TileLoc& L, int kt_lo, int kt_hi,
                                                                int nseg, int ctr, int pslot, int pslot0, int sstride,
                                                                uint32_t slot_bytes, __bf16* sA0, __bf16* sA1, __bf16* sB0, __bf16* sB1,
                                                                __bf16* sB2) {
    constexpr int BN = TP_BN;
    constexpr int BK = 64;
    constexpr int WM = BM / 2, WN = BN / 2;
    constexpr int FM = WM / 32, FN = WN / 32;
    constexpr int AV = BM / 32;                     // 8-row load instructions per wave and K tile
    constexpr int BV = BN / 32;
    static_assert(FN % 2 == 0, "gate/up pairs need an even number of 32-column blocks");
    static_assert(BM % 64 == 0 && BN % 64 == 0, "an even number of load instructions per wave");
    constexpr uint32_t OOR = 0x80000000u;           // offset past every buffer: reads zero
    // the split-tile arrival flag and (down) the gate weights of the tile's rows
    // live in sB2, which is idle from the end of a K loop until the first K tile
    // of the next one (a prologue loads sA0, sA1, sB0 and sB1 only), so that the
    // buffers of 256-row tiles fill the LDS
    int* const s_last = (int*)sB2;
    float* const s_roww = (float*)sB2 + 64;
    static_assert(256 + BM * 4 <= BN * 64 * 2, "flag and row weights fit sB2");
    // the thread index passes through an empty asm once per tile, so that
    // the thread-dependent offsets below are recomputed per tile instead of
    // being held (and spilled to scratch) across the whole persistent loop
    int tid_r = threadIdx.x;
    asm volatile("" : "+v"(tid_r));
    const int lane_r = tid_r & 63, wave_r = tid_r >> 6;
    const int wm_r = wave_r >> 1, wn_r = wave_r & 1;
    // the wave index as a scalar: the LDS destinations of the loads into LDS
    // (the M0 operand) are then scalar expressions, not VGPRs held per buffer
    const int wave_u = __builtin_amdgcn_readfirstlane(wave_r);
    const bool shared = L.g >= p.n_routed;
    const int K = L.K;
    const __bf16* Bw = shared ? (const __bf16*)p.Ws
                              : (const __bf16*)p.Wr + (size_t)L.g * L.N * K;
    const __amdgpu_buffer_rsrc_t rb_rs = make_rsrc(Bw, (uint32_t)((size_t)L.N * K * 2));
    // LDS rows of 64 K values (128 bytes, unpadded); 16-byte chunk q of
    // row r holds the operand's chunk q ^ ((r >> 1) & 7), so that the 16
    // rows a fragment read serves per LDS cycle (16 lanes of 16 bytes over
    // the 64 banks) fall on distinct banks.  Load instruction v of wave_r w
    // covers rows (w AV + v) 8 .. +7 of the tile: lane_r l takes row + l / 8
    // and fetches the chunk that the direct-to-LDS load writes at position
    // l & 7 of that row, (l & 7) ^ ((r >> 1) & 7); with AV, BV even that is
    // gc0 for even v and gc1 for odd v.
    const int gc0 = (lane_r & 7) ^ (lane_r >> 4);
    const int gc1 = (lane_r & 7) ^ (4 | (lane_r >> 4));
    const int rsub = lane_r >> 3;
    // A: the gathered token rows of X (gate/up) or the group's activation rows (down)
    const __bf16* Ab = MODE == 0 ? (const __bf16*)p.X
                                 : (shared ? (const __bf16*)p.As : (const __bf16*)p.Ar + (size_t)L.rowbase * K);
    const __amdgpu_buffer_rsrc_t ra_rs =
        make_rsrc(Ab, MODE == 0 ? p.x_bytes : (uint32_t)((size_t)L.R * K * 2));
    // down: thread tid_r < BM reads the gate weight of tile row tid_r now (one
    // branch-free load, rows past the group read zero) and parks it in LDS
    // after the K loop, so that the epilogue waits for no global load
    float roww = 0.f;
    if constexpr (MODE == 1) {
        const __amdgpu_buffer_rsrc_t rw_rs = make_rsrc(p.row_w + L.rowbase, (uint32_t)L.R * 4u);
        const int rr = L.m0 + tid_r;
        roww = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                             rw_rs, tid_r < BM && rr < L.R ? rr * 4 : (int)OOR, 0, 0));
    }
    uint32_t aoff[AV];
#pragma unroll
    for (int v = 0; v < AV; ++v) {
        const int row = L.m0 + (wave_r * AV + v) * 8 + rsub;
        const uint32_t src = MODE == 0 ? (row < L.R ? (uint32_t)p.row_tok[L.rowbase + row] : 0u) : (uint32_t)row;
        aoff[v] = row < L.R ? (src * (uint32_t)(MODE == 0 ? p.ldx : K) + ((v & 1) ? gc1 : gc0) * 8) * 2u : OOR;
    }
    // B: the blocked weights (256-row blocks of 64-deep K steps, 128-byte
    // rows): load instruction v of wave_r w covers rows (w BV + v) 8 .. +7
    // of the tile's block, 1 KB in a row; the K step goes in the scalar offset
    static_assert(BN == WB_ROWS, "a tile's weight rows are one block");
    const uint32_t bblk = (uint32_t)(L.n0 / BN) * (uint32_t)(K / WB_K) * (uint32_t)(BN * WB_K * 2) +
                          (uint32_t)(wave_r * BV * 8 + rsub) * (WB_K * 2u);

    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // the loads of a K tile go from memory straight into LDS buffer b
    auto dmaA = [&](__bf16* sa, int k0) {
#pragma unroll
        for (int v = 0; v < AV; ++v) {
            // (a local copy: the host pass drops the kernel when an array
            // element captured by reference is the builtin's operand)
            const uint32_t vo = aoff[v];
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra_rs, (lds_ptr)(sa + (wave_u * AV + v) * 8 * 64), 16, vo,
                                                     (uint32_t)k0 * 2u, 0, 0);
        }
    };
    auto dmaB = [&](__bf16* sb, int k0) {
#pragma unroll
        for (int v = 0; v < BV; ++v)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rb_rs, (lds_ptr)(sb + (wave_u * BV + v) * 8 * 64), 16,
                                                     bblk + v * 1024u + (uint32_t)((v & 1) ? gc1 : gc0) * 16u,
                                                     (uint32_t)k0 * (uint32_t)(BN * 2), 0, BAUX);
    };
    // fragment of row (lane_r & 31) of each 32-row block, K chunk 2 ks + lane_r / 32
    const int arow = (wm_r * WM + (lane_r & 31)) * 64;
    const int brow = (wn_r * WN + (lane_r & 31)) * 64;
    bf16x8 af[2][FM], bfm[2][FN];
    auto fload = [&](const __bf16* sa, const __bf16* sb, int ks, int slot) {
        const int pos = ((2 * ks + (lane_r >> 5)) ^ ((lane_r >> 1) & 7)) * 8;   // row & 31 = lane_r & 31
#pragma unroll
        for (int i = 0; i < FM; ++i) af[slot][i] = *(const bf16x8*)(sa + arow + i * 32 * 64 + pos);
#pragma unroll
        for (int j = 0; j < FN; ++j) bfm[slot][j] = *(const bf16x8*)(sb + brow + j * 32 * 64 + pos);
    };
    // the first sub-step's fragments after the barrier, in the order the
    // MFMAs consume them (A0 B0, then B1.., then A1..), each read fenced so
    // that the first MFMAs wait for their own operands only (the scheduler
    // had issued B0 and B1 last, so every K tile began by waiting for seven
    // of the eight reads)
    auto fload_first = [&](const __bf16* sa, const __bf16* sb) {
        const int pos = ((lane_r >> 5) ^ ((lane_r >> 1) & 7)) * 8;   // sub-step 0
        af[0][0] = *(const bf16x8*)(sa + arow + pos);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            bfm[0][j] = *(const bf16x8*)(sb + brow + j * 32 * 64 + pos);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 1; i < FM; ++i) {
            af[0][i] = *(const bf16x8*)(sa + arow + i * 32 * 64 + pos);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto mfmas = [&](int slot) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[slot][i], bfm[slot][j], acc[i][j], 0, 0, 0);
    };
    // Each K tile of 64 is four MFMA sub-steps of 16; every sub-step reads
    // the fragments of the next one.  The buffers are separate LDS arrays
    // and the loop is unrolled over a pass of six tiles (A cycles over two
    // buffers, B over three), so that every access names a fixed array and
    // the loads into one buffer are never taken to alias the reads of
    // another.  The barrier of K tile t sits before its last sub-step.
    // Sub-step 0 issues the B loads of tile t + 2 (into the buffer tile
    // t - 1 read, free since barrier t - 1); after sub-step 2 every fragment
    // of tile t has been read, so the wave waits for its own loads of tile
    // t + 1 (everything but the B loads just issued) and its reads, and the
    // barrier follows; sub-step 3's MFMAs then overlap the first fragment
    // reads of tile t + 1 and the A loads of tile t + 2 into the A buffer
    // tile t has just finished with.  The A loads keep a lead of four
    // sub-steps, the B loads of seven; no tile starts by waiting for its
    // first fragments.  Loads past the piece re-read its last K tile into
    // an idle buffer.
    constexpr int NM = FM * FN, NR = FM + FN;
    constexpr int VMEM_READ = 0x020;
    auto ktile = [&](__bf16* ca, __bf16* cb, __bf16* na, __bf16* nbn, __bf16* nbl, int kn2)
                     __attribute__((always_inline)) {
        dmaB(nbl, kn2);
        fload(ca, cb, 1, 1);
        mfmas(0);
        sched_interleave<0, NM, NR, BV, VMEM_READ>();
        __builtin_amdgcn_sched_barrier(0);
        fload(ca, cb, 2, 0);
        mfmas(1);
        sched_interleave<0, NM, NR, 0, VMEM_READ>();
        __builtin_amdgcn_sched_barrier(0);
        fload(ca, cb, 3, 1);
        mfmas(0);
        sched_interleave<0, NM, NR, 0, VMEM_READ>();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(waitcnt_enc(BV, 0));
        lds_barrier();
        dmaA(ca, kn2);
        fload(na, nbn, 0, 0);
        mfmas(1);
        sched_interleave<0, NM, NR, AV, VMEM_READ>();
        __builtin_amdgcn_sched_barrier(0);
    };
    // the piece's K tiles [kt_lo, kt_hi): an even number (K units of 128)
    const int klast = kt_hi - 1;
    auto kc = [&](int k) { return (k < kt_hi ? k : klast) * BK; };
    // buffers of tile kt + u of a pass (compile-time u)
    auto bufA = [&](auto u) -> __bf16* { return decltype(u)::value % 2 == 0 ? sA0 : sA1; };
    auto bufB = [&](auto u) -> __bf16* {
        constexpr int j = decltype(u)::value % 3;
        if constexpr (j == 0) return sB0; else if constexpr (j == 1) return sB1; else return sB2;
    };
    // prologue: tiles kt_lo and kt_lo + 1 of both operands
    dmaA(sA0, kt_lo * BK);
    dmaB(sB0, kt_lo * BK);
    dmaB(sB1, kc(kt_lo + 1));
    dmaA(sA1, kc(kt_lo + 1));
    static_assert(AV + BV < 64, "vmcnt field");
    __builtin_amdgcn_s_waitcnt(waitcnt_enc(AV + BV, 15));   // tile kt_lo's loads are in LDS
    lds_barrier();
    fload_first(sA0, sB0);
    __builtin_amdgcn_sched_barrier(0);
    auto step = [&](auto u, int kt) __attribute__((always_inline)) {
        constexpr int U = decltype(u)::value;
        using N1 = std::integral_constant<int, U + 1>;
        using N2 = std::integral_constant<int, U + 2>;
        ktile(bufA(u), bufB(u), bufA(N1{}), bufB(N1{}), bufB(N2{}), kc(kt + U + 2));
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    using I4 = std::integral_constant<int, 4>;
    using I5 = std::integral_constant<int, 5>;
    int kt = kt_lo;
    for (; kt + 6 <= kt_hi; kt += 6) {
        step(I0{}, kt); step(I1{}, kt); step(I2{}, kt);
        step(I3{}, kt); step(I4{}, kt); step(I5{}, kt);
    }
    // the two or four tiles left start a pass
    if (kt < kt_hi) {
        step(I0{}, kt); step(I1{}, kt);
        if (kt + 2 < kt_hi) { step(I2{}, kt); step(I3{}, kt); }
    }
    // loads of the tiles after the last may still be in flight: this wave waits
    // for its own, and the barrier holds until every wave's have arrived.  Which
    // rows a wave loads depends on the tile height, so without it a late wave's
    // loads could overwrite rows that another wave loads for the next tile; the
    // epilogues also reuse sB2.
    __builtin_amdgcn_s_waitcnt(0x0F70);
    lds_barrier();

    if (nseg > 1) {
        // a piece of a split tile: its partial sums go to slot j sstride + ctr
        // (its position in the round), thread tid_r's 16-byte group h of
        // block (i, j) at byte (((i FN + j) 4 + h) 256 + tid_r) 16 of the slot
        // (each store instruction writes 4 KB in a row).  Buffer stores and loads keep the lane_r's offset in
        // one register and the slot and group in the scalar offset.  They
        // carry the sc1 cache bit (the bit of agent-scope atomic loads and
        // stores), so each location is coherent across the XCDs' L2 caches
        // without a whole-cache write-back or invalidate, which would also
        // evict the tiles of every other workgroup on the XCD.  The stores
        // complete (vmcnt 0) before the arrival is counted, and the last
        // arrival's loads are issued after the count is read.
        const __amdgpu_buffer_rsrc_t rp = make_rsrc(p.sk_part, (uint32_t)(SK_MAX_GRID - 1) * 256u * BN * 4u);
        const uint32_t lo = (uint32_t)tid_r * 16u;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const f32x4 v{acc[i][j][4 * h], acc[i][j][4 * h + 1], acc[i][j][4 * h + 2], acc[i][j][4 * h + 3]};
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rp, (int)lo,
                                                           (int)((uint32_t)pslot * slot_bytes +
                                                                 (uint32_t)((i * FN + j) * 4 + h) * 4096u), SC1);
                }
        __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0): this wave_r's stores are done
        __syncthreads();
        if (tid_r == 0) *s_last = atomicAdd(p.sk_cnt + MODE * SK_MAX_GRID + ctr, 1) == nseg - 1;
        __syncthreads();
        if (!*s_last) return;
        // the last arrival: the tile is the sum of its pieces in K order
        // (piece j in slot j * sstride + ctr).  Every group reads SK_SPLIT
        // pieces without a branch, so that the loads of many groups are in
        // flight together: the pieces past nseg have a lane_r offset past the
        // buffer (the range check covers the lane_r offset) and read as
        // zeros, and adding them leaves the sum as it is (up to the sign of
        // a zero).
        uint32_t pbase[SK_SPLIT], plo[SK_SPLIT];
#pragma unroll
        for (int sg = 0; sg < SK_SPLIT; ++sg) {
            pbase[sg] = sg < nseg ? (uint32_t)(pslot0 + sg * sstride) * slot_bytes : 0u;
            plo[sg] = sg < nseg ? lo : OOR;
        }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const uint32_t go = (uint32_t)((i * FN + j) * 4 + h) * 4096u;
                    f32x4 pv[SK_SPLIT];
#pragma unroll
                    for (int sg = 0; sg < SK_SPLIT; ++sg) {
                        const uint32_t vo = plo[sg];
                        pv[sg] = __builtin_bit_cast(
                            f32x4, __builtin_amdgcn_raw_buffer_load_b128(rp, (int)vo, (int)(pbase[sg] + go), SC1));
                    }
                    f32x4 v = pv[0];
#pragma unroll
                    for (int sg = 1; sg < SK_SPLIT; ++sg) v += pv[sg];
                    acc[i][j][4 * h] = v[0];
                    acc[i][j][4 * h + 1] = v[1];
                    acc[i][j][4 * h + 2] = v[2];
                    acc[i][j][4 * h + 3] = v[3];
                }
    }

    // epilogue: element e of a 32x32 block is row (e/4)*8 + (lane_r/32)*4 + e%4,
    // column lane_r%32.  Down scales each row by its gate weight, parked in
    // LDS by the workgroup (in sB2, idle since the barrier after the K loop; the
    // previous tile's reads precede this tile's K-loop barriers).
    if constexpr (MODE == 1) {
        if (tid_r < BM) s_roww[tid_r] = roww;
        __syncthreads();     // (waits for the write, which the bare barrier does not; no load is in flight)
    }
    const int rbase = L.m0 + wm_r * WM + (lane_r >> 5) * 4;
    if constexpr (MODE == 0) {
        __bf16* out = shared ? (__bf16*)p.Os : (__bf16*)p.Or;
        const int ldo = L.N / 2;
        const int orow0 = shared ? 0 : L.rowbase;
        const int cbase = (L.n0 + wn_r * WN) / 2 + (lane_r & 31);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = rbase + i * 32 + (e >> 2) * 8 + (e & 3);
                if (row < L.R) {
#pragma unroll
                    for (int q = 0; q < FN / 2; ++q) {
                        const float gv = acc[i][2 * q][e], uv = acc[i][2 * q + 1][e];
                        out[(size_t)(orow0 + row) * ldo + cbase + q * 32] = (__bf16)(silu_f(gv) * uv);
                    }
                }
            }
    } else {
        __bf16* out = (__bf16*)p.Or;
        const int ldo = L.N;
        const int cbase = L.n0 + wn_r * WN + (lane_r & 31);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = rbase + i * 32 + (e >> 2) * 8 + (e & 3);
                const float wr = s_roww[row - L.m0];
                if (row < L.R) {
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        out[(size_t)(L.rowbase + row) * ldo + cbase + j * 32] = (__bf16)(acc[i][j][e] * wr);
                }
            }
    }
}

// The persistent kernel: every workgroup walks the published work list, whole
// rounds of items in snake order (odd rounds reversed), then the items left
// over, cut along K where the list says so.  What bounds it is the weight stream
// (few rows per expert) or the MFMA rate at the card's power limit (many).  Tile
// heights follow the row counts: with 256-row (down: 192) tiles alone an expert
// of 12 rows cost as much as one of 256.  Gate/up, down before and now: 8 experts
// of 77 rows and 512 shared rows of d = 2048, f = 1408: 49 and 48 -> 40 and 30 us;
// 15 of 12 and 126 shared: 51 and 65 -> 44 and 35; 32 of 43 rows of d = 4096,
// f = 1536: 178 and 94 -> 132 and 82; 2 of 1119 of d = 4096, f = 14336: even.
template <int MODE>
__global__ void __launch_bounds__(256, 1) ggemm_bf16(const GemmArgs p) {
    __shared__ __attribute__((aligned(16))) __bf16 sA0[256 * 64], sA1[256 * 64], sB0[TP_BN * 64], sB1[TP_BN * 64];
    __shared__ __attribute__((aligned(16))) __bf16 sB2[TP_BN * 64];
    const TilePlan* P = p.plan;
    const int grid = (int)gridDim.x;                // a multiple of 8, at most SK_MAX_GRID
    const int vid = (blockIdx.x & 7) * (grid >> 3) + (blockIdx.x >> 3);
    const int H = P->H, rounds = P->rounds, items = P->items, sp0 = P->sp0, split = P->split, q = P->q, nsh = P->nsh;
    const bool spread = P->spread != 0;
    const uint32_t slot_bytes = (uint32_t)H * 64u * TP_BN * 4u;
    const int head = rounds * grid, whole = sp0 - head, ns = items - sp0;
    const TileSeg Ssh = P->seg[p.n_routed];         // the shared group
    for (int r = 0; r <= rounds; ++r) {
        const int pos = round_pos(vid, r, r < rounds ? grid : whole + split * ns, grid, spread);
        if (pos < 0) break;
        int item = r * grid + pos, lj = 0;
        const bool cut = r == rounds && split > 1 && pos >= whole;
        if (cut) {
            lj = (pos - whole) / ns;                             // K piece of a left-over item
            item = sp0 + (pos - whole) - lj * ns;
        }
        // the group of the item: lane g reads routed group g's segment (again for every
        // tile: held across the K loop it would spill), and the last one that starts at or
        // before the item is it (an empty group starts where the next one does)
        const int lane = threadIdx.x & 63, n = p.n_routed;
        const TileSeg V = P->seg[lane < n ? lane : n];
        const bool shared = item < nsh * q;
        int g = n, mt_hl = Ssh.mt_hl, t = item - Ssh.first;
        TileLoc L;
        L.R = Ssh.R;
        L.rowbase = Ssh.off;
        if (!shared) {
            g = 63 - __builtin_clzll(__builtin_amdgcn_ballot_w64(lane < n && V.first <= item));
            mt_hl = __builtin_amdgcn_readlane(V.mt_hl, g);
            t = item - __builtin_amdgcn_readlane(V.first, g);
            L.R = __builtin_amdgcn_readlane(V.R, g);
            L.rowbase = __builtin_amdgcn_readlane(V.off, g);
        }
        L.g = g;
        L.N = shared ? p.Ns : p.Nr;
        L.K = shared ? p.Ks : p.Kr;
        const int mt = mt_hl >> 3;
        const int units = L.K / 128;                             // K in steps of two K tiles
        int kt_lo = 0, kt_hi = 2 * units, nseg = 1, ctr = 0, pslot = 0, pslot0 = 0, sstride = 0;
        if (shared && q > 1) {
            const int j = t / nsh;
            t -= j * nsh;
            nseg = q;
            ctr = pslot0 = t;
            sstride = nsh;
            pslot = t + j * nsh;
            kt_lo = 2 * (j * units / q);
            kt_hi = 2 * ((j + 1) * units / q);
        } else if (cut) {
            // (shared pieces have the first slots and counters)
            nseg = split;
            ctr = (q > 1 ? nsh : 0) + item - sp0;
            sstride = ns;
            pslot0 = (q > 1 ? nsh * q : 0) + item - sp0;
            pslot = pslot0 + lj * ns;
            kt_lo = 2 * (lj * units / split);
            kt_hi = 2 * ((lj + 1) * units / split);
        }
        const int ni = t / mt, mi = t - ni * mt;
        L.n0 = ni * TP_BN;
        L.m0 = mi * H * 64;
        const int h = mi == mt - 1 ? mt_hl & 7 : H;
        if constexpr (MODE == 0) {
            // weights that one short row tile reads, of a layer that outgrows the
            // caches: non-temporal, as in the thin GEMM (GemmArgs::stream)
            if (p.stream && mt == 1 && h <= 2) {
                if (h == 2) bf16_tile<128, MODE, NT>(p, L, kt_lo, kt_hi, nseg, ctr, pslot, pslot0, sstride, slot_bytes, sA0, sA1, sB0, sB1, sB2);
                else bf16_tile<64, MODE, NT>(p, L, kt_lo, kt_hi, nseg, ctr, pslot, pslot0, sstride, slot_bytes, sA0, sA1, sB0, sB1, sB2);
                continue;
            }
        }
        if (h == 4) bf16_tile<256, MODE>(p, L, kt_lo, kt_hi, nseg, ctr, pslot, pslot0, sstride, slot_bytes, sA0, sA1, sB0, sB1, sB2);
        else if (h == 3) bf16_tile<192, MODE>(p, L, kt_lo, kt_hi, nseg, ctr, pslot, pslot0, sstride, slot_bytes, sA0, sA1, sB0, sB1, sB2);
        else if (h == 2) bf16_tile<128, MODE>(p, L, kt_lo, kt_hi, nseg, ctr, pslot, pslot0, sstride, slot_bytes, sA0, sA1, sB0, sB1, sB2);
        else bf16_tile<64, MODE>(p, L, kt_lo, kt_hi, nseg, ctr, pslot, pslot0, sstride, slot_bytes, sA0, sA1, sB0, sB1, sB2);
    }
}

// Thin grouped GEMM for small batches (decode): a few rows per expert, so the
// time is the weight stream from HBM and the MFMA work is incidental.  A
// workgroup computes 32 rows x 64 weight rows (a gate/up granule pair, or 64
// output columns of the down projection) over the whole K.  Its 4 waves take
// interleaved K steps of 64 (wave w: steps w, w+4, ...), so the workgroup
// streams 512 contiguous bytes of each weight row per round.  The weight rows
// are read coalesced (a wave instruction covers 8 rows x 128 bytes, whole cache
// lines) into registers, passed through the wave's own LDS rows (padded by 16
// bytes) into the v_mfma_f32_32x32x16_bf16 layout (lane: row lane%32, K
// elements 8*(lane/32) .. +7 of each 16); the activation rows go from global
// memory straight into MFMA registers.  Two register sets keep the next step's
// reads in flight during the current step.  The waves' partial sums meet in LDS
// and are added in wave order, then the epilogue of ggemm_bf16 runs on the
// sums.  The weights of an expert of at most 32 rows are read exactly once, in a
// layer of STREAM_BYTES or more with non-temporal loads: those stream at 7.0 TB/s
// here, ordinary ones at 6.2 (64 tokens, 30 experts of d = 4096, f = 1536: layer
// 245 -> 225 us; one token 58 -> 55 us).  With more row tiles the tiles after the
// first find the weights in L2, which non-temporal loads would forfeit (2 x 35 rows
// of d = 4096, f = 14336: 205 -> 231 us), so those keep ordinary loads.
constexpr int TH_BM = 32, TH_BN = 64, TH_WAVES = 4;
constexpr int TH_LDK = 144;                        // bytes per staged weight row
constexpr int TH_LDS = TH_WAVES * TH_BN * TH_LDK;  // staging; reused for the partial sums

template <int MODE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
ggemm_thin(const GemmArgs p) {
    __shared__ __attribute__((aligned(16))) char th_lds[TH_LDS];
    static_assert(sizeof(float) * TH_WAVES * 2 * 16 * 64 <= TH_LDS, "partial sums fit the staging rows");
    float (*red)[2][16][64] = (float (*)[2][16][64])th_lds;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: K offsets go in SGPRs
    const int c = lane & 31, h = lane >> 5;
    const int total = *p.ntiles;
    const int per_xcd = gridDim.x >> 3;
    const int vid = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    constexpr uint32_t OOR = 0x80000000u;

    // rounds of gridDim.x tiles; the last, partial round shared evenly by the
    // XCDs when every tile has the same K
    const bool spread = !(p.G > p.n_routed && p.Ks != p.Kr);
    const GroupScan gs = scan_groups<TH_BM, TH_BN>(p, lane);
    for (int r = 0; r * (int)gridDim.x < total; ++r) {
        const int n = total - r * (int)gridDim.x;
        const int pos = round_pos(vid, 0, n, (int)gridDim.x, spread);
        if (pos < 0) break;
        const int tile = r * (int)gridDim.x + pos;
        TileLoc L;
        if (!find_tile<TH_BM, TH_BN>(p, gs, tile, lane, L)) break;
        const bool shared = L.g >= p.n_routed;
        const int K = L.K;
        const __bf16* Bw = shared ? (const __bf16*)p.Ws
                                  : (const __bf16*)p.Wr + (size_t)L.g * L.N * K;
        const __amdgpu_buffer_rsrc_t rb_rs = make_rsrc(Bw, (uint32_t)((size_t)L.N * K * 2));
        // weight reads from the blocked layout: the tile's 64 rows of one K step
        // are 8 KB in a row; lane l takes row 8i + l/8, 16-byte chunk l%8 of
        // that row's 128 bytes, and the K step goes in the scalar offset
        const uint32_t wblk0 = (uint32_t)(L.n0 / WB_ROWS) * (uint32_t)(K / WB_K) * (uint32_t)(WB_ROWS * WB_K * 2) +
                               (uint32_t)((L.n0 % WB_ROWS) + (lane >> 3)) * (WB_K * 2u) + (uint32_t)(lane & 7) * 16u;
        char* stg = th_lds + wave * (TH_BN * TH_LDK);
        char* wdst = stg + (lane >> 3) * TH_LDK + (lane & 7) * 16;
        const char* frag = stg + c * TH_LDK + h * 16;                  // row c, chunk 2i + h
        const int row = L.m0 + c;
        __amdgpu_buffer_rsrc_t ra_rs;
        uint32_t aoff;
        if (MODE == 0) {
            ra_rs = make_rsrc(p.X, p.x_bytes);
            aoff = row < L.R ? ((uint32_t)p.row_tok[L.rowbase + row] * (uint32_t)p.ldx + 8u * h) * 2u : OOR;
        } else {
            const __bf16* Ab = shared ? (const __bf16*)p.As : (const __bf16*)p.Ar + (size_t)L.rowbase * K;
            ra_rs = make_rsrc(Ab, (uint32_t)((size_t)L.R * K * 2));
            aoff = row < L.R ? ((uint32_t)row * (uint32_t)K + 8u * h) * 2u : OOR;
        }
        const int KS = K / 64;
        const int nst = (KS - wave + TH_WAVES - 1) / TH_WAVES;   // steps of this wave

        f32x16 acc0, acc1;
#pragma unroll
        for (int e = 0; e < 16; ++e) { acc0[e] = 0.f; acc1[e] = 0.f; }
        bf16x8 w[2][8], a[2][4];
        // weights that one row tile reads are read once: non-temporal where the
        // layer outgrows the caches
        const bool once = p.stream && L.R <= TH_BM;
        auto load = [&](auto nt, int buf, int it) {
            constexpr int AUX = decltype(nt)::value;
            const int st = wave + it * TH_WAVES;
            // a step past the end reads zeros through the range check and adds nothing
            const uint32_t ok = it < nst ? 0u : OOR;
            const uint32_t k0 = (uint32_t)st * 128u;   // bytes into a token or activation row
            const uint32_t kb = (uint32_t)st * (uint32_t)(WB_ROWS * WB_K * 2);   // bytes into the weight blocks
#pragma unroll
            for (int i = 0; i < 8; ++i) w[buf][i] = buf_load16<AUX>(rb_rs, (wblk0 + i * 1024u) | ok, kb);
#pragma unroll
            for (int i = 0; i < 4; ++i) a[buf][i] = buf_load16(ra_rs, aoff | ok, k0 + 32u * i);
        };
        auto mma = [&](int buf) {
            // the wave's own LDS rows: stores, then fragment reads, in program order
#pragma unroll
            for (int i = 0; i < 8; ++i) *(bf16x8*)(wdst + i * 8 * TH_LDK) = w[buf][i];
            bf16x8 b0[4], b1[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                b0[i] = *(const bf16x8*)(frag + i * 32);
                b1[i] = *(const bf16x8*)(frag + 32 * TH_LDK + i * 32);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[buf][i], b0[i], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[buf][i], b1[i], acc1, 0, 0, 0);
            }
        };
        auto kloop = [&](auto nt) __attribute__((always_inline)) {
            load(nt, 0, 0);
            for (int it = 0; it < nst; it += 2) {
                load(nt, 1, it + 1);
                __builtin_amdgcn_sched_barrier(0);
                mma(0);
                __builtin_amdgcn_sched_barrier(0);
                load(nt, 0, it + 2);
                __builtin_amdgcn_sched_barrier(0);
                mma(1);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (once) kloop(std::integral_constant<int, NT>{});
        else kloop(std::integral_constant<int, 0>{});
        __syncthreads();     // every wave is done with its staging rows
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            red[wave][0][e][lane] = acc0[e];
            red[wave][1][e][lane] = acc1[e];
        }
        __syncthreads();
        // element e of lane l in a 32x32 block: row (e/4)*8 + (l/32)*4 + e%4, column l%32
        if (MODE == 0) {
            __bf16* out = shared ? (__bf16*)p.Os : (__bf16*)p.Or;
            const int ldo = L.N / 2;
            const int orow0 = shared ? 0 : L.rowbase;
            const int col = tid & 31, rg = tid >> 5;
            const int ln = col + 32 * (rg >> 2);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = rg + 8 * i;            // row inside the tile
                const int e = 4 * i + (rg & 3);
                float gv = 0.f, uv = 0.f;
#pragma unroll
                for (int w = 0; w < TH_WAVES; ++w) { gv += red[w][0][e][ln]; uv += red[w][1][e][ln]; }
                if (L.m0 + r < L.R)
                    out[(size_t)(orow0 + L.m0 + r) * ldo + L.n0 / 2 + col] = (__bf16)(silu_f(gv) * uv);
            }
        } else {
            __bf16* out = (__bf16*)p.Or;
            const int ldo = L.N;
            const int col = tid & 63, rg = tid >> 6;
            const int j = col >> 5, cl = col & 31;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int r = rg + 4 * i;
                const int e = 4 * (r >> 3) + (r & 3);
                const int ln = cl + 32 * ((r >> 2) & 1);
                float v = 0.f;
#pragma unroll
                for (int w = 0; w < TH_WAVES; ++w) v += red[w][j][e][ln];
                if (L.m0 + r < L.R) {
                    const float wr = p.row_w[L.rowbase + L.m0 + r];
                    out[(size_t)(L.rowbase + L.m0 + r) * ldo + L.n0 + col] = (__bf16)(v * wr);
                }
            }
        }
        __syncthreads();
    }
}

// fp32 storage: C = A B^T per tile of BM x 64 by v_mfma_f32_32x32x2_f32, whose
// products and sums are the fp32 FMA's.  4 waves: BM / 32 row blocks x 2 column
// blocks of 32 x KW slices of K, so a tile occupies all four matrix units of a
// CU whatever its height; the slices' sums meet in LDS and are added in slice
// order.  A K step is KW slices of 32 floats; the rows of a slice (128 bytes)
// go from memory straight into LDS with the 16-byte chunks permuted as in
// ggemm_bf16, three buffers, the loads of a step issued two steps ahead.  A
// fragment read is 16 bytes: chunk 2 q + lane / 32 holds the K values 8 q + 4
// (lane / 32) .. +3 of its row, which feed four MFMAs.  Two workgroups share a
// CU, so that one's fragment reads and epilogue run beside the other's MFMAs.
// Two shapes: 64-row tiles, and 32-row tiles with two K slices when the 64-row
// tiles would leave CUs without work (fewer than F32_TALL_TILES in all); the
// choice is made here, from the row counts on the device.  What bounds it is
// the fp32 matrix rate (157 TFLOP/s) at many rows, and at a few hundred rows
// the length of one tile's K loop.  Measured against 64 x 64 tiles of scalar
// loads and vector FMAs: 290 rows, d = 512, f = 1024: gate/up 59 -> 15 us, down
// 145 -> 14 us; 641 rows, d = 1024, f = 640: 131 -> 26 and 98 -> 19 us.
constexpr int F32_BM = 64, F32_BN = 64, F32_THREADS = 256, F32_PER_CU = 2;
constexpr int F32_TALL_TILES = 512;
constexpr int F32_BUF = 2 * (32 + 64) * 32;         // floats of one buffer: the 32-row shape's two slices

template <int MODE, int BM, int KW>
__device__ inline void f32_tiles(const GemmArgs& p, float* b0, float* b1, float* b2) {
    constexpr int WPS = BM / 32 * 2;                // waves per K slice
    constexpr int AV = BM / 8 / WPS, BV = F32_BN / 8 / WPS;   // 8-row load instructions per wave and step
    constexpr int SLICE = (BM + F32_BN) * 32;       // floats of one K slice in a buffer
    static_assert(WPS * KW == F32_THREADS / 64 && SLICE * KW <= F32_BUF, "four waves, one buffer");
    static_assert(F32_THREADS / 64 * 16 * 64 <= F32_BUF, "the waves' sums fit a buffer");
    constexpr uint32_t OOR = 0x80000000u;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = wave / WPS, ws = wave % WPS;     // K slice, wave inside it
    const int wm = ws >> 1, wn = ws & 1;
    const int grid = (int)gridDim.x;                // a multiple of 8
    const int vid = (blockIdx.x & 7) * (grid >> 3) + (blockIdx.x >> 3);
    const int rsub = lane >> 3;
    const GroupScan gs = scan_groups<BM, F32_BN>(p, lane);
    for (int tile = vid;; tile += grid) {
        TileLoc L;
        if (!find_tile<BM, F32_BN>(p, gs, tile, lane, L)) break;
        const bool shared = L.g >= p.n_routed;
        const int K = L.K;
        const float* Bw = shared ? (const float*)p.Ws : (const float*)p.Wr + (size_t)L.g * L.N * K;
        const float* Ab = MODE == 0 ? (const float*)p.X
                                    : (shared ? (const float*)p.As : (const float*)p.Ar + (size_t)L.rowbase * K);
        const __amdgpu_buffer_rsrc_t rb_rs = make_rsrc(Bw, (uint32_t)((size_t)L.N * K * 4));
        const __amdgpu_buffer_rsrc_t ra_rs = make_rsrc(Ab, MODE == 0 ? p.x_bytes : (uint32_t)((size_t)L.R * K * 4));
        uint32_t aoff[AV], boff[BV];
#pragma unroll
        for (int v = 0; v < AV; ++v) {
            const int r = (ws * AV + v) * 8 + rsub, row = L.m0 + r;
            const uint32_t src = MODE == 0 ? (row < L.R ? (uint32_t)p.row_tok[L.rowbase + row] : 0u) : (uint32_t)row;
            const uint32_t ch = (lane & 7) ^ ((r >> 1) & 7);
            aoff[v] = row < L.R ? (src * (uint32_t)(MODE == 0 ? p.ldx : K) + ch * 4) * 4u : OOR;
        }
#pragma unroll
        for (int v = 0; v < BV; ++v) {
            const int r = (ws * BV + v) * 8 + rsub;
            const uint32_t ch = (lane & 7) ^ ((r >> 1) & 7);
            boff[v] = ((uint32_t)(L.n0 + r) * (uint32_t)K + ch * 4) * 4u;
        }
        const int nslices = K / 32, nsteps = (nslices + KW - 1) / KW;
        // the loads of this wave's share of K step st into buffer b (slices past K: zeros)
        auto issue = [&](float* b, int st) {
            const int sl = st * KW + ks;
            const uint32_t past = sl < nslices ? 0u : OOR, so = sl < nslices ? (uint32_t)sl * 128u : 0u;
            float* d = b + ks * SLICE;
#pragma unroll
            for (int v = 0; v < AV; ++v) {
                const uint32_t vo = aoff[v] | past;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ra_rs, (lds_ptr)(d + (ws * AV + v) * 8 * 32), 16, vo, so, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < BV; ++v) {
                const uint32_t vo = boff[v] | past;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rb_rs, (lds_ptr)(d + BM * 32 + (ws * BV + v) * 8 * 32), 16, vo,
                                                         so, 0, 0);
            }
        };
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.f;
        const int fa = (wm * 32 + (lane & 31)) * 32, fb = (BM + wn * 32 + (lane & 31)) * 32;
        auto mma = [&](const float* b) {
            const float* d = b + ks * SLICE;
            f32x4 av[4], bv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ch = ((2 * q + (lane >> 5)) ^ ((lane >> 1) & 7)) * 4;   // row & 31 = lane & 31
                av[q] = *(const f32x4*)(d + fa + ch);
                bv[q] = *(const f32x4*)(d + fb + ch);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[q][j], bv[q][j], acc, 0, 0, 0);
        };
        // step st: its loads have arrived (the younger step's may be in flight),
        // every wave is past step st - 1, whose buffer takes the loads of st + 2
        auto step = [&](float* cur, float* nxt, int st) {
            __builtin_amdgcn_s_waitcnt(waitcnt_enc(AV + BV, 0));
            lds_barrier();
            issue(nxt, st + 2);
            mma(cur);
        };
        issue(b0, 0);
        issue(b1, 1);
        int st = 0;
        for (; st + 3 <= nsteps; st += 3) {
            step(b0, b2, st);
            step(b1, b0, st + 1);
            step(b2, b1, st + 2);
        }
        if (st < nsteps) step(b0, b2, st);
        if (st + 1 < nsteps) step(b1, b0, st + 1);
        // loads past the last step may still be in flight into a buffer
        __builtin_amdgcn_s_waitcnt(waitcnt_enc(0, 0));
        lds_barrier();
        float* red = b0;                            // [4 waves][16][64]
#pragma unroll
        for (int e = 0; e < 16; ++e) red[(wave * 16 + e) * 64 + lane] = acc[e];
        __syncthreads();
        // element e of lane l of a 32 x 32 block: row (e/4)*8 + (l/32)*4 + e%4, column l%32
        auto sum = [&](int w, int e) {              // over the K slices, in order
            float v = red[(w * 16 + e) * 64 + lane];
#pragma unroll
            for (int z = 1; z < KW; ++z) v += red[((z * WPS + w) * 16 + e) * 64 + lane];
            return v;
        };
        if constexpr (MODE == 0) {
            // block 0 holds 32 gate columns, block 1 the matching up columns
            float* out = shared ? (float*)p.Os : (float*)p.Or;
            const int ldo = L.N / 2, orow0 = shared ? 0 : L.rowbase;
            for (int i = wave; i < BM / 32 * 16; i += F32_THREADS / 64) {
                const int m = i >> 4, e = i & 15;
                const int row = L.m0 + m * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
                const float gv = sum(2 * m, e), uv = sum(2 * m + 1, e);
                if (row < L.R)
                    out[(size_t)(orow0 + row) * ldo + L.n0 / 2 + (lane & 31)] =
                        gv / (1.0f + __expf(-gv)) * uv;   // fp32: IEEE divide
            }
        } else {
            float* out = (float*)p.Or;
            for (int i = wave; i < BM / 32 * 2 * 16; i += F32_THREADS / 64) {
                const int w = i >> 4, e = i & 15;
                const int row = L.m0 + (w >> 1) * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
                const float v = sum(w, e);
                if (row < L.R)
                    out[(size_t)(L.rowbase + row) * L.N + L.n0 + (w & 1) * 32 + (lane & 31)] =
                        v * p.row_w[L.rowbase + row];
            }
        }
        __syncthreads();                            // before the next tile's loads overwrite the sums
    }
}

template <int MODE>
__global__ void __launch_bounds__(F32_THREADS) ggemm_f32(const GemmArgs p) {
    __shared__ __attribute__((aligned(16))) float b0[F32_BUF], b1[F32_BUF], b2[F32_BUF];
    // (the tile count is of 64-row tiles)
    if (*p.ntiles >= F32_TALL_TILES) f32_tiles<MODE, F32_BM, 1>(p, b0, b1, b2);
    else f32_tiles<MODE, 32, 2>(p, b0, b1, b2);
}

struct CombineArgs {
    int64_t T;
    int d, stride, dtype;
    const int32_t* tok_rows;
    const void* obuf;
    void* y;
};

__global__ void __launch_bounds__(256) combine_kernel(const CombineArgs c) {
    const int64_t t = blockIdx.x;
    int rows[MAXR];
    int n = 0;
    for (int i = 0; i < c.stride; ++i) {
        const int r = c.tok_rows[t * c.stride + i];
        if (r >= 0) rows[n++] = r;
    }
    if (c.dtype == ORDERMOE_BF16) {
        const __bf16* O = (const __bf16*)c.obuf;
        __bf16* Y = (__bf16*)c.y + t * c.d;
        for (int col = threadIdx.x * 8; col < c.d; col += 256 * 8) {
            float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            for (int i = 0; i < n; ++i) {
                const bf16x8 v = *(const bf16x8*)(O + (int64_t)rows[i] * c.d + col);
#pragma unroll
                for (int q = 0; q < 8; ++q) s[q] += (float)v[q];
            }
            bf16x8 o;
#pragma unroll
            for (int q = 0; q < 8; ++q) o[q] = (__bf16)s[q];
            *(bf16x8*)(Y + col) = o;
        }
    } else {
        const float* O = (const float*)c.obuf;
        float* Y = (float*)c.y + t * c.d;
        for (int col = threadIdx.x; col < c.d; col += 256) {
            float s = 0.f;
            for (int i = 0; i < n; ++i) s += O[(int64_t)rows[i] * c.d + col];
            Y[col] = s;
        }
    }
}


// bf16 batches that take the thin GEMM, THIN_PER_CU resident workgroups per CU.
// Up to THIN_MAX_T tokens it is the safe choice whatever rows the experts get: the
// tiled one takes half as long again when the local experts get few rows (15
// experts of d = 2048, f = 1408, one row: 24 us thin, 36 tiled), the thin one at
// most twice as long when a few experts get all tokens.  With two exceptions.
// TILED_SHARED shared experts in a layer of STREAM_BYTES, above TILED_SHARED_T tokens:
// they form one group with as many times the routed K, which the thin GEMM runs whole
// and the tiled one in K pieces (thin over tiled time, three layers in turn, 33 to 128
// tokens over seven row profiles, d = 2048, f = 1408, with shared rows and without any:
// 3 shared 1.09 to 1.20 and 0.90 to 0.97; 4 shared 1.18 to 1.28 and 0.90 to 0.98, 0.63
// at a single row in all; 2 shared 1.01 to 1.09 and 0.90 to 0.98; 4 shared of d = 1024,
// f = 640, 20 MB: 0.75 to 0.91).  And where THIN_ROWS rows per expert are the mean and
// one expert's gate/up tiles fill half the chip (f >= TILED_F): 2 experts of f = 14336, 128 tokens, three layers in turn, 2 x 2, 2 x
// 32 and 2 x 128 rows: thin 136, 166 and 319 us, tiled 135, 141 and 159 (and 90 against
// 102 at a single row); f = 12288: tiled at most the time that thin takes, f = 7168: 79
// against 68 with few rows.
// Above, with a mean of at most THIN_ROWS rows per expert: a layer of less than
// STREAM_BYTES up to THIN_SMALL_T tokens, where thin is faster whatever the rows (8
// experts of d = 1024, f = 640, 140 tokens: even rows 22 against 30 us, five experts
// of 140 rows 30 and 34; 200 tokens: five of 200, 37 and 35).  In a larger one up to
// THIN_SPARSE_T tokens the rows that the experts do get decide on the device
// (group_layout): both are launched, and the one that is not wanted finds no tiles,
// which costs 5 us.  Routing that leaves few rows per expert gains (32 of 128
// experts of d = 4096, f = 1536, 140 to 320 tokens, even rows: 200 to 207 us, tiled
// alone 216 to 222), hot experts pay only these (8 of 320 rows: 149 us, thin 325,
// tiled alone 145).
constexpr int64_t THIN_MAX_T = 128, THIN_SMALL_T = 160, THIN_SPARSE_T = 512;
constexpr int THIN_ROWS = 20, TILED_F = 12288, TILED_SHARED = 3, TILED_SHARED_T = 32;
// Routed gate/up weights of at least this many bytes are streamed with non-temporal
// loads by short single row tiles and by the thin GEMM.  Tiled gate/up: 805 MB (32
// experts of d = 4096, f = 1536) 148 -> 131 us, 92 MB (8 of d = 2048, f = 1408)
// 53 -> 49 us; smaller ones are found in the caches by the next call, which such
// loads forfeit: 21 MB (8 of d = 1024, f = 640) 15 -> 19 us.  Thin, the whole layer
// at 4 and 64 tokens: over three layers in turn 92 MB and 173 MB (15 of d = 2048,
// f = 1408) 2 to 5% faster, 21 MB 5 to 8% slower; over one layer of 92 MB again and
// again, which then stays in the caches, 6% slower.  (In the tiled down GEMM the
// further tile variants spilled: 78 -> 85 us at the first shape; it keeps ordinary
// loads.)
constexpr int64_t STREAM_BYTES = 64 << 20;
constexpr int THIN_PER_CU = 3;

int persistent_grid(int64_t upper_tiles, int per_cu) {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) cus = v;
    }
    int64_t g = (int64_t)cus * per_cu;
    if (upper_tiles < g) g = upper_tiles;
    g = (g + 7) & ~int64_t(7);
    return (int)(g < 8 ? 8 : g);
}

// grid of a bf16 GEMM launch: up to SK_SPLIT workgroups per tile (the split
// tiles are shared out over them), at most SK_MAX_GRID
int bf16_grid(int64_t upper_tiles) {
    const int g = persistent_grid((int64_t)SK_SPLIT * upper_tiles, 1);
    return g < SK_MAX_GRID ? g : SK_MAX_GRID;
}

}  // namespace

size_t forward_split_counters() { return 2 * SK_MAX_GRID; }

size_t forward_split_floats(int gemms) {
    if (!(gemms & GEMM_TILED)) return 0;
    static_assert(2 * sizeof(TilePlan) <= 256 * TP_BN * sizeof(float), "the work lists fit the last slot");
    return (size_t)SK_MAX_GRID * 256 * TP_BN;
}

int forward_tokens_per_block() { return FT_TB; }

int forward_gemms(int dtype, int64_t T, int k, int E, int f, int n_shared, int64_t gu_bytes, bool room) {
    if (dtype != ORDERMOE_BF16) return 0;
    const bool few = T * k <= (int64_t)THIN_ROWS * E;
    if (T <= THIN_MAX_T) {
        const bool wide = f >= TILED_F && n_shared < 2 && !few;
        const bool shared = n_shared >= TILED_SHARED && T > TILED_SHARED_T && gu_bytes >= STREAM_BYTES;
        return (wide || shared) && room ? GEMM_TILED : GEMM_THIN;
    }
    if (!few || T > THIN_SPARSE_T || n_shared >= 2) return GEMM_TILED;
    if (gu_bytes < STREAM_BYTES) return T <= THIN_SMALL_T || !room ? GEMM_THIN : GEMM_TILED;
    return room ? GEMM_THIN | GEMM_TILED : GEMM_THIN;
}

int launch_local_forward(const ForwardArgs& f, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    const int has_sh = f.n_shared > 0 ? 1 : 0;
    const int G = f.n_local + has_sh;
    const bool thin = f.gemms & GEMM_THIN, tiled = f.gemms & GEMM_TILED;
    const int64_t rows_r = f.rmax_routed, rows_s = has_sh ? f.T : 0;
    // upper bounds of the tiles, for the grids (of the tiled bf16 GEMMs: of the shortest tiles)
    auto ub_gu = [&](int bm, int bn) {
        return ((rows_r + bm - 1) / bm + f.n_local) * (2 * f.f / bn) +
               (has_sh ? ((rows_s + bm - 1) / bm + 1) * (2 * f.n_shared * f.f / bn) : 0);
    };
    auto ub_dn = [&](int bm, int bn) { return ((rows_r + rows_s + bm - 1) / bm + G) * (f.d / bn); };
    // tiles of the GEMMs without a work list
    const int bm = thin ? TH_BM : F32_BM, bn = thin ? TH_BN : F32_BN;
    TilePlan* plan = tiled ? (TilePlan*)(f.sk_part + (size_t)(SK_MAX_GRID - 1) * 256 * TP_BN) : nullptr;

    RowsArgs r;
    r.T = f.T; r.k = f.k; r.E = f.E; r.n_local = f.n_local; r.has_shared = has_sh; r.server = f.server;
    r.w = f.w; r.exec_k = f.exec_k; r.exec_m = f.exec_m; r.loc_in = f.loc_in;
    for (int i = 0; i < ORDERMOE_MAX_EXPERTS; ++i) r.lidx[i] = f.lidx[i];
    r.blk_rows = f.blk_rows; r.row_offsets = f.row_offsets;
    r.row_tok = f.row_tok; r.row_w = f.row_w; r.tok_rows = f.tok_rows; r.tile_info = f.tile_info;
    r.sk_cnt = f.sk_cnt; r.nblk = f.nblk;
    r.bm_gu = r.bm_dn = bm; r.bn_gu = r.bn_dn = bn;
    r.n_gu_r = 2 * f.f; r.n_gu_s = 2 * f.n_shared * f.f; r.n_dn = f.d;
    r.plan = plan;
    r.choose = thin && tiled;
    for (int w = 0; w < 2; ++w) {
        PlanShape& c = r.shape[w];
        c.nt_r = (w == 0 ? r.n_gu_r : r.n_dn) / TP_BN;
        c.nt_s = (w == 0 ? r.n_gu_s : r.n_dn) / TP_BN;
        c.kt_r = (w == 0 ? f.d : f.f) / 64;
        c.kt_s = (w == 0 ? f.d : f.n_shared * f.f) / 64;
        c.q = has_sh && c.kt_s >= 2 * c.kt_r ? (c.kt_s / c.kt_r < SK_SPLIT ? c.kt_s / c.kt_r : SK_SPLIT) : 1;
        c.grid = bf16_grid(w == 0 ? ub_gu(64, TP_BN) : ub_dn(64, TP_BN));
        c.grid_inv = (uint32_t)(((1ull << 32) + c.grid - 1) / c.grid);
    }

    hipError_t e;
    if (f.T <= SCAN_THREADS) {
        {
            KernelTimer kt_("rows_small", st);
            hipLaunchKernelGGL(rows_small_kernel, dim3(1), dim3(SCAN_THREADS), 0, st, r);
        }
        if ((e = hipGetLastError()) != hipSuccess) return (int)e;
        if (f.nblk == 0) return 0;
    } else {
        {
            KernelTimer kt_("rows_count", st);
            hipLaunchKernelGGL(rows_count_kernel, dim3(f.nblk), dim3(FT_TB), 0, st, r);
        }
        if ((e = hipGetLastError()) != hipSuccess) return (int)e;
        {
            KernelTimer kt_("rows_scatter", st);
            hipLaunchKernelGGL(rows_scatter_kernel, dim3(f.nblk + (plan ? 1 : 0)), dim3(FT_TB), 0, st, r);
        }
        if ((e = hipGetLastError()) != hipSuccess) return (int)e;
    }

    GemmArgs g{};
    g.offsets = f.row_offsets; g.G = G; g.n_routed = f.n_local;
    g.X = f.x; g.row_tok = f.row_tok; g.ldx = f.d; g.row_w = f.row_w;
    g.x_bytes = (uint32_t)((size_t)f.T * f.d * (f.dtype == ORDERMOE_BF16 ? 2 : 4));
    g.sk_part = f.sk_part; g.sk_cnt = f.sk_cnt;
    g.stream = (int64_t)f.n_local * 2 * f.f * f.d * 2 >= STREAM_BYTES;

    // gate/up: [rows][d] x [2f][d]^T -> activations [rows][f]
    g.ntiles = f.tile_info + 0;
    g.Nr = 2 * f.f; g.Kr = f.d; g.Ns = 2 * f.n_shared * f.f; g.Ks = f.d;
    g.Wr = f.w_gu; g.Ws = f.w_sh_gu; g.Ar = nullptr; g.As = nullptr; g.Or = f.act_r; g.Os = f.act_s;
    {
        KernelTimer kt_("gemm_gate_up", st);
        if (thin) ggemm_thin<0><<<dim3(persistent_grid(ub_gu(bm, bn), THIN_PER_CU)), dim3(256), 0, st>>>(g);
        if (tiled) {
            g.plan = plan;
            ggemm_bf16<0><<<dim3(r.shape[0].grid), dim3(256), 0, st>>>(g);
        }
        if (!f.gemms) ggemm_f32<0><<<dim3(persistent_grid(2 * ub_gu(bm, bn), F32_PER_CU)), dim3(F32_THREADS), 0, st>>>(g);
    }
    if ((e = hipGetLastError()) != hipSuccess) return (int)e;

    // down: activations [rows][f] x [d][f]^T -> row outputs [rows][d], scaled by the gate
    g.ntiles = f.tile_info + 1;
    g.Nr = f.d; g.Kr = f.f; g.Ns = f.d; g.Ks = f.n_shared * f.f;
    g.Wr = f.w_dn; g.Ws = f.w_sh_dn; g.Ar = f.act_r; g.As = f.act_s; g.Or = f.obuf; g.Os = nullptr;
    {
        KernelTimer kt_("gemm_down", st);
        if (thin) ggemm_thin<1><<<dim3(persistent_grid(ub_dn(bm, bn), THIN_PER_CU)), dim3(256), 0, st>>>(g);
        if (tiled) {
            g.plan = plan + 1;
            ggemm_bf16<1><<<dim3(r.shape[1].grid), dim3(256), 0, st>>>(g);
        }
        if (!f.gemms) ggemm_f32<1><<<dim3(persistent_grid(2 * ub_dn(bm, bn), F32_PER_CU)), dim3(F32_THREADS), 0, st>>>(g);
    }
    if ((e = hipGetLastError()) != hipSuccess) return (int)e;

    CombineArgs c;
    c.T = f.T; c.d = f.d; c.stride = f.k + 1; c.dtype = f.dtype; c.tok_rows = f.tok_rows;
    c.obuf = f.obuf; c.y = f.y;
    {
        KernelTimer kt_("combine", st);
        hipLaunchKernelGGL(combine_kernel, dim3((unsigned)f.T), dim3(256), 0, st, c);
        }
    if ((e = hipGetLastError()) != hipSuccess) return (int)e;
    return 0;
}

static int launch_pack(int dtype, int n, int rows, int K, bool gate_up, const void* a, const void* b, void* out,
                       void* stream) {
    const int64_t nr = (int64_t)n * rows;
    if (nr == 0) return 0;
    hipStream_t st = (hipStream_t)stream;
    if (dtype == ORDERMOE_BF16) {                      // rows are a multiple of 256 here
        pack_bf16_kernel<<<dim3((unsigned)(nr / 8)), PK_THREADS, 0, st>>>(rows, K, gate_up, (const __bf16*)a,
                                                                          (const __bf16*)b, (__bf16*)out);
    } else {
        pack_f32_kernel<<<dim3((unsigned)nr), PK_THREADS, 0, st>>>(rows, K, gate_up, (const float*)a, (const float*)b,
                                                                   (float*)out);
    }
    return (int)hipGetLastError();
}

int launch_pack_gate_up(int dtype, int n, int f, int d, const void* g, const void* u, void* out, void* stream) {
    return launch_pack(dtype, n, 2 * f, d, true, g, u, out, stream);
}

int launch_pack_down(int dtype, int n, int d, int f, const void* w, void* out, void* stream) {
    return launch_pack(dtype, n, d, f, false, w, nullptr, out, stream);
}

}  // namespace ordermoe
