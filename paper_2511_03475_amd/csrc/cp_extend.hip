// cp_extend: prefix-cached "extend" prefill attention over a paged KV cache for gfx950.
//
// Kernels behind the C ABI of cp_extend.h:
//   write_kv_kernel       cache append (paper, Section 1: the prefix cache stores prior K/V)
//   extend_attn_kernel    suffix rows attend to cached prefix pages + their own K/V
//                         (paper, Section 1 / Section 2.1: prefill over a prefix cache); in batches of
//                         unequal lengths also the decode-shaped requests, next to the others
//   decode_attn_kernel    the same for calls with few rows per KV head or few keys (wavefronts share the keys)
//   merge_splits_kernel, merge_few_splits_kernel, merge_tail_kernel, merge_mixed_kernel   combine partial results over key ranges
//   check_tables_kernel   optional check of block_table against the pool size
//
// Attention kernel layout.  One workgroup = 8 wavefronts = 256 (token, q head) rows of one KV
// head; each wavefront owns 32 rows.  Keys are streamed in tiles of 64 through LDS.  Scores are computed
// transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16 so that the accumulator lane
// (lane % 32) is a query row: the softmax row reductions are then in-lane plus one exchange
// between the two half-waves, the bf16 probabilities already sit in the B-operand layout of the
// second product O^T = V^T P^T, and the per-row rescale of O is a per-lane scalar multiply.
// V^T fragments come from LDS through the transposing read ds_read_b64_tr_b16.  The K/V tiles
// reach LDS by direct loads (global_load_lds_dwordx4), without a pass through registers.  The
// query fragments carry softmax_scale * log2(e), rounded to bf16 once per row, so that the
// accumulators of S^T are the arguments of exp2 as they stand.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>
#include <type_traits>
#include <vector>

#include "cp_extend.h"

namespace {

constexpr int kD = 128;       // head dim
constexpr int kPS = 16;       // tokens per page
constexpr int kBM = 256;      // query rows per workgroup, at most
constexpr int kTileShift = 8; // its logarithm
constexpr int kBN = 64;       // keys per tile
constexpr int kThreads = 512; // 8 wavefronts
constexpr int kXcds = 8;      // accelerator complex dies; workgroup ids round-robin over them
constexpr int kMaxSplits = 64;
constexpr int kWaves = kThreads / 64;
constexpr int kNKB = kBN / 32;            // 32-key blocks per tile
constexpr int kLoadRows = kWaves * 4;     // key rows one load step of the workgroup covers
static_assert(kBM == kWaves * 32 && kBM == 1 << kTileShift && kBN == 2 * kLoadRows, "tile shape");

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

struct AttnParams {
    const uint16_t *q;
    const uint16_t *k_new;
    const uint16_t *v_new;
    const uint16_t *kv_pages;
    const int32_t *block_table;
    const int32_t *prefix_lens;
    const int32_t *extend_lens;
    uint16_t *out;
    float *part_o;  // [nsplit][T][Hq][D]   unnormalised partial outputs (mixed: [part_rows][Hq][D];
                    // tail: [Hkv][tail_units][nsplit][kBM][D])
    float *part_ml; // [nsplit][T][Hq][2]   running max (log2 domain) and sum
    int32_t batch, Hq, Hkv, G, max_pages, T;
    int32_t nsplit;
    int32_t whole_units;    // row tiles of a KV head in front of those that are split (all requests equal), else 0
    int32_t tail_units;     // ... and those that are, 0: all or none
    int32_t alternate;      // see row_tile_of
    int32_t tile_shift;     // rows of a tile: 1 << tile_shift
    int32_t dec_row_blocks; // decode kernel: blocks of 32 (head, token) rows per (request, KV head)
    int32_t items_per_head; // work items per KV head
    int32_t total_items;    // items_per_head * Hkv
    int32_t items_per_xcd;  // list positions of each XCD, see work_item
    int32_t xcds_per_head;  // XCDs that share the items of one KV head
    float scale_log2;       // softmax_scale * log2(e)
    uint32_t g_magic;       // see over_heads, 0: plain division
};
// Requests of a mixed batch: their order travels in the kernel's arguments.  Planning 512 takes the host 23 us, the call 85 if
// they are short (up to 100 cached tokens, a fifth of them with up to 60 new ones, the others with one; 32/8 heads).
constexpr int kMixedMaxBatch = 512;
struct MixedParams : AttnParams {
    int32_t seg_tiles;  // key tiles per work item of a row-tiled request, at most
    int32_t dec_blocks; // key blocks of 32 per wavefront of a decode-shaped request, at most
    uint64_t dec_share; // items of decode-shaped work among all, as a 32-bit fraction, see decode_items_before
    uint8_t order[kMixedMaxBatch]; // per group of 64 requests: which lane's request is first, second, ...
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Maximum across the two half-waves (lane l and lane l ^ 32 end with the same value).
__device__ __forceinline__ float halfwave_max(float x)
{
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float halfwave_sum(float x)
{
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The item list of a call is KV head by KV head, items_per_head each.  Consecutive workgroup ids go
// round the XCDs, and an XCD works on one KV head at a time, so that the workgroups resident on it
// stream the same K/V through its L2.  With 8 KV heads or more an XCD gets a contiguous range of the
// list.  With 1, 2 or 4 several XCDs share a head: a contiguous range each is right when that is about
// the same work for all of them (contiguous_ranges), otherwise, because the longest row tiles of a
// request come first, the head's items are dealt out one at a time (one prompt of 32768 tokens, 8/2
// heads: 2.81 -> 1.85 ms; of 8192: 211 -> 151 us).
// Position of this workgroup's item in the list, or -1.
__device__ __forceinline__ int work_item(int bid, const AttnParams &p, int &kvh)
{
    const int xcd = bid % kXcds, at = bid / kXcds;
    int item;
    if (p.xcds_per_head > 1) {
        kvh = xcd / p.xcds_per_head;
        item = at * p.xcds_per_head + xcd % p.xcds_per_head;
        return item < p.items_per_head ? item : -1;
    }
    item = xcd * p.items_per_xcd + at;
    if (item >= p.total_items) return -1;
    kvh = item / p.items_per_head;
    return item - kvh * p.items_per_head;
}

// n / G: a multiplication where the host says that it is exact for every row of the call, (n + 1) G <= 2^32 with
// g_magic = floor((2^32 - 1) / G).  A division by a number that the compiler does not know takes some 40
// instructions, and an item starts with four of them.
__device__ __forceinline__ int over_heads(int n, const AttnParams &p)
{
    return p.g_magic ? (int)__umulhi((uint32_t)n + 1u, p.g_magic) : n / p.G;
}
// Row tiles of one request for one KV head: its E x G (token, q head) rows, token by token and within a token
// head by head, are cut into tiles of 1 << shift.  So only a request's last tile can hold padding, whatever E and G are,
// all rows of a tile end at about the same key, and the rows of a token lie side by side in q and out.  Before, a tile
// took rows of 1, 2, 4 or 8 whole heads: 9 requests, P = 190, E = 190, 32/8 heads (36 tiles, now 27) 33.5 -> 21.6 us; 40
// requests of which 8 bring 34 to 582 tokens 141 -> 135.
__host__ __device__ inline int64_t row_tiles(int E, int G, int shift)
{
    return E <= 0 ? 0 : ((int64_t)E * G + (1 << shift) - 1) >> shift;
}
constexpr int kAlternateRounds = 16;
// Row tile of a request for its unit-th work unit.  The longest first, so that the last items of the list are
// short.  In a batch of equal requests every second one takes the shortest first: a CU that has had longer items
// of one request than others has shorter ones of the next, while the list stays request by request, which the
// L2 wants.  8 requests, P = 6144, E = 2304, 32/8 heads (288 items of a KV head on 32 CUs, 97 to 132 key tiles): 1944
// -> 1868 us, the attention launch, with the same row tiles; with tiles of whole heads in one order it was 1944 too.  2 row
// tiles a request and 2 items a CU (32, P = 10240, E = 128): no difference, 647 to 660 us.  Calls of more than
// kAlternateRounds items a CU gain nothing and stay as they are.
__device__ __forceinline__ int row_tile_of(int unit, int nt, int r, int batch, int alternate)
{
    return alternate && ((batch - r) & 1) == 0 ? unit : nt - 1 - unit;
}
// Few new tokens: the rows of a KV head (G heads x E tokens) fit into kDecMaxRowBlocks blocks.
constexpr int kDecRows = 32;        // (head, token) rows per wavefront
constexpr int kDecMaxRowBlocks = 2; // row blocks per (request, KV head): G x E_r <= 64 (beyond, the row-tiled kernel is faster)
__host__ __device__ inline bool decode_shaped(int E, int G) { return E <= kDecRows * kDecMaxRowBlocks && E * G <= kDecRows * kDecMaxRowBlocks; }
// Mixed batches: key ranges of a request (partial results per row; 1 = the result is written directly).
__host__ __device__ inline int splits_of_request(int P, int E, int G, int seg_tiles, int dec_blocks)
{
    if (E <= 0) return 0;
    if (decode_shaped(E, G)) return ((P + E + 31) / 32 + dec_blocks - 1) / dec_blocks;
    const int tiles = (P + kBN - 1) / kBN + (E + kBN - 1) / kBN;
    const int ns = (tiles + seg_tiles - 1) / seg_tiles;
    return ns < kMaxSplits ? ns : kMaxSplits;
}
// Mixed batches: how many of the first n items of a KV head are decode-shaped work.  They are spread evenly
// over the list: side by side they wait for memory, of which row-tiled items need little.  dec_share is
// rounded up, so that all of them are counted at the end.
__device__ __forceinline__ int decode_items_before(int n, uint64_t dec_share) { return (int)((uint64_t)n * dec_share >> 32); }
// Inclusive prefix sum over the 64 lanes of a wavefront.
__device__ __forceinline__ int wave_inclusive_scan(int x, int lane)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    return x;
}

// A request of a mixed batch and the place of one unit of its work.
struct Owner {
    int r;      // request, batch: none
    int unit;   // index among the request's units
    int P, E;
    int cu;     // packed row of its first new token
    int parts;  // rows of partial results of the requests before it
    int splits; // its key ranges
};
// The request that owns position `at` of a list of units.  kDecode: the decode-shaped requests, row
// blocks x key chunks each.  Otherwise the row-tiled requests, row tiles x key ranges
// each.  The list takes the requests of a group of 64 in the order that the host gives (most keys
// first, so that the items that start last are short).  Every lane takes one request; the first unit
// of each is a sum over the lanes.
template <bool kDecode>
__device__ __forceinline__ Owner find_owner(int at, const MixedParams &p, int lane)
{
    Owner w{p.batch, at, 0, 0, 0, 0, 1};
    for (int base = 0; base < p.batch; base += 64) {
        const int rr = base + lane;
        const int e = rr < p.batch ? p.extend_lens[rr] : 0;
        const int pl = rr < p.batch ? p.prefix_lens[rr] : 0;
        const int from = p.order[rr];
        const int ns = splits_of_request(pl, e, p.G, p.seg_tiles, p.dec_blocks);
        int units = 0;
        if (e > 0 && decode_shaped(e, p.G) == kDecode)
            units = (kDecode ? (e * p.G + kDecRows - 1) / kDecRows : (int)row_tiles(e, p.G, p.tile_shift)) * ns;
        const int sorted = __shfl(units, from, 64);
        const int incl = wave_inclusive_scan(sorted, lane);
        const int parts = ns > 1 ? ns * e : 0;
        const int incl_e = wave_inclusive_scan(e, lane);
        const int incl_p = wave_inclusive_scan(parts, lane);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        if (w.unit < total) {
            const int place = __builtin_ctzll(__builtin_amdgcn_ballot_w64(incl > w.unit));
            const int first = __builtin_amdgcn_readlane(from, place);
            w.r = base + first;
            w.unit -= __builtin_amdgcn_readlane(incl - sorted, place);
            w.cu += __builtin_amdgcn_readlane(incl_e - e, first);
            w.parts += __builtin_amdgcn_readlane(incl_p - parts, first);
            w.E = __builtin_amdgcn_readlane(e, first);
            w.P = __builtin_amdgcn_readlane(pl, first);
            w.splits = __builtin_amdgcn_readlane(ns, first);
            return w;
        }
        w.unit -= total;
        w.cu += __builtin_amdgcn_readlane(incl_e, 63);
        w.parts += __builtin_amdgcn_readlane(incl_p, 63);
    }
    return w;
}

// ---- decode-shaped calls ------------------------------------------------------------------
// When every request brings so few new tokens that all its rows for one KV head (G heads x E_r
// tokens) fit a few 32-column MFMA tiles, the call is bound by reading the cached K/V once,
// and the row-tiled kernel below wastes its wavefronts (most hold no valid row) and keeps too
// little in flight.  This kernel turns the work around: a wavefront is the unit, owns the one or two
// blocks of 32 rows of one (request, KV head) and a share of its keys, in blocks of 32, and runs alone - no
// barrier, no shared tile.  It loads the K and V rows of a block with fully coalesced 16-byte loads
// (one instruction = four whole rows), stages them in registers while the previous block is
// computed, and passes them through a private LDS area from which the MFMA operands are read (K rows
// as they are, V rows transposed).  Prefix and suffix keys form one sequence of N = P + E keys;
// blocks inside the prefix take their two pages from the block table with scalar loads, the last
// blocks resolve every row on its own.  The results of a workgroup's wavefronts (m, l, O) are added up
// through LDS; a merge launch is left only where several workgroups share the keys of a request.
// Bound by reading the cache.  32 requests of 10240 tokens, 32/8 heads, with the merge: 217 -> 212 us for 1 new
// token (6.3 TB/s), 254 -> 222 for 16 (two blocks of rows, each of which read the keys for itself before;
// a pair of wavefronts that shares its keys behind barriers took 281); 64 of 100 tokens 11.6 -> 7.0; 20 of
// 9000, 64/8 heads 141 -> 118.
// LDS bytes per K row / V row: 256 + padding.  16 consecutive K rows at the same column fall into
// 16 different 16-byte bank groups, the four consecutive V rows of a transposing read into four
// different 64-byte bank groups, and every read address is a per-lane base plus an immediate.
constexpr int kDecPitchK = 272;
constexpr int kDecPitchV = 320;
constexpr int kDecLdsK = 32 * kDecPitchK;
constexpr int kDecLdsPerWave = kDecLdsK + 32 * kDecPitchV;
constexpr int kDecLeastWaves = 4;       // wavefronts of the smallest workgroup
constexpr int kDecMaxChunks = 256;      // partial results per (request, KV head), at most

struct DecBlock { // one block of 32 keys as loaded: piece i is row (lane / 16) + 4 i, chunk lane % 16
    u32x4 k[8];
    u32x4 v[8];
};

// What a wavefront has after its keys for a block of 32 rows: unnormalised, reference m (log2 domain), sum l
// over this half-wave's keys; o[db][v] is O^T[d = db*32 + 8*(v/4) + 4*h + v%4][row j].
struct DecResult {
    f32x16 o[4];
    float m, l;
};

// One wavefront: kRowBlocks blocks of 32 rows, from rb on, of (request r, KV head kvh) against the key blocks
// b, b + step, ... below b1.
template <int kRowBlocks>
__device__ __forceinline__ void decode_keys(const AttnParams &p, char *lds_k, int lane, int r, int kvh, int P, int E,
                                            int cu, int rb, int b, int b1, int step, DecResult (&res)[kRowBlocks])
{
    char *const lds_v = lds_k + kDecLdsK;
    const int j = lane & 31; // (head, token) row of the accumulators; key row of the K operand
    const int h = lane >> 5;
    const int N = P + E;

    // Q fragments, B operand of S^T = K Q^T: lane (row j, h) holds q[row][16 kk + 8 h .. + 8).
    // Row 32 rb + j of the (request, KV head) is token e of head hg of the group; rows beyond
    // G E are padding.
    u32x4 qf[kRowBlocks][8];
    int e_row[kRowBlocks];
#pragma unroll
    for (int q = 0; q < kRowBlocks; ++q) {
        const int row = (rb + q) * kDecRows + j;
        const int hg = row < p.G * E ? row / E : 0;
        const int e = row < p.G * E ? row - hg * E : 0;
        e_row[q] = e;
        const uint16_t *qp = p.q + ((int64_t)(cu + e) * p.Hq + kvh * p.G + hg) * kD + 8 * h;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) qf[q][kk] = *(const __attribute__((address_space(1))) u32x4 *)(qp + 16 * kk);
    }

    // loads: lane covers rows ld_sub + 4 i (i = 0..7) of the block, 16-byte chunk ld_chunk
    const int ld_sub = lane >> 4, ld_chunk = lane & 15;
    const __attribute__((address_space(4))) int32_t *table =
        (const __attribute__((address_space(4))) int32_t *)(p.block_table + (int64_t)r * p.max_pages);
    const int64_t v_plane = (int64_t)p.Hkv * kPS * kD;
    const int64_t page_stride = 2 * v_plane;
    const uint16_t *pages_head = p.kv_pages + (int64_t)kvh * (kPS * kD) + ld_chunk * 8;
    auto load_block = [&](int b, DecBlock &blk) {
        if (b * 32 + 32 <= P) {
            // inside the prefix: rows 0..15 in page 2 b, rows 16..31 in page 2 b + 1
            const int64_t pg[2] = {table[2 * b], table[2 * b + 1]};
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint16_t *krow = pages_head + pg[i >> 2] * page_stride + ((ld_sub + 4 * i) & 15) * kD;
                blk.k[i] = *(const __attribute__((address_space(1))) u32x4 *)(krow);
                blk.v[i] = *(const __attribute__((address_space(1))) u32x4 *)(krow + v_plane);
            }
        } else {
            // last blocks: every row resolves its own key (clamped to the last one; masked below)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int key = min(b * 32 + ld_sub + 4 * i, N - 1);
                const uint16_t *krow, *vrow;
                if (key < P) {
                    krow = pages_head + (int64_t)p.block_table[(int64_t)r * p.max_pages + (key >> 4)] * page_stride +
                           (key & 15) * kD;
                    vrow = krow + v_plane;
                } else {
                    const int64_t off = ((int64_t)(cu + key - P) * p.Hkv + kvh) * kD + ld_chunk * 8;
                    krow = p.k_new + off;
                    vrow = p.v_new + off;
                }
                blk.k[i] = *(const __attribute__((address_space(1))) u32x4 *)(krow);
                blk.v[i] = *(const __attribute__((address_space(1))) u32x4 *)(vrow);
            }
        }
    };
    const int st_k = ld_sub * kDecPitchK + ld_chunk * 16;
    const int st_v = ld_sub * kDecPitchV + ld_chunk * 16;
    auto store_block = [&](const DecBlock &blk) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            *reinterpret_cast<u32x4 *>(lds_k + st_k + 4 * i * kDecPitchK) = blk.k[i];
            *reinterpret_cast<u32x4 *>(lds_v + st_v + 4 * i * kDecPitchV) = blk.v[i];
        }
    };
    // operand reads, as in the row-tiled kernel below, with padded rows instead of swizzled ones
    const int k_lane = j * kDecPitchK + h * 16;
    const int v_lane = (4 * h + ((lane & 15) >> 2)) * kDecPitchV + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;

#pragma unroll
    for (int q = 0; q < kRowBlocks; ++q) {
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) res[q].o[db][v] = 0.f;
        res[q].m = -INFINITY;
        res[q].l = 0.f;
    }
    const float c = p.scale_log2;
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

    // all rows against key block b, which is staged in LDS; the row blocks are chains of their own, so one
    // computes while the other waits for its result
    auto compute_block = [&](int b) {
        f32x16 s[kRowBlocks];
        u32x4 pb[kRowBlocks][2];
        float alpha[kRowBlocks];
#pragma unroll
        for (int q = 0; q < kRowBlocks; ++q)
#pragma unroll
            for (int v = 0; v < 16; ++v) s[q][v] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const u32x4 a = *reinterpret_cast<const u32x4 *>(lds_k + k_lane + kk * 32);
#pragma unroll
            for (int q = 0; q < kRowBlocks; ++q)
                s[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                                __builtin_bit_cast(bf16x8, qf[q][kk]), s[q], 0, 0, 0);
        }
        // accumulator element v is key 32 b + 8 (v / 4) + 4 h + v % 4; row j sees keys <= P + e
        if (b * 32 + 31 > P) {
#pragma unroll
            for (int q = 0; q < kRowBlocks; ++q) {
                const int vis = P + e_row[q] - b * 32 - 4 * h; // visible: 8 (v / 4) + v % 4 <= vis
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (8 * (v >> 2) + (v & 3) > vis) s[q][v] = -INFINITY;
            }
        }
        bool moved = false;
#pragma unroll
        for (int q = 0; q < kRowBlocks; ++q) {
            float mx = s[q][0];
#pragma unroll
            for (int v = 1; v + 1 < 16; v += 2) mx = fmaxf(fmaxf(mx, s[q][v]), s[q][v + 1]);
            mx = halfwave_max(fmaxf(mx, s[q][15]));
            const float m_new = fmaxf(res[q].m, mx * c);
            const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
            alpha[q] = fast_exp2(res[q].m - m_use);
            float psum = 0.f;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    f32x2 x;
                    x[0] = fast_exp2(fmaf(s[q][8 * u + 2 * w], c, -m_use));
                    x[1] = fast_exp2(fmaf(s[q][8 * u + 2 * w + 1], c, -m_use));
                    const bf16x2 y = __builtin_convertvector(x, bf16x2);
                    psum = __builtin_amdgcn_fdot2_f32_bf16(y, ones, psum, false);
                    pb[q][u][w] = __builtin_bit_cast(unsigned, y);
                }
            res[q].l = res[q].l * alpha[q] + psum;
            res[q].m = m_new;
            moved |= alpha[q] != 1.f;
        }
        if (__builtin_amdgcn_ballot_w64(moved) != 0) {
#pragma unroll
            for (int q = 0; q < kRowBlocks; ++q)
#pragma unroll
                for (int db = 0; db < 4; ++db)
#pragma unroll
                    for (int v = 0; v < 16; ++v) res[q].o[db][v] *= alpha[q];
        }
        // O^T += V^T P^T: 2 steps of 16 keys x 4 blocks of 32 d
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int db = 0; db < 4; ++db) {
                const char *a = lds_v + v_lane + db * 64 + ks * 16 * kDecPitchV;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4 *)(a));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4 *)(a + 8 * kDecPitchV));
                const s16x8 vv = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int q = 0; q < kRowBlocks; ++q)
                    res[q].o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vv),
                                                                            __builtin_bit_cast(bf16x8, pb[q][ks]), res[q].o[db], 0, 0, 0);
            }
    };

    DecBlock blk;
    if (b < b1) load_block(b, blk);
    for (; b < b1; b += step) {
        // block b: registers -> private LDS (one wavefront's LDS operations are served in order,
        // so these writes come after the reads of the block before), then the next one into flight
        store_block(blk);
        if (b + step < b1) load_block(b + step, blk);
        compute_block(b);
    }
}

// Writes row `row` (token e of a head, -1: padding) of a finished wavefront: out, or its partial result.
__device__ __forceinline__ void store_decode_row(const AttnParams &p, const DecResult &res, int lane, int64_t out_row, int64_t part_row,
                                                 int head, bool row_valid)
{
    const int h = lane >> 5;
    const float l_tot = halfwave_sum(res.l);
    if (!row_valid) return;
    if (part_row < 0) {
        const float inv = 1.f / l_tot;
        uint16_t *po = p.out + (out_row * p.Hq + head) * kD;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                bf16x4 x;
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = (__bf16)(res.o[db][4 * gq + i] * inv);
                *reinterpret_cast<bf16x4 *>(po + db * 32 + 8 * gq + 4 * h) = x;
            }
        return;
    }
    const int64_t prow = part_row * p.Hq + head;
    float *po = p.part_o + prow * kD;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            f32x4 x = {res.o[db][4 * gq], res.o[db][4 * gq + 1], res.o[db][4 * gq + 2], res.o[db][4 * gq + 3]};
            *reinterpret_cast<f32x4 *>(po + db * 32 + 8 * gq + 4 * h) = x;
        }
    if (h == 0) {
        p.part_ml[prow * 2] = res.m;
        p.part_ml[prow * 2 + 1] = l_tot;
    }
}

// One wavefront on its own: row block rb against the key blocks b0 .. b1 - 1.  The partial result of token
// e goes to row part_row + e of the partial results; part_row < 0 says that these are all the keys and
// writes the finished rows instead.
__device__ __forceinline__ void decode_chunk(const AttnParams &p, char *lds_k, int lane, int r, int kvh, int P, int E,
                                             int cu, int rb, int b0, int b1, int64_t part_row)
{
    const int row = rb * kDecRows + (lane & 31);
    const bool row_valid = row < p.G * E;
    const int hg = row_valid ? row / E : 0;
    const int e = row_valid ? row - hg * E : 0;
    const int head = kvh * p.G + hg;
    if (rb * kDecRows >= p.G * E) return;
    if (b0 >= b1) { // nothing to do for this chunk: the merge skips entries whose sum is zero
        if (row_valid && lane < 32) {
            const int64_t prow = (part_row + e) * p.Hq + head;
            p.part_ml[prow * 2] = -INFINITY;
            p.part_ml[prow * 2 + 1] = 0.f;
        }
        return;
    }
    DecResult res[1];
    decode_keys<1>(p, lds_k, lane, r, kvh, P, E, cu, rb, b0, b1, 1, res);
    store_decode_row(p, res[0], lane, cu + e, part_row < 0 ? -1 : part_row + e, head, row_valid);
}

// A workgroup takes kRowBlocks blocks of 32 rows of one (request, KV head) and one of the nsplit chunks of
// its keys; its wavefronts take the chunk's key blocks in turn.  With two row blocks a wavefront
// needs twice the registers and a CU holds four of them instead of eight: enough, four read 61 GB/s with one
// row block and 35 with two, and the memory gives every CU 25.
constexpr int kDecPitchO = kD + 4; // floats between rows of O in LDS: rows in different banks
static_assert((32 * kDecPitchO + 64) * 4 <= kDecLdsPerWave, "a wavefront's result fits where its keys were");
template <int kDecWaves, int kRowBlocks>
__global__ __launch_bounds__(kDecWaves * 64, kRowBlocks == 1 ? 2 : 1) void decode_attn_kernel(const AttnParams p)
{
    __shared__ __attribute__((aligned(16))) char lds[kDecWaves * kDecLdsPerWave];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;

    // work unit: row blocks fastest, then key chunk, KV head, request.  Row blocks of the same keys stay on one
    // XCD where the number of units allows it, so that its L2 fetches the keys once.
    const int row_groups = (p.dec_row_blocks + kRowBlocks - 1) / kRowBlocks;
    int rg = blockIdx.x % row_groups, uc = blockIdx.x / row_groups;
    if (row_groups > 1 && gridDim.x / row_groups % kXcds == 0) {
        const int at = blockIdx.x / kXcds;
        rg = at % row_groups;
        uc = at / row_groups * kXcds + blockIdx.x % kXcds;
    }
    const int chunk = uc % p.nsplit;
    const int rk = uc / p.nsplit;
    const int kvh = rk % p.Hkv;
    const int r = rk / p.Hkv;
    if (r >= p.batch) return;
    const int E = p.extend_lens[r];
    const int rows = min(p.G * E - rg * kRowBlocks * kDecRows, kRowBlocks * kDecRows); // of this workgroup
    if (rows <= 0) return;
    const int P = p.prefix_lens[r];
    // packed row of the request's first token: sum of the earlier extend lengths, 64 per step
    int cu = 0;
    for (int base = 0; base < r; base += 64) cu += base + lane < r ? p.extend_lens[base + lane] : 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cu += __shfl_xor(cu, off, 64);
    cu = __builtin_amdgcn_readfirstlane(cu);
    // no row of a block sees keys behind its last token
    const int end_e = kRowBlocks > 1 ? E : min(rg * kDecRows % E + kDecRows, E);
    const int nblk = (P + end_e + 31) >> 5;
    const int per = (nblk + p.nsplit - 1) / p.nsplit;
    const int b0 = chunk * per;
    const int b1 = min(nblk, b0 + per);

    DecResult res[kRowBlocks];
    decode_keys<kRowBlocks>(p, lds + wave * kDecLdsPerWave, lane, r, kvh, P, E, cu, rg * kRowBlocks, b0 + wave, b1,
                            kDecWaves, res);

    // ---- the wavefronts' results through LDS, a block of rows at a time
    const int d4 = (threadIdx.x & 31) * 4;
#pragma unroll
    for (int q = 0; q < kRowBlocks; ++q) {
        if (q * kDecRows >= rows) return;
        const float l_tot = halfwave_sum(res[q].l);
        if (q > 0) __syncthreads(); // the block before has been read
        {
            float *const mine = reinterpret_cast<float *>(lds + wave * kDecLdsPerWave);
            const int j = lane & 31, h = lane >> 5;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const f32x4 x = {res[q].o[db][4 * gq], res[q].o[db][4 * gq + 1], res[q].o[db][4 * gq + 2], res[q].o[db][4 * gq + 3]};
                    *reinterpret_cast<f32x4 *>(mine + j * kDecPitchO + db * 32 + 8 * gq + 4 * h) = x;
                }
            if (h == 0) *reinterpret_cast<f32x2 *>(mine + 32 * kDecPitchO + 2 * j) = f32x2{res[q].m, l_tot};
        }
        __syncthreads();
        for (int i = threadIdx.x >> 5; i < min(kDecRows, rows - q * kDecRows); i += kDecWaves * 2) {
            f32x2 ml[kDecWaves];
            f32x4 x[kDecWaves];
#pragma unroll
            for (int w = 0; w < kDecWaves; ++w) {
                const float *const part = reinterpret_cast<const float *>(lds + w * kDecLdsPerWave);
                ml[w] = *reinterpret_cast<const f32x2 *>(part + 32 * kDecPitchO + 2 * i);
                x[w] = *reinterpret_cast<const f32x4 *>(part + i * kDecPitchO + d4);
            }
            float m_star = -INFINITY;
#pragma unroll
            for (int w = 0; w < kDecWaves; ++w)
                if (ml[w][1] != 0.f) m_star = fmaxf(m_star, ml[w][0]);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            float denom = 0.f;
#pragma unroll
            for (int w = 0; w < kDecWaves; ++w)
                if (ml[w][1] != 0.f) { // 0: no keys, or none that the row sees; NaN goes through
                    const float f = fast_exp2(ml[w][0] - m_star);
                    acc += x[w] * f;
                    denom += ml[w][1] * f;
                }
            const int row = (rg * kRowBlocks + q) * kDecRows + i, hg = row / E, e = row - hg * E;
            const int head = kvh * p.G + hg;
            if (p.nsplit == 1) {
                const float inv = 1.f / denom; // every row sees its own key
                bf16x4 y;
#pragma unroll
                for (int k = 0; k < 4; ++k) y[k] = (__bf16)(acc[k] * inv);
                *reinterpret_cast<bf16x4 *>(p.out + ((int64_t)(cu + e) * p.Hq + head) * kD + d4) = y;
            } else {
                const int64_t prow = ((int64_t)chunk * p.T + cu + e) * p.Hq + head;
                *reinterpret_cast<f32x4 *>(p.part_o + prow * kD + d4) = acc;
                if (d4 == 0) *reinterpret_cast<f32x2 *>(p.part_ml + prow * 2) = f32x2{m_star, denom};
            }
        }
    }
}

// LDS: four K buffers and five V buffers of one 64-key tile (16 KiB) each, K of tile t in buffer
// t % 4, V in buffer t % 5.  A tile is requested two iterations before its first use and V(t) is
// still read one iteration after K(t).  The workgroup meets at a barrier only after every second
// tile (tiles 2m+1 and 2m+2 form an interval): within an interval K(2m+1), K(2m+2), V(2m) and
// V(2m+1) are read, V(2m+2) is resident, and tiles 2m+3 and 2m+4 arrive, which takes four K
// buffers and five V buffers if no arriving tile is to overwrite one that a slower wavefront of
// the same interval still reads.
// The tiles come from global memory straight into LDS (global_load_lds_dwordx4: lane i of a
// wavefront writes 16 bytes at slot i of 1 KiB, no way through registers and no LDS store
// instruction), so rows cannot be padded: they are 256 bytes apart and the 16-byte chunks
// inside a row are swizzled instead.  K: chunk c of row r sits at slot c ^ (r & 15) (16
// consecutive rows at the same column fall into 16 different 16-byte bank groups); V: at slot
// c ^ ((r & 3) << 2) (the four consecutive rows of a transposing read fall into four different
// 64-byte bank groups).
constexpr int kNumBufs = 4;
constexpr int kPitchK = 256;
constexpr int kPitchV = 256;
constexpr int kTileBytesK = kBN * kPitchK;
constexpr int kTileBytesV = kBN * kPitchV;
constexpr int kNumBufsV = 5;
constexpr int kLdsBytes = kNumBufs * kTileBytesK + kNumBufsV * kTileBytesV;
// The operand reads find the 16-byte chunks of a row by exclusive or in bits 4 to 7 of an address: rows and buffers begin
// at multiples of this, and so does the array that holds them.
constexpr int kLdsAlign = 256;
static_assert(kPitchK % kLdsAlign == 0 && kPitchV % kLdsAlign == 0 && kTileBytesK % kLdsAlign == 0 && kTileBytesV % kLdsAlign == 0,
              "exclusive or in place of an addition");

constexpr int kMixedLdsBytes = kWaves * kDecLdsPerWave > kLdsBytes ? kWaves * kDecLdsPerWave : kLdsBytes;

// What one launch works on: whole key ranges, a split of every request's keys, or a mixed batch:
// requests of unequal lengths, each split by its own length, decode-shaped ones next to row-tiled ones.
// One number of splits for all leaves the longest request to finish alone, and a token that is
// decoded on a row tile of 256 rows occupies a CU for all its keys.  8 chunks of prompts next to 32
// decoding requests, up to 12000 cached tokens, 32/8 heads: 246 -> 157 us; 5 and 43, 8/2 heads: 144 -> 69;
// 21 prompts of 20 to 125 tokens, 64/8 heads: 87 -> 54.  Bound by the row-tiled items, which fill the CUs.
// The decode work is spread over the list: behind the row-tiled items it ran on all CUs at once and waited for
// memory (the first of these 157 us so, 146 spread out; 22 decoding beside 4 chunks 59.2 and 58.9).
enum Mode { kWhole, kSplit, kMixed };
template <Mode kMode>
__global__ __launch_bounds__(kThreads) void extend_attn_kernel(const std::conditional_t<kMode == kMixed, MixedParams, AttnParams> p)
{
    extern __shared__ __attribute__((aligned(kLdsAlign))) char lds[];
    char *const lds_k = lds;                          // [4][64 rows][256 B]
    char *const lds_v = lds + kNumBufs * kTileBytesK; // [5][64 rows][256 B]

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int j = lane & 31; // query row within the wave; also key row / d row of A operands
    const int h = lane >> 5; // half-wave

    int kvh = 0;
    const int rem = work_item(blockIdx.x, p, kvh);
    if (rem < 0) return;
    int r, cu, E, P, unit, split, nsplit, parts = 0;
    if constexpr (kMode == kMixed) {
        const int decode_before = decode_items_before(rem, p.dec_share);
        if (decode_items_before(rem + 1, p.dec_share) > decode_before) { // eight wavefronts of decode-shaped work, each on its own
            const Owner w = find_owner<true>(decode_before * kWaves + wave, p, lane);
            if (w.r >= p.batch) return;
            const int row_blocks = (w.E * p.G + kDecRows - 1) / kDecRows;
            const int rb = w.unit % row_blocks, chunk = w.unit / row_blocks; // row blocks of the same keys side by side
            const int nblk = (w.P + w.E + 31) / 32, per = (nblk + w.splits - 1) / w.splits;
            decode_chunk(p, lds + wave * kDecLdsPerWave, lane, w.r, kvh, w.P, w.E, w.cu, rb, chunk * per,
                         min(nblk, chunk * per + per), w.splits > 1 ? w.parts + (int64_t)chunk * w.E : -1);
            return;
        }
        const Owner w = find_owner<false>(rem - decode_before, p, lane);
        r = w.r;
        cu = w.cu;
        E = w.E;
        P = w.P;
        parts = w.parts;
        nsplit = max(w.splits, 1);
        split = w.unit % nsplit;
        unit = w.unit / nsplit;
    } else {
        nsplit = 1;
        split = 0;
        unit = rem;
        if (kMode == kSplit && rem >= p.whole_units) {
            nsplit = p.nsplit;
            const int piece = rem - p.whole_units;
            unit = p.whole_units + piece / nsplit;
            split = piece % nsplit;
        }
        const int tail_unit = unit - p.whole_units;
        r = p.batch;
        cu = E = P = 0;
        // Units of a KV head: requests in order; within a request the last (longest) row tile first.
        // The request that owns the unit is found 64 requests at a time: every lane takes one
        // request, a prefix sum over the wavefront gives the first unit of each (a sequential scan
        // costs a dependent scalar load and several integer divisions per request, ~1.5 us each).
        for (int base = 0; base < p.batch; base += 64) {
            const int rr = base + lane;
            const int e_l = rr < p.batch ? p.extend_lens[rr] : 0;
            const int units_l = (int)row_tiles(e_l, p.G, p.tile_shift);
            const int incl_u = wave_inclusive_scan(units_l, lane);
            const int incl_e = wave_inclusive_scan(e_l, lane);
            const int total_u = __builtin_amdgcn_readlane(incl_u, 63);
            if (unit < total_u) {
                const int first = __builtin_ctzll(__builtin_amdgcn_ballot_w64(incl_u > unit));
                r = base + first;
                unit -= __builtin_amdgcn_readlane(incl_u - units_l, first);
                cu += __builtin_amdgcn_readlane(incl_e - e_l, first);
                E = __builtin_amdgcn_readlane(e_l, first);
                break;
            }
            unit -= total_u;
            cu += __builtin_amdgcn_readlane(incl_e, 63);
        }
        if (r < p.batch) P = p.prefix_lens[r];
        if (p.tail_units > 0) parts = ((kvh * p.tail_units + tail_unit) * nsplit + split) * kBM + wave * 32;
    }
    if (r >= p.batch) return;
    const int t = row_tile_of(unit, (int)row_tiles(E, p.G, p.tile_shift), r, p.batch, kMode != kMixed && p.alternate);

    // Row i of the (request, KV head) is token i / G for q head i % G of the group; the q heads of the KV
    // head thus share the workgroup's K/V tiles.
    const int rows = E * p.G;
    const int tile_end = min(rows, (t + 1) << p.tile_shift);   // one past the tile's last row
    const int wave_row0 = (t << p.tile_shift) + wave * 32;     // first row of this wavefront
    const int wave_tok0 = over_heads(wave_row0, p);            // its token
    const int wave_tok1 = over_heads(wave_row0 + 31, p);       // token of the last row (may be >= E)
    const bool row_valid = wave_row0 + j < tile_end;
    const int row_tok = over_heads(min(wave_row0 + j, rows - 1), p); // this lane's token
    const int head = kvh * p.G + min(wave_row0 + j, rows - 1) - row_tok * p.G;
    const int rows_end = over_heads(tile_end - 1, p) + 1; // one past the tile's last token
    const int np_tiles = (P + kBN - 1) / kBN;        // prefix key tiles
    const int ns_tiles = (rows_end + kBN - 1) / kBN; // suffix key tiles up to the diagonal
    const int n_tiles = np_tiles + ns_tiles;
    // mixed: a row tile with fewer keys than the last one of its request takes fewer ranges, the rest stay empty.  None is
    // longer than the last one's: with ranges up to seg_tiles, which the last one's need not reach, a tile of 15 key tiles
    // next to one of 16 in 2 ranges was left whole (20 requests, of which 16 decode, 32/8 heads: 39.4 us with ranges of
    // at most 15 key tiles, 29.6 of at most 11).  250 random batches take 0.996 of the time, 0.875 to 1.042.
    int n_ranges = nsplit;
    if constexpr (kMode == kMixed) {
        const int longest = (np_tiles + (E + kBN - 1) / kBN + nsplit - 1) / nsplit;
        n_ranges = min(nsplit, (n_tiles + longest - 1) / longest);
    }
    const int per_split = (n_tiles + n_ranges - 1) / n_ranges;
    const int kt_begin = split * per_split;
    const int kt_end = min(n_tiles, kt_begin + per_split);
    const int n_it = kt_end - kt_begin;              // key tiles of this work item

    const int64_t out_row = (int64_t)(cu + row_tok);
    const bool partial = kMode != kWhole && nsplit > 1;
    // row of the partial results
    auto part_row = [&]() -> int64_t {
        if (kMode == kSplit && p.tail_units > 0) return parts + j;
        return (kMode == kMixed ? parts + (int64_t)split * E + row_tok : (int64_t)split * p.T + out_row) * p.Hq + head;
    };

    if (n_it <= 0) {
        // empty split: the merge skips entries whose sum is zero
        if (partial && row_valid && h == 0) {
            float *ml = p.part_ml + part_row() * 2;
            ml[0] = -INFINITY;
            ml[1] = 0.f;
        }
        return;
    }

    // ---- Q fragments, B operand of S^T = K Q^T: lane (j, h) holds q[row j][16 kk + 8 h ..+8)
    // The fragments hold q * softmax_scale * log2(e), rounded to bf16 (nearest even) once per
    // row: the accumulators of S^T are then the arguments of exp2 as they stand, which saves one
    // multiply-add per score (a third of the softmax instructions).  The rounding moves every
    // query element by at most half a bf16 unit in the last place.
    const float c = p.scale_log2;
    bf16x8 qf[8];
    {
        const uint16_t *qp = p.q + (out_row * p.Hq + head) * kD + 8 * h;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const bf16x8 raw = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(qp + 16 * kk));
#pragma unroll
            for (int e = 0; e < 8; ++e) qf[kk][e] = (__bf16)((float)raw[e] * c);
        }
    }

    // ---- this thread's share of a K/V tile: key rows ld_row and ld_row + kLoadRows, 16-byte chunk
    // ld_chunk.  The four rows a wavefront loads per step share one page, so the block-table
    // lookup and the page base are scalar; rows past the end of the prefix (or of the suffix)
    // re-read the last valid row so that no uninitialised cache slot is ever touched.
    const int ld_sub = lane >> 4;         // row within the wavefront's group of four
    const int ld_row = wave * 4 + ld_sub; // 0..kLoadRows-1
    const int ld_chunk = lane & 15;
    // read-only for the whole launch and every index is wavefront-uniform: the constant address
    // space keeps these loads on the scalar unit although the direct loads below write memory
    const __attribute__((address_space(4))) int32_t *table =
        (const __attribute__((address_space(4))) int32_t *)(p.block_table + (int64_t)r * p.max_pages);
    const int64_t v_plane = (int64_t)p.Hkv * kPS * kD; // K slab -> V slab inside a page
    const int64_t row_pitch = (int64_t)p.Hkv * kD;     // elements between rows of k_new

    // Full tiles (no row to clamp) take a shorter address path: a scalar base per page, or per
    // load step of the suffix, plus a per-lane byte offset that never changes.
    typedef const __attribute__((address_space(1))) char *gptr;
    const uint32_t row_bytes = (uint32_t)row_pitch * 2u;
    // Direct loads put lane i's 16 bytes into slot i of the wavefront's 1 KiB of LDS (4 rows of
    // 16 slots), so the swizzle is applied on the source side: slot s of row r holds chunk
    // s ^ (r & 15) of a K row and chunk s ^ ((r & 3) << 2) of a V row.
    const int ck = ld_chunk ^ (ld_row & 15);
    const int cv = ld_chunk ^ ((ld_row & 3) << 2);
    const uint32_t pg_lane_k = (uint32_t)(((ld_row & 15) * kD + ck * 8) * 2); // inside a page's K slab
    const uint32_t pg_lane_v = (uint32_t)(((ld_row & 15) * kD + cv * 8) * 2) + (uint32_t)(v_plane * 2);
    const uint32_t sfx_lane_k = (uint32_t)ld_row * row_bytes + (uint32_t)ck * 16u;
    const uint32_t sfx_lane_v = (uint32_t)ld_row * row_bytes + (uint32_t)cv * 16u;
    // Four direct loads of 16 bytes per lane: K and V rows ld_row and ld_row + 32 of buffer buf.
    // M0 carries the LDS address of the wavefront's 1 KiB.  The loads are written as assembly
    // because the compiler, for the builtin, waits for every direct load in flight before the
    // next LDS read of the wavefront, whichever buffer that read goes to; here the only reader
    // of the loaded buffer is two barriers away, and dma_wait() in front of each barrier is the
    // wait that is needed.  The compiler's own counts stay conservative: it does not see these
    // loads, loads complete in order, so its waits can only cover more than it meant.
    const uint32_t lds_k_wave = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_k + wave * (4 * kPitchK);
    const uint32_t lds_v_wave = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_v + wave * (4 * kPitchV);
    auto dma_tile = [&](gptr k0, gptr v0, gptr k1, gptr v1, int kbuf, int vbuf) {
        const uint32_t dk0 = __builtin_amdgcn_readfirstlane(lds_k_wave + kbuf * kTileBytesK);
        const uint32_t dv0 = __builtin_amdgcn_readfirstlane(lds_v_wave + vbuf * kTileBytesV);
        const uint32_t dk1 = dk0 + kLoadRows * kPitchK, dv1 = dv0 + kLoadRows * kPitchV;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, off\n\t"
                     "s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %5, off\n\t"
                     "s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %6, off\n\t"
                     "s_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %7, off"
                     :
                     : "s"(dk0), "s"(dv0), "s"(dk1), "s"(dv1), "v"(k0), "v"(v0), "v"(k1), "v"(v1)
                     : "memory"); // m0 is reserved: the compiler keeps nothing in it across statements
    };
    // all of this wavefront's direct loads have landed (the barrier that follows publishes them)
    auto dma_wait = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    const uint64_t page_bytes = (uint64_t)p.Hkv * (2u * kPS * kD * 2u);
    const gptr pages_head = (gptr)p.kv_pages + (int64_t)kvh * (kPS * kD * 2);
    const gptr knew_head = (gptr)p.k_new + ((int64_t)cu * p.Hkv + kvh) * (kD * 2);
    const gptr vnew_head = (gptr)p.v_new + ((int64_t)cu * p.Hkv + kvh) * (kD * 2);
    auto load_tile = [&](int kt, int t) { // t: tile number inside the work item
        const int kbuf = t & 3, vbuf = t % kNumBufsV;
        if (kt < np_tiles && (kt + 1) * kBN <= P) {
            gptr kp[2], vp[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t page = (uint32_t)table[kt * (kBN / kPS) + 2 * i + (wave >> 2)];
                const gptr base = pages_head + (uint64_t)page * page_bytes;
                kp[i] = base + pg_lane_k;
                vp[i] = base + pg_lane_v;
            }
            dma_tile(kp[0], vp[0], kp[1], vp[1], kbuf, vbuf);
            return;
        }
        if (kt >= np_tiles && (kt - np_tiles + 1) * kBN <= E) {
            const int64_t tile_off = (int64_t)(kt - np_tiles) * kBN * row_bytes;
            const int64_t off1 = tile_off + (int64_t)kLoadRows * row_bytes;
            dma_tile(knew_head + tile_off + sfx_lane_k, vnew_head + tile_off + sfx_lane_v,
                     knew_head + off1 + sfx_lane_k, vnew_head + off1 + sfx_lane_v, kbuf, vbuf);
            return;
        }
        const uint16_t *ks[2];
        const uint16_t *vs[2];
        if (kt < np_tiles) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int tok0 = min(kt * kBN + i * kLoadRows + wave * 4, P - 1); // wave-uniform
                const int sub = min(ld_sub, P - 1 - tok0);
                const int64_t page = table[tok0 >> 4];
                const uint16_t *base = p.kv_pages + (page * 2 * p.Hkv + kvh) * (kPS * kD);
                ks[i] = base + ((((tok0 + sub) & 15) * kD) + ck * 8);
                vs[i] = base + ((((tok0 + sub) & 15) * kD) + cv * 8) + v_plane;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int srow0 = min((kt - np_tiles) * kBN + i * kLoadRows + wave * 4, E - 1);
                const int sub = min(ld_sub, E - 1 - srow0);
                const int64_t base = ((int64_t)(cu + srow0) * p.Hkv + kvh) * kD;
                const int off = sub * (int)row_pitch;
                ks[i] = p.k_new + base + off + ck * 8;
                vs[i] = p.v_new + base + off + cv * 8;
            }
        }
        dma_tile((gptr)ks[0], (gptr)vs[0], (gptr)ks[1], (gptr)vs[1], kbuf, vbuf);
    };

    // ---- per-lane LDS read offsets (bytes inside a tile buffer)
    // K, A operand of S^T: lane (j, h) reads 16 bytes of key row kb*32 + j at chunk 2 kk + h,
    // which the swizzle puts at slot (2 kk + h) ^ (j & 15): the offset for kk = 0 with bits 5 to 7
    // exchanged.  Eight offsets kept in registers cost no fewer instructions (the buffer is added to each)
    // and leave the loop short of registers.
    const int k_lane = j * kPitchK + ((h ^ (j & 15)) << 4);
    // V^T, A operand of O^T = V^T P^T, through the transposing read: within a group of 16
    // lanes, lane i supplies the address of 4 consecutive d of key row k0 + i / 4 and receives
    // V[k0 .. k0+3][d0 + i].  Here k0 = 4 h (+ 8 for the second read), d0 = 32 db + 16 (lane/16 % 2);
    // the swizzle exchanges the 64-byte column blocks: block db of row r sits at db ^ (r & 3), the
    // offset for db = 0 with bits 6 and 7 exchanged.
    const int v_lane = (4 * h + ((lane & 15) >> 2)) * kPitchV + (((lane >> 2) & 3) << 6) + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    typedef __attribute__((address_space(3))) const char *lptr;
    const uint32_t lds_k0 = (uint32_t)(uintptr_t)(lptr)lds_k, lds_v0 = (uint32_t)(uintptr_t)(lptr)lds_v; // multiples of kLdsAlign

    f32x16 o[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
    float m_ref = -INFINITY; // reference maximum of the exponentials, log2 domain
    float l_run = 0.f;       // running sum over this half-wave's keys only
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

    typedef f32x16 STile[kNKB];     // scores: 32-key blocks x 32 query rows
    typedef bf16x8 PTile[2 * kNKB]; // probabilities: one B operand per 16 keys

    // S^T = K Q^T for the tile in K buffer kbuf.
    auto qk_tile = [&](int kbuf, STile &s) {
        const uint32_t kb = lds_k0 + kbuf * kTileBytesK + k_lane;
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < kNKB; ++b) s[b] = zero;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
#pragma unroll
            for (int bb = 0; bb < kNKB; ++bb) {
                const int b = kk >= 4 ? kNKB - 1 - bb : bb;
                const u32x4 a = *reinterpret_cast<__attribute__((address_space(3))) const u32x4 *>((lptr)(uintptr_t)(kb ^ (kk << 5)) + b * 32 * kPitchK);
                s[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), qf[kk], s[b], 0, 0, 0);
            }
        }
        // Issue order: kFragsAhead fragment reads first, then one read behind every MFMA, so
        // that an operand is requested kFragsAhead MFMAs before it is used (left alone, the
        // scheduler reads two fragments and waits for them at once).
        constexpr int kFragsAhead = 8;
        __builtin_amdgcn_sched_group_barrier(0x100, kFragsAhead, 0);
#pragma unroll
        for (int i = 0; i < 8 * kNKB - kFragsAhead; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, kFragsAhead, 0);
    };
    // O^T += V^T P^T for the tile in V buffer vbuf: 4 d blocks x steps of 16 keys.
    auto pv_tile = [&](int vbuf, const PTile &pb) {
        const uint32_t vb = lds_v0 + vbuf * kTileBytesV + v_lane;
#pragma unroll
        for (int ks = 0; ks < 2 * kNKB; ++ks) { // keys ks*16 .. ks*16+15
#pragma unroll
            for (int db = 0; db < 4; ++db) {
                const lptr a = (lptr)(uintptr_t)(vb ^ (db << 6)) + ks * 16 * kPitchV;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4 *)(a));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4 *)(a + 8 * kPitchV));
                const s16x8 vv = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vv), pb[ks], o[db], 0, 0, 0);
            }
        }
        // Same for the V fragments (two transposing reads each), five MFMAs ahead, with up to
        // four VALU instructions of the next tile's softmax (64 in all: 32 exponentials, 16
        // conversions, 16 row-sum steps) behind every MFMA where the caller has them in the same
        // block.
        constexpr int kFragsAhead = 5;
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * kFragsAhead, 0);
#pragma unroll
        for (int i = 0; i < 8 * kNKB; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (i < 8 * kNKB - kFragsAhead) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x400, 4, 0);
        }
    };
    // Masks the keys of a boundary tile that the lane's row must not see.  Accumulator element
    // v of block b is key b*32 + 8*(v/4) + 4*h + v%4 of the tile.
    auto mask_tile = [&](int vis, STile &s) {
        const int vis_h = vis - 4 * h;
#pragma unroll
        for (int b = 0; b < kNKB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (b * 32 + 8 * (v >> 2) + (v & 3) >= vis_h) s[b][v] = -INFINITY;
    };
    // Exponentials of one tile against the reference m_use (log2 domain), one query row per
    // lane: bf16 probabilities in B-operand order (pb[2b + u] element e is accumulator element
    // 8u + e of block b); returns their sum over this lane's keys.  `plain` says that the
    // reference is 0 for every row of the wavefront: then there is nothing to subtract.
    auto exp_tile = [&](const STile &s, PTile &pb, float m_use, auto plain) -> float {
        constexpr bool kPlain = decltype(plain)::value;
        float psum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e += 2)
#pragma unroll
            for (int t = 0; t < 2 * kNKB; ++t) {
                f32x2 x;
                const float s0 = s[t >> 1][8 * (t & 1) + e], s1 = s[t >> 1][8 * (t & 1) + e + 1];
                x[0] = fast_exp2(kPlain ? s0 : s0 - m_use);
                x[1] = fast_exp2(kPlain ? s1 : s1 - m_use);
                const bf16x2 y = __builtin_convertvector(x, bf16x2);
                pb[t][e] = y[0];
                pb[t][e + 1] = y[1];
            }
        // The row sums come after all conversions (the empty statement says so): mixed with them by the scheduler they
        // wait for each other between the last MFMAs of P V (4 requests, P = 24576, E = 8192, 64/8 heads 25.09 -> 25.02 ms; 1, P = 0,
        // E = 131072, 32/8 heads 114.7 -> 114.1; medians of 12 rounds in turn that differ by 0.2 to 0.4 %).
        u32x4 w[2 * kNKB];
#pragma unroll
        for (int t = 0; t < 2 * kNKB; ++t) w[t] = __builtin_bit_cast(u32x4, pb[t]);
        asm("" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]));
#pragma unroll
        for (int t = 0; t < 2 * kNKB; ++t) pb[t] = __builtin_bit_cast(bf16x8, w[t]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < 2 * kNKB; ++t) psum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, (unsigned)w[t][e]), ones, psum, false);
        return psum;
    };
    auto row_max = [&](const STile &s) -> float {
        float mx = s[0][0];
#pragma unroll
        for (int i = 1; i + 1 < 16 * kNKB; i += 2) // pairs, so that three-input maxima can be used
            mx = fmaxf(fmaxf(mx, s[i >> 4][i & 15]), s[(i + 1) >> 4][(i + 1) & 15]);
        mx = fmaxf(mx, s[kNKB - 1][15]);
        return halfwave_max(mx);
    };
    auto rescale_o = [&](float alpha) {
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
    };

    // ---- main loop, one barrier per two key tiles.  Iteration `it`:
    //     request tile it+2: global memory -> K buffer (it+2) % 4, V buffer (it+2) % 5, asynchronously
    //     S = K(it) Q^T                                            (MFMA)
    //     p = exp2(S - m_ref) next to O += V(it-1)^T P(it-1)^T     (VALU next to MFMA)
    //     if `it` is even: wait for the requested tiles, barrier
    // (S already carries softmax_scale * log2(e), see the Q fragments.)  The exponentials are
    // taken against the running reference m_ref WITHOUT first reducing the row maximum of the
    // tile.  Only when some row of the wavefront has no reference yet, or its sum shows that the
    // reference is stale by a factor 2^80 or more, is the tile redone the classic way (row
    // maximum, new reference, rescale of O and l).  Any reference gives the same result after
    // the final division as long as nothing overflows or vanishes: a row maximum inside
    // [-kSnap, kSnap] takes the reference 0 (exponentials between 2^-64 and 2^64 at the top of
    // the row, nothing to subtract), and below the trigger the sums stay under 2^80 times the
    // number of keys, which fp32 holds up to 2^47 keys of magnitude 1.
    load_tile(kt_begin, 0);
    if (n_it > 1) load_tile(kt_begin + 1, 1);
    dma_wait();
    __syncthreads();

    bool have_prev = false; // the previous tile's probabilities still wait for their P V
    constexpr float kStale = 1.2089258196146292e24f; // 2^80
    constexpr float kSnap = 64.f; // a row whose maximum lies in [-64, 64] takes the reference 0

    // Classic online-softmax step: row maximum, new reference, rescale of O and l.
    auto redo_tile = [&](const STile &s, PTile &pb) -> float {
        float m_new = fmaxf(m_ref, row_max(s));
        if (fabsf(m_new) <= kSnap) m_new = 0.f;
        const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
        const float alpha = fast_exp2(m_ref - m_use);
        rescale_o(alpha);
        l_run *= alpha;
        m_ref = m_new;
        return exp_tile(s, pb, m_use, std::false_type{});
    };
    // first key of tile kt in its own numbering (prefix tokens or suffix rows)
    auto tile_key0 = [&](int kt) { return kt >= np_tiles ? (kt - np_tiles) * kBN : kt * kBN; };
    auto masked_qk = [&](int kt, int buf, STile &s) {
        const bool suffix = kt >= np_tiles;
        const int key0 = tile_key0(kt);
        qk_tile(buf, s);
        const bool need_mask = suffix ? (key0 + kBN - 1 > wave_tok0) : (key0 + kBN > P);
        if (need_mask) mask_tile(suffix ? (row_tok - key0 + 1) : (P - key0), s);
    };
    // a suffix tile entirely above this wavefront's rows shows it nothing, and neither does
    // any later tile; a wavefront whose 32 rows all lie past the end of the request (short
    // extends, decode) computes nothing at all and only takes part in the cooperative loads
    const bool no_rows = wave_row0 >= tile_end;
    auto skipped = [&](int kt) { return no_rows || (kt >= np_tiles && tile_key0(kt) > wave_tok1); };

    PTile pb_a, pb_b; // probabilities of the previous / the current tile

    // iteration 0: no previous tile yet, and no reference: classic step
    {
        const bool prefetch = 2 < n_it;
        if (prefetch) load_tile(kt_begin + 2, 2);
        if (!skipped(kt_begin)) {
            STile s;
            masked_qk(kt_begin, 0, s);
            l_run += redo_tile(s, pb_a);
            have_prev = true;
        }
        dma_wait();
        __syncthreads();
    }
    // The barrier comes after every second tile (after the even ones): a function of the tile
    // number alone, so every wavefront meets the same barriers whichever loop it is in.
    auto pair_barrier = [&](int it) {
        if (!(it & 1)) {
            dma_wait();
            __syncthreads();
        }
    };
    // One full step; only called for tiles this wavefront does not skip (so the previous tile
    // was not skipped either and its probabilities are pending).
    auto tile_step = [&](int it, PTile &pb_cur, PTile &pb_prev) {
        const int buf = it & 3;
        const int kt = kt_begin + it;
        const bool prefetch = it + 2 < n_it;
        if (prefetch) load_tile(kt + 2, it + 2);
        STile s;
        masked_qk(kt, buf, s);
        // one basic block: the exponentials (VALU) interleave with P V (MFMA)
        float psum = exp_tile(s, pb_cur, (m_ref == -INFINITY) ? 0.f : m_ref, std::false_type{});
        pv_tile((it - 1) % kNumBufsV, pb_prev);
        if (__builtin_amdgcn_ballot_w64(!(psum < kStale) || m_ref == -INFINITY) != 0)
            psum = redo_tile(s, pb_cur);
        l_run += psum;
        pair_barrier(it);
    };
    int it = 1;
    if (have_prev) {
        // Steady state: while tile kt needs no mask for this wavefront and tile kt + 2 is a
        // full tile (inside the prefix, or suffix rows below the diagonal), the step has no
        // case distinctions, and the block-table entries of a tile are fetched one iteration
        // before its loads are issued (the general step spends ~500 of ~4200 cycles per tile
        // between the barrier and its first MFMA on tile kinds, table lookups and addresses,
        // with the matrix pipe idle).  A prefix that ends inside a tile leaves two such stretches, with the
        // general step between them (P = 777, E = 16000, 32/8 heads: 2038 -> 1927 us with the second one).
        for (;;) {
            const bool two_stretches = P % kBN != 0 && kt_begin + it < np_tiles; // the first one is ahead
            const int last_unmasked = np_tiles + (wave_tok0 >= kBN - 1 ? (wave_tok0 - (kBN - 1)) / kBN : -1);
            const int last_full = np_tiles + E / kBN - 1;
            const int fast_end = min(two_stretches ? P / kBN - 2 : min(last_unmasked + 1, last_full - 1), kt_end - 2) - kt_begin;
            if (it < fast_end) {
                const int tsel = wave >> 2;
                const int last_entry = (P + E + kPS - 1) / kPS - 1; // last page of the request: nothing beyond it is read
                auto entry = [&](int kt, int i) {
                    return (uint32_t)table[min(kt * (kBN / kPS) + 2 * i + tsel, last_entry)];
                };
                uint32_t pg0 = entry(kt_begin + it + 2, 0), pg1 = entry(kt_begin + it + 2, 1);
                int vprev = (it - 1) % kNumBufsV; // V buffer of tile it - 1
                auto vnext = [](int v, int n) { v += n; return v >= kNumBufsV ? v - kNumBufsV : v; };
                // while every row of the wavefront has the reference 0 (the usual case, see kSnap);
                // otherwise the general step below takes over
                for (; it < fast_end && __builtin_amdgcn_ballot_w64(m_ref != 0.f) == 0; ++it) {
                    const int buf = it & 3;
                    const int kt2 = kt_begin + it + 2;
                    gptr k0, v0, k1, v1;
                    if (kt2 < np_tiles) {
                        const gptr b0 = pages_head + (uint64_t)pg0 * page_bytes;
                        const gptr b1 = pages_head + (uint64_t)pg1 * page_bytes;
                        k0 = b0 + pg_lane_k;
                        v0 = b0 + pg_lane_v;
                        k1 = b1 + pg_lane_k;
                        v1 = b1 + pg_lane_v;
                    } else {
                        const int64_t off = (int64_t)(kt2 - np_tiles) * kBN * row_bytes;
                        k0 = knew_head + off + sfx_lane_k;
                        v0 = vnew_head + off + sfx_lane_v;
                        k1 = k0 + (int64_t)kLoadRows * row_bytes;
                        v1 = v0 + (int64_t)kLoadRows * row_bytes;
                    }
                    dma_tile(k0, v0, k1, v1, (buf + 2) & 3, vnext(vprev, 3));
                    pg0 = entry(kt_begin + it + 3, 0);
                    pg1 = entry(kt_begin + it + 3, 1);
                    STile s;
                    qk_tile(buf, s);
                    float psum = exp_tile(s, pb_b, 0.f, std::true_type{});
                    pv_tile(vprev, pb_a);
                    if (__builtin_amdgcn_ballot_w64(!(psum < kStale) || m_ref == -INFINITY) != 0)
                        psum = redo_tile(s, pb_b);
                    l_run += psum;
                    pair_barrier(it);
                    vprev = vnext(vprev, 1);
#pragma unroll
                    for (int t = 0; t < 2 * kNKB; ++t) pb_a[t] = pb_b[t];
                }
            }
            // the general step: one call site, so that the accumulators stay in the same registers
            const int stop = two_stretches ? min(n_it, np_tiles - kt_begin) : n_it;
            for (; it < stop && !skipped(kt_begin + it); ++it) {
                tile_step(it, pb_b, pb_a);
#pragma unroll
                for (int t = 0; t < 2 * kNKB; ++t) pb_a[t] = pb_b[t];
            }
            if (it >= n_it || skipped(kt_begin + it)) break;
        }
        // P V of the last tile this wavefront computed (tile it - 1)
        pv_tile((it - 1) % kNumBufsV, pb_a);
    }
    // remaining tiles are invisible to this wavefront: only take part in the cooperative loads
    for (; it < n_it; ++it) {
        const bool prefetch = it + 2 < n_it;
        if (prefetch) {
            load_tile(kt_begin + it + 2, it + 2);
        }
        pair_barrier(it);
    }

    // ---- epilogue.  o[db][v] is O^T[d = db*32 + 8*(v/4) + 4*h + v%4][row j]
    const float l_tot = halfwave_sum(l_run);
    if (!row_valid) return;
    if (partial) {
        const int64_t prow = part_row();
        float *po = p.part_o + prow * kD;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                f32x4 x = {o[db][4 * gq], o[db][4 * gq + 1], o[db][4 * gq + 2], o[db][4 * gq + 3]};
                *reinterpret_cast<f32x4 *>(po + db * 32 + 8 * gq + 4 * h) = x;
            }
        if (h == 0) {
            p.part_ml[prow * 2] = m_ref;
            p.part_ml[prow * 2 + 1] = l_tot;
        }
    } else {
        const float inv = 1.f / l_tot;
        uint16_t *po = p.out + (out_row * p.Hq + head) * kD;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                bf16x4 x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = (__bf16)(o[db][4 * gq + e] * inv);
                *reinterpret_cast<bf16x4 *>(po + db * 32 + 8 * gq + 4 * h) = x;
            }
    }
}

// out[row, head, :] = sum_s w_s O_s / sum_s w_s l_s with w_s = 2^(m_s - max_s m_s).
// Entries with l_s = 0 (empty splits) are skipped, and nothing else is: a sum that is not a number, or a value
// behind a weight of 0 that is not, reaches the result as it does without a split.  A row whose scores are
// all minus infinity is 0 / 0 in either case.  Two forms, chosen by the number of splits; in both every
// sum runs in a fixed order, so the result is reproducible.
//
// Many splits: one workgroup per (row, head).  kMergeGroups groups of 32 threads take the splits
// s = g, g + kMergeGroups, ... (at most kMergePerGroup each; 4 consecutive d per thread), then the
// partial sums of the groups are added in group order.
constexpr int kMergeGroups = 32;
constexpr int kMergePerGroup = 8; // splits per group: up to 256 partial results in all
// Up to kMergeFewSplits splits the second form is used, and for as many (row, head) pairs as fill the device up to
// kMergeSomeSplits: the first form then runs many workgroups of 1024 threads after each other.
// Attention and merge of 12 ranges, first and second form: 64 rows x 32 heads 36.4 and 26.7 us; 128 x 32 50.0 and 31.0;
// 256 x 32 162 and 125; of 32 ranges 32 and 25 for 1600 pairs, 191 and 150 for 8192.  One decoded row of 32
// heads, 24 to 64 ranges, is better off with the first form, whose threads share the ranges.
constexpr int kMergeFewSplits = 8, kMergeSomeSplits = 32, kMergeSomeRows = 1024;
__global__ __launch_bounds__(32 * kMergeGroups) void merge_splits_kernel(const float *__restrict__ part_o,
                                                                          const float *__restrict__ part_ml,
                                                                          uint16_t *__restrict__ out,
                                                                          int64_t n_rh, int nsplit)
{
    __shared__ float s_max[kMergeGroups];
    __shared__ float s_den[kMergeGroups];
    __shared__ f32x4 s_acc[kMergeGroups][32];
    const int64_t rh = blockIdx.x;
    const int g = threadIdx.x >> 5, t = threadIdx.x & 31;
    const int d4 = t * 4;
    // all loads of the group first (one round of memory latency), then the arithmetic
    float ms[kMergePerGroup], ls[kMergePerGroup];
    f32x4 x[kMergePerGroup];
#pragma unroll
    for (int i = 0; i < kMergePerGroup; ++i) {
        const int s = g + i * kMergeGroups;
        const bool on = s < nsplit;
        const f32x2 ml = on ? *reinterpret_cast<const f32x2 *>(part_ml + ((int64_t)s * n_rh + rh) * 2) : f32x2{0.f, 0.f};
        ms[i] = ml[0];
        ls[i] = ml[1];
        x[i] = on ? *reinterpret_cast<const f32x4 *>(part_o + ((int64_t)s * n_rh + rh) * kD + d4) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // maximum over all splits: inside the group every thread holds the same values; across groups
    // through LDS
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < kMergePerGroup; ++i)
        if (ls[i] != 0.f) m = fmaxf(m, ms[i]);
    if (t == 0) s_max[g] = m;
    __syncthreads();
    float m_star = s_max[0];
#pragma unroll
    for (int i = 1; i < kMergeGroups; ++i) m_star = fmaxf(m_star, s_max[i]);

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float denom = 0.f;
#pragma unroll
    for (int i = 0; i < kMergePerGroup; ++i)
        if (ls[i] != 0.f) {
            const float w = fast_exp2(ms[i] - m_star);
            acc += x[i] * w;
            denom += ls[i] * w;
        }
    s_acc[g][t] = acc;
    if (t == 0) s_den[g] = denom;
    __syncthreads();
    if (g != 0) return;
#pragma unroll
    for (int i = 1; i < kMergeGroups; ++i) {
        acc += s_acc[i][t];
        denom += s_den[i];
    }
    const float inv = 1.f / denom;
    bf16x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = (__bf16)(acc[e] * inv);
    *reinterpret_cast<bf16x4 *>(out + rh * kD + d4) = y;
}

// Few splits: a group of 32 threads per (row, head), eight of them per workgroup, each walking
// over its splits in order with all loads of a pass in flight together.  Partial result s of a row is row
// first + s * step.
template <int kSplits>
__device__ __forceinline__ void merge_row(const float *__restrict__ part_o, const float *__restrict__ part_ml,
                                          uint16_t *__restrict__ out, int64_t first, int64_t step, int64_t rh, int nsplit)
{
    const int d4 = (threadIdx.x & 31) * 4;
    float ms[kSplits], ls[kSplits];
    f32x4 x[kSplits];
#pragma unroll
    for (int s = 0; s < kSplits; ++s) {
        const bool on = s < nsplit;
        const f32x2 ml = on ? *reinterpret_cast<const f32x2 *>(part_ml + (first + s * step) * 2) : f32x2{0.f, 0.f};
        ms[s] = ml[0];
        ls[s] = ml[1];
        x[s] = on ? *reinterpret_cast<const f32x4 *>(part_o + (first + s * step) * kD + d4) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float m_star = -INFINITY;
#pragma unroll
    for (int s = 0; s < kSplits; ++s)
        if (ls[s] != 0.f) m_star = fmaxf(m_star, ms[s]);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float denom = 0.f;
#pragma unroll
    for (int s = 0; s < kSplits; ++s)
        if (ls[s] != 0.f) {
            const float w = fast_exp2(ms[s] - m_star);
            acc += x[s] * w;
            denom += ls[s] * w;
        }
    const float inv = 1.f / denom;
    bf16x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = (__bf16)(acc[e] * inv);
    *reinterpret_cast<bf16x4 *>(out + rh * kD + d4) = y;
}

template <int kSplits>
__global__ __launch_bounds__(256) void merge_few_splits_kernel(const float *__restrict__ part_o,
                                                               const float *__restrict__ part_ml,
                                                               uint16_t *__restrict__ out, int64_t n_rh, int nsplit)
{
    const int64_t rh = (int64_t)blockIdx.x * 8 + (threadIdx.x >> 5);
    if (rh < n_rh) merge_row<kSplits>(part_o, part_ml, out, rh, n_rh, rh, nsplit);
}

// The row tiles of a batch of equal requests that were split (the last tail_units of every KV head).
constexpr int kMaxTailSplits = 16;
template <int kSplits>
__global__ __launch_bounds__(256) void merge_tail_kernel(const AttnParams p)
{
    constexpr int kBlocks = kBM / 8; // of a row tile
    const int tile = blockIdx.x / kBlocks, i = (int)(blockIdx.x % kBlocks) * 8 + (int)(threadIdx.x >> 5);
    const int kvh = tile / p.tail_units, tail_unit = tile - kvh * p.tail_units;
    const int E = p.extend_lens[0], nt = (int)row_tiles(E, p.G, kTileShift);
    const int r = (p.whole_units + tail_unit) / nt, unit = (p.whole_units + tail_unit) - r * nt;
    const int row = row_tile_of(unit, nt, r, p.batch, p.alternate) * kBM + i;
    if (row >= E * p.G) return;
    const int tok = over_heads(row, p);
    merge_row<kSplits>(p.part_o, p.part_ml, p.out, (int64_t)tile * p.nsplit * kBM + i, kBM,
                       ((int64_t)r * E + tok) * p.Hq + kvh * p.G + (row - tok * p.G), p.nsplit);
}

static_assert(kDecMaxChunks <= kMergeGroups * kMergePerGroup && kMaxSplits <= kMergeGroups * kMergePerGroup,
              "the merge kernel holds all partial results of a row in registers");

// Mixed batches: the rows whose requests have more than one key range (at most kMaxSplits), packed.  A
// workgroup takes one of them and eight heads, 32 threads each: thread t first reads (m, l) of the
// splits t and t + 32, then every thread adds up 4 consecutive d over the splits in order.
constexpr int kMergeHeads = 8;
__global__ __launch_bounds__(32 * kMergeHeads) void merge_mixed_kernel(const MixedParams p)
{
    const int head_blocks = (p.Hq + kMergeHeads - 1) / kMergeHeads;
    const int head = (int)(blockIdx.x % head_blocks) * kMergeHeads + (threadIdx.x >> 5);
    const int lane = threadIdx.x & 63, t = threadIdx.x & 31;
    int row = blockIdx.x / head_blocks; // among the rows to merge
    int ns = 0, E = 0, cu = 0;
    int64_t parts = 0;
    for (int base = 0; base < p.batch; base += 64) {
        const int rr = base + lane;
        const int e = rr < p.batch ? p.extend_lens[rr] : 0;
        const int pl = rr < p.batch ? p.prefix_lens[rr] : 0;
        const int s = splits_of_request(pl, e, p.G, p.seg_tiles, p.dec_blocks);
        const int rows = s > 1 ? e : 0;
        const int incl_r = wave_inclusive_scan(rows, lane);
        const int incl_e = wave_inclusive_scan(e, lane);
        const int incl_p = wave_inclusive_scan(rows * s, lane);
        const int total = __builtin_amdgcn_readlane(incl_r, 63);
        if (row < total) {
            const int first = __builtin_ctzll(__builtin_amdgcn_ballot_w64(incl_r > row));
            row -= __builtin_amdgcn_readlane(incl_r - rows, first);
            cu += __builtin_amdgcn_readlane(incl_e - e, first);
            parts += __builtin_amdgcn_readlane(incl_p - rows * s, first);
            E = __builtin_amdgcn_readlane(e, first);
            ns = __builtin_amdgcn_readlane(s, first);
            break;
        }
        row -= total;
        cu += __builtin_amdgcn_readlane(incl_e, 63);
        parts += __builtin_amdgcn_readlane(incl_p, 63);
    }
    if (head >= p.Hq) return;
    const int64_t first = (parts + row) * p.Hq + head, step = (int64_t)E * p.Hq; // partial result s: first + s * step
    f32x2 ml[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        ml[i] = t + 32 * i < ns ? *reinterpret_cast<const f32x2 *>(p.part_ml + (first + (t + 32 * i) * step) * 2) : f32x2{0.f, 0.f};
    float m_star = fmaxf(ml[0][1] != 0.f ? ml[0][0] : -INFINITY, ml[1][1] != 0.f ? ml[1][0] : -INFINITY);
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) m_star = fmaxf(m_star, __shfl_xor(m_star, off, 32));
    float w[2]; // -1: an empty range, which left no values
#pragma unroll
    for (int i = 0; i < 2; ++i) w[i] = ml[i][1] != 0.f ? fast_exp2(ml[i][0] - m_star) : -1.f;
    float denom = ml[0][1] * w[0] + ml[1][1] * w[1];
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) denom += __shfl_xor(denom, off, 32);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    // `many` loads in flight at a time: a decode row has up to kMaxSplits partial results and few others beside it
    auto add_up = [&](auto many) {
        constexpr int kMany = decltype(many)::value;
        for (int s0 = 0; s0 < ns; s0 += kMany) {
            f32x4 x[kMany];
#pragma unroll
            for (int i = 0; i < kMany; ++i)
                x[i] = s0 + i < ns ? *reinterpret_cast<const f32x4 *>(p.part_o + (first + (s0 + i) * step) * kD + t * 4)
                                   : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < kMany; ++i) {
                const float ws = __shfl(s0 < 32 ? w[0] : w[1], (s0 + i) & 31, 32);
                if (!(ws < 0.f)) acc += x[i] * ws; // a weight that is not a number counts
            }
        }
    };
    if (ns <= 4) add_up(std::integral_constant<int, 4>{});
    else add_up(std::integral_constant<int, 16>{});
    const float inv = 1.f / denom;
    bf16x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = (__bf16)(acc[e] * inv);
    *reinterpret_cast<bf16x4 *>(p.out + ((int64_t)(cu + row) * p.Hq + head) * kD + t * 4) = y;
}

// A wavefront copies four consecutive packed rows of two KV heads; thread (row, 16-byte chunk).  It finds
// the requests of its rows 64 at a time (a prefix sum of extend_lens across the lanes).  For a few rows
// the time is the chain of dependent loads: lengths, then the block table, then the store.  The rows
// themselves do not wait for it, they are requested first.  With all heads in one wavefront, two at a
// time, the chain goes on: 32 rows, 8 KV heads 3.1 us a launch with two heads, 3.4 with four, 3.9 with eight
// (5.8-6.5 with the rows requested after the table); 8000 rows 10.9, 11.4, 12.0; 18432 rows 23.9, 23.7, 24.2
// (6.3 TB/s); 32768 rows 43.2, 45.0, 47.6.
constexpr int kWriteRows = 16; // rows per workgroup
constexpr int kWriteHeads = 2; // KV heads per workgroup
__global__ __launch_bounds__(256) void write_kv_kernel(const uint16_t *__restrict__ k_new,
                                                       const uint16_t *__restrict__ v_new,
                                                       uint16_t *__restrict__ kv_pages,
                                                       const int32_t *__restrict__ block_table,
                                                       const int32_t *__restrict__ prefix_lens,
                                                       const int32_t *__restrict__ extend_lens,
                                                       int batch, int Hkv, int max_pages, int T)
{
    const int lane = threadIdx.x & 63;
    const int groups = (Hkv + kWriteHeads - 1) / kWriteHeads; // workgroups that share the rows
    const int row0 = (int)(blockIdx.x / groups) * kWriteRows + (int)(threadIdx.x >> 6) * 4;
    const int head0 = (int)(blockIdx.x % groups) * kWriteHeads, head1 = min(head0 + 1, Hkv - 1);
    if (row0 >= T) return;
    const int row = row0 + (lane >> 4);
    const int ch = lane & 15; // 16-byte chunk of a 256-byte head row
    const int64_t src = (int64_t)min(row, T - 1) * Hkv * kD + ch * 8;
    // the last of an odd number of heads is copied twice: the same bytes to the same place
    const uint4 k0 = *reinterpret_cast<const uint4 *>(k_new + src + (int64_t)head0 * kD);
    const uint4 v0 = *reinterpret_cast<const uint4 *>(v_new + src + (int64_t)head0 * kD);
    const uint4 k1 = *reinterpret_cast<const uint4 *>(k_new + src + (int64_t)head1 * kD);
    const uint4 v1 = *reinterpret_cast<const uint4 *>(v_new + src + (int64_t)head1 * kD);

    int req = -1, tok = 0; // owner of this thread's row and the row's token inside it
    int cu = 0;            // rows of the requests before `base`
    for (int base = 0; base < batch; base += 64) {
        const int rr = base + lane;
        const int e = rr < batch ? extend_lens[rr] : 0;
        const int pl = rr < batch ? prefix_lens[rr] : 0;
        const int incl = wave_inclusive_scan(e, lane);
        const int total = __builtin_amdgcn_readlane(incl, 63);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = row0 + i - cu; // the row's index among the rows of this group of requests
            if (t >= 0 && t < total) {
                const int first = __builtin_ctzll(__builtin_amdgcn_ballot_w64(incl > t));
                const int at = __builtin_amdgcn_readlane(pl - incl + e, first) + t;
                if ((lane >> 4) == i) {
                    req = base + first;
                    tok = at;
                }
            }
        }
        if (row0 + 3 - cu < total) break;
        cu += total;
    }
    if (req < 0 || row >= T) return;
    const int64_t page = block_table[(int64_t)req * max_pages + (tok >> 4)];
    uint16_t *kdst = kv_pages + ((page * 2 * Hkv) * kPS + (tok & 15)) * (int64_t)kD + ch * 8;
    uint16_t *vdst = kdst + (int64_t)Hkv * kPS * kD;
    const int64_t head_pitch = (int64_t)kPS * kD; // one KV head's slab inside a page
    *reinterpret_cast<uint4 *>(kdst + head0 * head_pitch) = k0;
    *reinterpret_cast<uint4 *>(vdst + head0 * head_pitch) = v0;
    *reinterpret_cast<uint4 *>(kdst + head1 * head_pitch) = k1;
    *reinterpret_cast<uint4 *>(vdst + head1 * head_pitch) = v1;
}


// ---- optional check of the device-side tables ------------------------------------------------
// The attention and append kernels trust block_table and the device copies of the lengths.  This
// kernel reads them without following any page id: thread (request r, slot i) looks at
// block_table[r][i] for the slots the request uses, i < ceil((P_r + E_r) / 16), with P_r and E_r
// taken from the device arrays, and records the first offence (smallest code of request and slot)
// in one 64-bit word.
constexpr int kCheckThreads = 256;
enum : uint32_t { kCheckOk = 0u, kCheckBadLength = 1u, kCheckBadPage = 2u };
__global__ __launch_bounds__(kCheckThreads) void check_tables_kernel(const int32_t *__restrict__ block_table,
                                                                     const int32_t *__restrict__ prefix_lens,
                                                                     const int32_t *__restrict__ extend_lens,
                                                                     int batch, int max_pages, int num_pages,
                                                                     unsigned long long *__restrict__ first_bad)
{
    const int r = blockIdx.y;
    if (r >= batch) return;
    const int64_t P = prefix_lens[r], E = extend_lens[r];
    const int64_t used = (P + E + kPS - 1) / kPS;
    // key of an offence: kind in the top bits so that a bad length outranks a bad page, then the
    // request, then the slot; the smallest key wins
    auto report = [&](uint32_t kind, int slot) {
        const unsigned long long key = ((unsigned long long)(kind == kCheckBadLength ? 0u : 1u) << 62) |
                                       ((unsigned long long)(uint32_t)r << 31) | (unsigned long long)(uint32_t)slot;
        atomicMin(first_bad, key);
    };
    if (P < 0 || E < 0 || used > max_pages) {
        if (blockIdx.x == 0 && threadIdx.x == 0) report(kCheckBadLength, 0);
        return;
    }
    for (int64_t i = (int64_t)blockIdx.x * kCheckThreads + threadIdx.x; i < used; i += (int64_t)gridDim.x * kCheckThreads) {
        const int32_t page = block_table[(int64_t)r * max_pages + i];
        if (page < 0 || page >= num_pages) report(kCheckBadPage, (int)i);
    }
}

// Scratch of the check above and of the entry point that takes no workspace: file-scope device
// arrays, so that no call allocates.  In host code the arrays' names are stand-ins, not device
// addresses; the per-device address comes from hipGetSymbolAddress (device_scratch below).
__device__ __align__(256) unsigned long long g_check_report[32];

// ------------------------------------------------------------------ host side
struct Plan {
    int64_t q_tiles = 0; // row tiles per KV head, summed over requests
    int32_t max_key_tiles = 0;
    int32_t nsplit = 1;
    bool decode = false;    // few rows per (request, KV head): decode_attn_kernel
    int32_t row_blocks = 1; // ... in this many blocks of 32 rows
    int32_t dec_groups = 1; // ... by this many workgroups that share a request's keys
    int32_t dec_share = 1;  // ... with this many blocks of rows per wavefront
    bool small = false; // few rows and keys: decode_attn_kernel with a workgroup per block of 32 rows
    int32_t tile_shift = kTileShift;
    int32_t tail_units = 0; // row tiles per KV head that are split, the last ones of the list; 0: all or none
    bool mixed = false; // unequal lengths: extend_attn_kernel<kMixed>, with
    int32_t seg_tiles = 1, dec_blocks = 1;       // at most so many keys per item
    int64_t row_items = 0, dec_units = 0;        // row-tiled items and decode wavefronts per KV head
    int64_t merge_rows = 0, part_rows = 0;       // rows with more than one key range, their partial results
};

// Compute units of the device the first caller runs on (every device this library is built
// for has the same count); read once, any number of host threads may race to be that caller.
int num_cus()
{
    static std::atomic<int> cached{0};
    int n = cached.load(std::memory_order_relaxed);
    if (n == 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cached.store(n, std::memory_order_relaxed);
    }
    return n;
}

// The attention kernel uses more LDS than the default per-workgroup limit; raise it once.
bool allow_large_lds()
{
    static std::once_flag once;
    static bool ok = false;
    std::call_once(once, [] {
        const hipError_t a = hipFuncSetAttribute(reinterpret_cast<const void *>(&extend_attn_kernel<kWhole>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        const hipError_t b = hipFuncSetAttribute(reinterpret_cast<const void *>(&extend_attn_kernel<kSplit>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        const hipError_t c = hipFuncSetAttribute(reinterpret_cast<const void *>(&extend_attn_kernel<kMixed>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kMixedLdsBytes);
        ok = a == hipSuccess && b == hipSuccess && c == hipSuccess;
    });
    return ok;
}

int validate(const cp_shape *s)
{
    if (!s) return CP_ERR_NULL;
    if (!s->h_prefix_lens || !s->h_extend_lens) return CP_ERR_NULL;
    if (s->batch < 1 || s->num_q_heads < 1 || s->num_kv_heads < 1) return CP_ERR_SHAPE;
    if (s->num_q_heads % s->num_kv_heads != 0) return CP_ERR_SHAPE;
    if (s->head_dim != kD || s->page_size != kPS) return CP_ERR_SHAPE;
    if (s->num_pages < 1 || s->max_pages_per_req < 1 || s->total_extend < 0) return CP_ERR_SHAPE;
    if (!(s->softmax_scale > 0.f) || !(s->softmax_scale < 3.0e38f)) return CP_ERR_SHAPE;
    if (s->num_splits < 0 || s->num_splits > kMaxSplits) return CP_ERR_SHAPE;
    int64_t sum = 0;
    for (int r = 0; r < s->batch; ++r) {
        const int64_t P = s->h_prefix_lens[r], E = s->h_extend_lens[r];
        if (P < 0 || E < 0) return CP_ERR_SHAPE;
        if ((P + E + kPS - 1) / kPS > s->max_pages_per_req) return CP_ERR_SHAPE;
        if (P + E > INT32_MAX - 2 * kBM) return CP_ERR_SHAPE;
        sum += E;
    }
    if (sum != s->total_extend) return CP_ERR_SHAPE;
    return CP_OK;
}

bool equal_lengths(const cp_shape *s)
{
    for (int r = 1; r < s->batch; ++r)
        if (s->h_prefix_lens[r] != s->h_prefix_lens[0] || s->h_extend_lens[r] != s->h_extend_lens[0]) return false;
    return true;
}

// The row tiles that a plan counts: of 256 rows, of 128, or of the rows of 1, 2, 4 or 8 whole q heads, the least number
// that leaves no head fewer rows than E.  No kernel runs the last ones any more, but callers have sized
// their scratch by them: see too_little_scratch.
enum TileKind { kFullTiles, kHalfTiles, kWholeHeads, kTileKinds };
constexpr int shift_of(TileKind kind) { return kind == kHalfTiles ? kTileShift - 1 : kTileShift; }
struct TileCount {
    int64_t tiles;   // of one request and KV head
    int64_t lengths; // how many of them have different numbers of keys
};
TileCount count_tiles(int64_t E, int G, TileKind kind)
{
    if (kind != kWholeHeads) {
        const int64_t n = row_tiles((int)E, G, shift_of(kind));
        return {n, n};
    }
    int shift = 0; // the heads' logarithm
    while (shift < 3 && (G & ((2 << shift) - 1)) == 0 && E << (shift + 1) <= kBM) ++shift;
    return {((E << shift) + kBM - 1) / kBM * (G >> shift), (E + kBM - 1) / kBM};
}

// What the plans of a call are made from.  A call is planned up to four times (tiles of 256 rows and of 128,
// tiles of whole heads, less scratch); its lengths are read and its requests sorted once for all of them, and a search ends
// where its answer is known.  With a table, a sort and a search to the end for every plan the host of an MI355X took 4.0 us for a batch
// of 40 requests, 32 of which decode, now 1.8; for 512, 410 of which do, 53 and 23; for 32 equal ones, 128 new tokens, 0.54 and 0.06.
struct RowWork { // of one kind of tile
    int64_t q_tiles = 0; // row tiles of a KV head
    double tiles = 0.0;  // key tiles of all row tiles and KV heads
    bool alike = true;   // no request has row tiles of different lengths
    bool known = false;
};
class Requests {
public:
    explicit Requests(const cp_shape *s);
    const RowWork &work(TileKind kind);                          // fills units[kind] and mean[kind] too
    void write_order(uint8_t *order) const;                      // MixedParams::order

    const cp_shape *const s;
    const int G;
    bool equal = true;        // all requests have the same lengths
    bool by_request = false;  // a plan that splits request by request is one to look at, and what follows is there
    bool decode_rows = false; // some, not all, are decode-shaped
    int64_t max_e = 0, max_n = 0;  // most new tokens, most keys
    int64_t row_blocks = 0;        // blocks of 32 rows per KV head, the most of a request
    int32_t max_key_tiles = 0;
    int64_t decode_work = 0;       // key blocks of all decode wavefronts
    int64_t all_dec_units = 0;     // row blocks of all decode-shaped requests
    int32_t key_blocks = 1;        // of 32, the most of a decode-shaped request
    int32_t range_tiles = 1;       // key tiles of the longest request, with two blocks of a decode-shaped one to a tile
    // Requests with new tokens: row-tiled ones first, most keys first
    int32_t n = 0, row_tiled = 0;  // all, and how many are row-tiled
    int32_t index[kMixedMaxBatch]; // in the batch
    int32_t extend[kMixedMaxBatch];
    int32_t length[kMixedMaxBatch];            // key tiles of the last row tile, or key blocks of 32
    int32_t dec_units[kMixedMaxBatch];         // row blocks of a decode-shaped request
    int64_t units[kTileKinds][kMixedMaxBatch]; // row tiles of a row-tiled one
    float mean[kTileKinds][kMixedMaxBatch];    // key tiles of a row tile on average

private:
    RowWork work_[kTileKinds];
    int16_t place_[kMixedMaxBatch]; // in the arrays above, by request
};

Requests::Requests(const cp_shape *shape) : s(shape), G(shape->num_q_heads / shape->num_kv_heads)
{
    const int32_t *const prefix = s->h_prefix_lens, *const added = s->h_extend_lens;
    for (int r = 1; r < s->batch && equal; ++r) equal = prefix[r] == prefix[0] && added[r] == added[0];
    by_request = !equal && s->batch <= kMixedMaxBatch;
    uint64_t key[kMixedMaxBatch];
    for (int r = 0; r < (equal ? 1 : s->batch); ++r) {
        const int32_t P = prefix[r], E = added[r];
        if (E == 0) continue;
        max_e = std::max<int64_t>(max_e, E);
        max_n = std::max<int64_t>(max_n, (int64_t)P + E);
        const int32_t tiles = (P + kBN - 1) / kBN + (E + kBN - 1) / kBN;
        max_key_tiles = std::max(max_key_tiles, tiles);
        if (!by_request) continue;
        const bool decode = decode_shaped(E, G);
        const int32_t keys = decode ? (P + E + 31) / 32 : tiles;
        decode_rows = decode_rows || decode;
        row_tiled += !decode;
        key[n++] = (uint64_t)decode << 63 | (uint64_t)(INT32_MAX - keys) << 32 | (uint32_t)r;
    }
    row_blocks = (max_e * G + kDecRows - 1) / kDecRows;
    if (!by_request) return;
    std::sort(key, key + n);
    for (int i = 0; i < n; ++i) {
        const int r = (int)(uint32_t)key[i];
        index[i] = r;
        place_[r] = (int16_t)i;
        extend[i] = added[r];
        length[i] = INT32_MAX - (int32_t)(key[i] >> 32 & INT32_MAX);
        if (i < row_tiled) continue;
        dec_units[i] = (extend[i] * G + kDecRows - 1) / kDecRows;
        all_dec_units += dec_units[i];
        decode_work += (int64_t)dec_units[i] * length[i] * s->num_kv_heads;
    }
    if (row_tiled > 0) range_tiles = std::max(range_tiles, length[0]);
    if (row_tiled < n) {
        key_blocks = std::max(key_blocks, length[row_tiled]);
        range_tiles = std::max(range_tiles, (length[row_tiled] + 1) / 2);
    }
}

const RowWork &Requests::work(TileKind kind)
{
    RowWork &w = work_[kind];
    if (w.known) return w;
    w.known = true;
    const int batch = equal ? 1 : s->batch;
    for (int r = 0; r < batch; ++r) {
        const int64_t P = s->h_prefix_lens[r], E = s->h_extend_lens[r];
        if (E == 0) continue;
        const TileCount c = count_tiles(E, G, kind);
        const int64_t before = (P + kBN - 1) / kBN, own = (E + kBN - 1) / kBN;
        w.alike = w.alike && c.lengths == 1;
        w.q_tiles += c.tiles;
        w.tiles += (double)c.tiles * s->num_kv_heads * ((double)before + 0.5 * (double)own * (1.0 + 1.0 / (double)c.lengths));
        if (!by_request || place_[r] >= row_tiled) continue;
        units[kind][place_[r]] = c.tiles;
        mean[kind][place_[r]] = (float)before + 0.5f * (float)own * (1.f + 1.f / (float)c.lengths);
    }
    if (equal) {
        w.q_tiles *= s->batch;
        w.tiles *= s->batch;
    }
    return w;
}

void Requests::write_order(uint8_t *order) const
{
    int at[kMixedMaxBatch / 64];
    for (int g = 0; g < kMixedMaxBatch / 64; ++g) at[g] = 64 * g;
    bool placed[kMixedMaxBatch] = {};
    for (int i = 0; i < n; ++i) {
        order[at[index[i] / 64]++] = (uint8_t)(index[i] % 64);
        placed[index[i]] = true;
    }
    for (int r = 0; r < (s->batch + 63) / 64 * 64; ++r) // no new tokens, or behind the batch's last request
        if (!placed[r]) order[at[r / 64]++] = (uint8_t)(r % 64);
}

size_t part_bytes(size_t rows, int heads)
{
    const size_t n = rows * (size_t)heads;
    return ((n * kD * sizeof(float) + 255) / 256) * 256 + ((n * 2 * sizeof(float) + 255) / 256) * 256;
}

// Plan of a mixed batch: the key ranges with the least estimated time.  What the estimate is made of,
// in us: a row-tiled item costs kItemUs and kTileUs per key tile of 64 on one CU, a decode workgroup (8
// wavefronts) kItemUs and kBlockUs per block of 32 keys; partial results are written and read once.
// Tiles of half the rows are for calls whose tiles do not fill the device: four wavefronts with a SIMD each take two
// thirds of the time of eight, and there are twice as many.  8/2 heads, P = 0: 3 requests, E = 959 28.0 -> 21.8 us;
// 17, E = 134 11.5 -> 10.0; 32/8 heads, 4, P = 0, E = 214 13.6 -> 11.4.  Two rounds of them are slower than one of full
// tiles (6 requests, P = 978, E = 842, 8/2 heads: 63 us, 52), so they have to fit the CUs at once, and they have to
// promise kHalfUs more, for their start costs more than an item's in a list (1 request, E = 124, 64/8 heads: 9.4 us as
// half tiles, 7.1 as a small call, which the estimates without it put the other way round).
constexpr double kHalfTileUs = 1.2, kHalfUs = 1.5;
constexpr double kItemUs = 4.0, kTileUs = 1.75, kBlockUs = 3.0, kMergeUs = 5.0, kPartBytesPerUs = 4.0e6;
// Batches of unequal lengths: what follows the items of a request at least (a part of its item's length), what the merge
// takes, and what a plan without a split counts for against one with.  Of sets of constants tried on 373 random batches
// those below choose plans that take 4.1 % more than the best number of ranges of each; the first ones, with
// which the line of too_little_scratch was drawn and which stay for it, 5.3 %.
struct UnequalCosts {
    double end, merge_us, part_bytes_per_us, last_item, unsplit;
    bool rounds; // items of one length take whole rounds over the CUs
};
constexpr UnequalCosts kUnequal{0.4, 6.0, 3.2e6, 0.5, 1.0, true}, kUnequalOfWholeHeads{0.5, kMergeUs, kPartBytesPerUs, 0.75, 0.85, false};
// x rounded up, for 0 <= x < 2^53
inline double round_up(double x)
{
    const double whole = (double)(int64_t)x;
    return whole < x ? whole + 1.0 : whole;
}

// Fills pl for at most seg_tiles key tiles per row-tiled item; returns the time, or any that is no less than `bound` if
// that is too long, and then pl is not filled.
double mixed_cost(const Requests &q, TileKind kind, int seg_tiles, int dec_blocks, const UnequalCosts &c, double bound, Plan &pl)
{
    pl.mixed = true;
    pl.tile_shift = shift_of(kind);
    pl.seg_tiles = seg_tiles;
    pl.dec_blocks = dec_blocks;
    // One KV head on its share of the CUs, in the order of the list: the items of the first requests alone take their sum
    // over the CUs and a part of the last one's length, no less than the longest, and no less than some CU
    // takes that has as many of them as the others or one more.
    const double per_cu = q.s->num_kv_heads / (double)num_cus(), tile_us = kind == kHalfTiles ? kHalfTileUs : kTileUs;
    double work = 0.0, most = 0.0, items = 0.0, shortest = 1e30; // of the items so far
    // ranges as in splits_of_request; a decode request has at most kMaxSplits by the choice of dec_blocks
    auto add = [&](int i, int limit, int64_t units, double mean, double step, double share) {
        const int length = q.length[i], ns = length <= limit ? 1 : std::min(kMaxSplits, (length + limit - 1) / limit);
        const double keys = mean * step, each = ns == 1 ? keys : keys / ns;
        const int longest = ns == 1 ? length : (length + ns - 1) / ns;
        work += (double)units * (ns * kItemUs + keys) * share;
        const double item = kItemUs + step * longest;
        most = std::max(most, std::max(item, work * per_cu + c.end * item));
        items += (double)(units * ns) * share;
        shortest = std::min(shortest, kItemUs + each);
        if (c.rounds) most = std::max(most, round_up(items * per_cu) * shortest);
        pl.nsplit = std::max(pl.nsplit, ns);
        if (ns > 1) {
            pl.merge_rows += q.extend[i];
            pl.part_rows += (int64_t)ns * q.extend[i];
        }
        return units * ns;
    };
    for (int i = 0; i < q.row_tiled && most < bound; ++i)
        pl.row_items += add(i, seg_tiles, q.units[kind][i], q.mean[kind][i], tile_us, 1.0);
    for (int i = q.row_tiled; i < q.n && most < bound; ++i)
        pl.dec_units += add(i, dec_blocks, q.dec_units[i], (float)q.length[i], kBlockUs, 1.0 / kWaves);
    double us = most;
    if (pl.part_rows > 0) us += c.merge_us + 2.0 * (double)part_bytes((size_t)pl.part_rows, q.s->num_q_heads) / c.part_bytes_per_us;
    return us;
}

// The best plan whose partial results fit into `room` bytes, and its time; false if there is none.  One that takes less
// than `enough` ends the search.
bool plan_mixed(Requests &q, size_t room, TileKind kind, Plan &best, double *estimate, double enough = -1.0)
{
    const cp_shape *const s = q.s;
    const int tiles = q.range_tiles;
    const RowWork &w = q.work(kind);
    // No plan has more partial results or items than there is room for: then one that turns out too slow need not be
    // added up to the end.
    const int64_t most_rows = (int64_t)s->total_extend * kMaxSplits, most_items = (w.q_tiles + q.all_dec_units) * kMaxSplits * s->num_kv_heads;
    const bool all_fit = most_rows <= INT32_MAX / 2 && most_items <= INT32_MAX / 2 && part_bytes((size_t)most_rows, s->num_q_heads) <= room;
    double best_us = -1.0;
    int worse = 0;
    for (int pieces = 1; pieces <= kMaxSplits && worse < 4; pieces += pieces < 8 ? 1 : pieces / 4) {
        const int seg = (tiles + pieces - 1) / pieces;
        if (pieces > 1 && seg < 2) break;
        // A decode wavefront's chunk takes about as long as a row-tiled item, but is no shorter than
        // twice its share of the decode work (8 wavefronts per CU), 4 to 16 blocks: finer chunks only
        // give the merge more to read (21 requests, 218 MB of decode K/V: 16 blocks 49 us, 8: 52, 4: 57).
        const int least = (int)std::min<int64_t>(16, std::max<int64_t>(4, 2 * q.decode_work / (8 * num_cus())));
        const int dec = std::max(std::max(least, (int)(seg * (kTileUs / kBlockUs))), (q.key_blocks + kMaxSplits - 1) / kMaxSplits);
        Plan pl;
        const double us = mixed_cost(q, kind, seg, dec, kind == kWholeHeads ? kUnequalOfWholeHeads : kUnequal,
                                     all_fit && best_us >= 0.0 ? best_us : HUGE_VAL, pl);
        if (pl.part_rows > INT32_MAX / 2 || (pl.part_rows > 0 && part_bytes((size_t)pl.part_rows, s->num_q_heads) > room)) continue;
        if ((pl.row_items + (pl.dec_units + kWaves - 1) / kWaves) * s->num_kv_heads > INT32_MAX / 2) continue;
        worse = best_us >= 0.0 && us >= best_us ? worse + 1 : 0;
        if (worse == 0) {
            best_us = us;
            best = pl;
            if (us < enough) break;
        }
    }
    *estimate = best_us;
    return best_us >= 0.0;
}

// A bound that is left out of a search counts for a little less, so that rounding cannot make it one that is not.
constexpr double kNearly = 1.0 - 1e-9;

// One number of key ranges for all requests: the least estimated time (see above).  A grid
// of two workgroups per CU is not split: it gains nothing then.  Row tiles of one length run in whole
// rounds over the CUs; if a request has several, of different lengths, the last round is about half empty.
// In a batch of unequal lengths the longest item may be among the last to begin, and more ranges than the cheaper merge
// takes are for the plan that splits only the requests which need it (10 requests, 39 ranges 36 us, 25).
// Against ranges of at least 8 tiles, two workgroups per CU: P = 512, E = 128, 8/2 heads (4 workgroups
// of 10 tiles before) 25.2 -> 19.0 us; 4 requests, P = 3000, E = 128, 32/8 heads 61 -> 45; 1 request,
// P = 2000, E = 700, 64/8 heads 100 -> 72; 12 requests, P = 20000, E = 128, 32/8 heads 538 -> 496.
void choose_splits(Requests &q, TileKind kind, size_t room, Plan &pl, double *estimate)
{
    const cp_shape *const s = q.s;
    const RowWork &w = q.work(kind);
    const double tile_us = kind == kHalfTiles ? kHalfTileUs : kTileUs;
    const bool mixed = q.by_request; // a plan to compare this one with
    const UnequalCosts &c = kind == kWholeHeads ? kUnequalOfWholeHeads : kUnequal;
    const int64_t items = w.q_tiles * s->num_kv_heads, cus = num_cus();
    pl.tile_shift = shift_of(kind);
    pl.q_tiles = w.q_tiles;
    pl.max_key_tiles = q.max_key_tiles;
    double best_us = 0.0;
    *estimate = 0.0;
    if (items >= 2 * cus && !mixed) return;
    const int32_t most = items >= 2 * cus ? 1 : std::min(mixed ? kMergeSomeSplits : kMaxSplits, std::max(1, pl.max_key_tiles / 2));
    for (int32_t ns = 1; ns <= most; ++ns) {
        const size_t bytes = ns > 1 ? part_bytes((size_t)ns * (size_t)s->total_extend, s->num_q_heads) : 0;
        if (bytes > room) break;
        const double merge = ns > 1 ? kMergeUs + 2.0 * (double)bytes / kPartBytesPerUs : 0.0;
        // more ranges than CUs: no less than the work, whose part that grows with the ranges takes no more ranges from here on
        if (ns > 1 && items * ns > cus && ((double)(items * ns) * kItemUs + tile_us * w.tiles) / (double)cus * kNearly + merge >= best_us) break;
        const double longest = kItemUs + tile_us * ((pl.max_key_tiles + ns - 1) / ns);
        const double mean = kItemUs + tile_us * w.tiles / ((double)items * ns);
        double us = longest;
        if (items * ns > cus && mixed)
            us = std::max(us, mean * ((double)(items * ns) / (double)cus) + c.last_item * longest);
        else if (items * ns > cus)
            us = std::max(us, w.alike ? (double)((items * ns + cus - 1) / cus) * mean : mean * ((double)(items * ns) / (double)cus + 0.5));
        us += merge;
        if (ns == 1 || us < best_us) {
            best_us = ns == 1 ? c.unsplit * us : us; // a split has to promise more than the estimate is off by
            pl.nsplit = ns;
            *estimate = us;
        }
    }
}

// Time of items that the CUs take one after another: their work and an uneven end, unless the CUs that take one
// more than the others (the shortest, if those are last) are later.  Against the list run item by item, 5000 random
// batches of equal requests: 0.99 of the time in the middle, 0.93 and 1.02 with a tenth of the batches outside.
double rounds_us(double items, double cus, double work, double shortest, double longest)
{
    if (items <= cus) return longest;
    const double rounds = std::ceil(items / cus), last = items - (rounds - 1.0) * cus, more = rounds * last / items;
    const double uneven = 0.2 * (longest - shortest) + (last < cus ? 0.2 * shortest : 0.0);
    return std::max(work / cus + uneven, rounds * (shortest + 0.5 * more * (longest - shortest)));
}

// Time of a key tile in the last row tile of a request, as a part of a full one's: a straight line through what was
// measured, which has a step where the fifth wavefront with rows is the second of a SIMD.  With 1 or 2, 4, 5, 6, 7 and 8 such wavefronts
// 1.32, 1.46, 1.76, 1.88, 2.04 and 2.16 us a tile (256 workgroups, no two with the same keys), that is 0.61, 0.68, 0.81, 0.87, 0.94
// and 1; the line has 0.65, 0.65, 0.74, 0.83, 0.91 and 1.  The plans are the same with either, but for 235 of 20000 random shapes of equal
// requests, and 70 of these took 0.997 of the time with the measured shares, 0.84 to 1.28: the estimate is not that good.
double last_tile_share(int64_t E, int G, TileKind kind)
{
    const int waves = (int)((E * G - 1) % kBM) / 32 + 1;
    if (kind != kFullTiles) return 1.0;
    return waves <= 4 ? 0.65 : 0.65 + 0.0875 * (waves - 4);
}

// The same for equal requests, which also have a third way: the items that would run in a last round of few are
// split, the others are not (pl.tail_units).  Then the call ends with all CUs busy, and only the rows of the last
// items are merged.  3 requests, P = 30000, E = 1100, 64/8 heads (105 items for 32 CUs) 3090 -> 2787 us; 6, P = 9046,
// E = 171 (36) 329 -> 290; 1, P = 10694, E = 2051, 32/8 heads (33) 405 -> 346; 33, P = 1500, E = 70, 8/8 heads (33) 67 -> 56.
// With 1, 2 or 4 KV heads and contiguous ranges for the XCDs (see work_item) there is no common last round.
constexpr double kTailGain = 0.97; // of the time without
bool contiguous_ranges(const cp_shape *s, const Plan &pl, int64_t items, int xcds);
void choose_equal_splits(const Requests &q, TileKind kind, size_t room, Plan &pl, double *estimate)
{
    const cp_shape *const s = q.s;
    const int G = s->num_q_heads / s->num_kv_heads, E = s->h_extend_lens[0], Hkv = s->num_kv_heads;
    const double cus = (double)num_cus() / Hkv; // that share the list of a KV head
    const double tile_us = kind == kHalfTiles ? kHalfTileUs : kTileUs;
    pl.tile_shift = shift_of(kind);
    const int64_t nt = row_tiles(E, G, pl.tile_shift), units = nt * s->batch;
    pl.q_tiles = units;
    pl.max_key_tiles = q.max_key_tiles;
    auto own_tiles = [&](int64_t t) { return (double)((std::min<int64_t>(E, (((t + 1) << pl.tile_shift) + G - 1) / G) + kBN - 1) / kBN); };
    const double prefix = (double)(((int64_t)s->h_prefix_lens[0] + kBN - 1) / kBN);
    const double last = last_tile_share(E, G, kind), one = nt == 1 ? last : 1.0;
    const double shortest = one * (prefix + own_tiles(0)), longest = one * (prefix + own_tiles(nt - 1));
    const double n = (double)units, tiles = ((double)(nt - 1) + last) * s->batch * (prefix + 0.5 * (own_tiles(0) + own_tiles(nt - 1)));
    double best_us = 0.0;
    const int32_t most = n >= 4.0 * cus ? 1 : std::min(kMaxSplits, std::max(1, pl.max_key_tiles / 2));
    for (int32_t ns = 1; ns <= most; ++ns) {
        const size_t bytes = ns > 1 ? part_bytes((size_t)ns * (size_t)s->total_extend, s->num_q_heads) : 0;
        if (bytes > room) break;
        const double merge = ns > 1 ? kMergeUs + 2.0 * (double)bytes / kPartBytesPerUs : 0.0, work = n * ns * kItemUs + tile_us * tiles;
        if (ns > 1 && n * ns > cus && work / cus * kNearly + merge >= best_us) break; // nor do more ranges take less
        const double us = rounds_us(n * ns, cus, work, kItemUs + tile_us * shortest / ns, kItemUs + tile_us * std::ceil(longest / ns)) + merge;
        if (ns == 1 || us < best_us) {
            best_us = ns == 1 ? 0.9 * us : us; // a split has to promise more than the estimate is off by
            pl.nsplit = ns;
            *estimate = us;
        }
    }
    const int64_t per_round = num_cus() / Hkv;
    if (pl.tile_shift != kTileShift) return;
    if (Hkv > kXcds || kXcds % Hkv != 0 || units <= per_round || units % per_round == 0 || units > INT32_MAX / kMaxTailSplits) return;
    if (Hkv < kXcds && contiguous_ranges(s, pl, units * pl.nsplit, kXcds / Hkv)) return;
    best_us = std::min(kTailGain * *estimate, best_us);
    // They are the shortest of the last request, as far as that has as many.  With a whole round more split the estimate was never
    // lower (60000 random shapes of equal requests, 1008 with a last round split).
    const int64_t tail = units % per_round;
    const double tail_longest = tail < nt ? prefix + own_tiles(tail - 1) : longest;
    const double whole = (n - (double)tail) * kItemUs + tile_us * (tiles - (double)tail * 0.5 * (shortest + tail_longest));
    for (int32_t ns = 2; ns <= kMaxTailSplits && 2 * ns <= (int32_t)shortest; ++ns) {
        const size_t bytes = part_bytes((size_t)(tail * ns) * kBM, Hkv);
        if (bytes > room) break;
        const double us = whole / cus + std::ceil((double)(tail * ns) / cus) * (kItemUs + tile_us * std::ceil(tail_longest / ns)) +
                          kMergeUs + 2.0 * (double)bytes / kPartBytesPerUs;
        if (us >= best_us) continue;
        best_us = us;
        *estimate = us;
        pl.nsplit = ns;
        pl.tail_units = (int32_t)tail;
    }
}

// Workgroups per (request, KV head) of a decode-shaped call: the least estimated time, returned in *estimate.  A
// workgroup of four wavefronts reads up to kDecGroupBytesPerUs until all together reach kDecBytesPerUs,
// and takes kDecStartUs to start and to end.  So some 160 workgroups read as fast as 2000 (1 request of
// 131072 tokens, 8 KV heads: 17 per head 95 us, 22 88, 29 90, 50 95, 67 106; 20 of 9000: 1 per head 117, 3 124, 4 126),
// and every one more is a partial result to merge.  Of those with one block of rows a CU holds two; CUs
// with one less than others cost bandwidth (45 of 7000: 1 per head, 360, 217 us; 2 205; 3 220; 4 210).
constexpr double kDecGroupBytesPerUs = 4.0e4, kDecBytesPerUs = 6.5e6;
constexpr double kDecStartUs = 4.0, kDecMergeUs = 5.0, kDecMergeManyUs = 1.5;
constexpr double kDecResolution = 0.995; // less of a gain than this the estimate cannot tell: fewer workgroups then
// Two blocks of rows.  Together in a wavefront they read the keys once, but a CU holds one such workgroup, its start
// and end take twice as long, and the next round begins when it ends (3 of 20000, 10 new tokens: 8 per
// head, 192, 55 us; 12, 288, 81; 20, 480, 61).  Apart, a CU holds two, and the L2 serves the second if both are on one
// XCD, for which their number has to be a multiple of the XCDs.  Together is better where the memory bounds the call (28 requests of 6494, 15
// new, 32/8 heads 136 us, apart 142; 25 of 9173, 7 new, 64/8 heads 174 and 182), apart where the chain of blocks
// does (32/8 heads: 3 of 48, 14 new 11.2 and 7.5; 48 of 1906, 14 new 94 and 76; 2 of 23880, 12 new 50 and 37).
constexpr double kDec2ApartBytesPerUs = 5.8e4, kDec2ApartStartUs = 4.4, kDec2ApartRoundUs = 2.0, kDec2ApartTwice = 1.6;
constexpr double kDec2BytesPerUs = 3.1e4, kDec2MemoryBytesPerUs = 7.0e6, kDec2StartUs = 4.2, kDec2RoundUs = 4.6, kDec2MergeUs = 2.0;
void choose_decode_groups(const cp_shape *s, int64_t max_n, Plan &pl, double *estimate)
{
    const double units = (double)s->batch * s->num_kv_heads, cus = num_cus();
    const double blocks = (double)((max_n + 31) / 32);
    double best_us = -1.0;
    for (int groups = 1; groups <= pl.nsplit && 4 * (groups - 1) < blocks; ++groups) {
        const double launched = units * groups;
        const double bytes = std::ceil(std::ceil(blocks / groups) / 4.0) * 4.0 * 16384.0; // of one workgroup
        const double traffic = 2.0 * (double)part_bytes((size_t)groups * (size_t)s->total_extend, s->num_q_heads) / kPartBytesPerUs;
        for (int share = 1; share <= pl.row_blocks; ++share) {
            const double workgroups = launched * pl.row_blocks / share, rounds = std::ceil(workgroups / cus);
            const double empty = rounds > 1.0 ? 1.0 - workgroups / (cus * rounds) : 0.0; // of the last round
            double us;
            if (pl.row_blocks == 1) {
                us = kDecStartUs * std::max(1.0, 0.5 * launched / cus) +
                     std::max(bytes / kDecGroupBytesPerUs, launched * bytes / kDecBytesPerUs * (1.0 + 0.3 * empty));
            } else if (share == 1) {
                const double twice = (int64_t)launched % kXcds == 0 ? 1.0 : kDec2ApartTwice;
                us = kDec2ApartStartUs + kDec2ApartRoundUs * std::max(1.0, launched / cus) +
                     std::max(bytes / kDec2ApartBytesPerUs, launched * bytes / kDecBytesPerUs * twice * (1.0 + 0.6 * empty));
            } else {
                us = kDec2StartUs + rounds * (kDec2RoundUs + std::max(bytes / kDec2BytesPerUs, std::min(launched, cus) * bytes / kDec2MemoryBytesPerUs));
            }
            if (groups > 1) us += (pl.row_blocks == 1 ? kDecMergeUs : kDec2MergeUs) + traffic;
            if (groups > kMergeFewSplits) us += kDecMergeManyUs;
            if (best_us < 0.0 || us < kDecResolution * best_us) {
                best_us = us;
                pl.dec_groups = groups;
                pl.dec_share = share;
            }
        }
    }
    *estimate = best_us;
}

// A call of few rows and few keys, none of it enough for the device: the decode kernel with a workgroup per 32
// rows, whose eight wavefronts share the keys and need no merge launch.  One round over the CUs only,
// because every workgroup reads all keys itself.  `us`: the estimate of the way it would go otherwise, then of this one.
// Against row tiles in the best number of key ranges and a merge: P = 512, E = 128, 8/2 heads 15.7 -> 11.0 us;
// P = 1500, E = 256, 32/8 heads 29.8 -> 21.1; 4 requests, P = 1000, E = 64 25.8 -> 15.3; P = 3000, E = 128, 8/2 heads
// would take 27.4 instead of 25.9.  Four wavefronts instead of eight: 11.7 us for the first, 32.3 for the last.
constexpr double kSmallStartUs = 5.0, kSmallBlockUs = 2.0; // a workgroup; a block of 32 keys per wavefront
// Of decode-shaped calls those with two row blocks and at most this many keys: 12 requests, 16 new tokens, 32/8
// heads, P = 3546 34.7 us, 39.6 otherwise; 57, 9 new, 8/2 heads, P = 15646 250, which is more than estimated, and 171.
constexpr int64_t kSmallDecodeKeys = 4096;
bool fits_once(const Requests &q) { return q.row_blocks * q.s->batch * q.s->num_kv_heads <= num_cus(); }
bool small_call(const Requests &q, double &us, Plan &pl)
{
    if (!fits_once(q)) return false;
    const double length = std::ceil((double)((q.max_n + 31) / 32) / 8.0) * kSmallBlockUs;
    if (kSmallStartUs + length >= us) return false;
    us = kSmallStartUs + length;
    pl.small = true;
    pl.dec_groups = 1;
    pl.row_blocks = (int32_t)q.row_blocks;
    return true;
}

// A batch of unequal lengths is split request by request where that promises kMixedUs less than one number of
// key ranges for all, whose kernel finds the owner of an item about 1 us faster; a small one (see above) needs
// neither.  12 requests, P up to 190, E up to 59, 8/2 heads: split request by request 20.8 us, one range each 15.6,
// small 8.9; 12, P up to 14891, E up to 2805, 64/8 heads 91, with one number of ranges 126.  Of 300 random
// batches of 2 to 64 requests 92 were more than 6 % slower than with one number of ranges of at least 8 tiles as long as
// all were split request by request; 10 are.
constexpr double kMixedUs = 2.0;
// The best plan with tiles of whole heads, in one number of key ranges or request by request; nothing runs its row tiles.
// kind_only: whether it is small, or request by request, is all that is asked.
Plan plan_of_whole_heads(Requests &q, size_t room, bool kind_only)
{
    Plan pl, mixed;
    double us, mixed_us;
    choose_splits(q, kWholeHeads, room, pl, &us);
    if (small_call(q, us, pl)) pl.nsplit = 1;
    const double limit = us - kMixedUs;
    if (q.by_request && plan_mixed(q, room, kWholeHeads, mixed, &mixed_us, kind_only ? limit * kNearly : -1.0) && mixed_us + kMixedUs < us)
        return mixed;
    return pl;
}
// `room`: bytes that the caller has for partial results.
// `order`: receives MixedParams::order of a mixed plan.
Plan make_plan(Requests &q, size_t room = SIZE_MAX, uint8_t *order = nullptr)
{
    const cp_shape *const s = q.s;
    Plan pl;
    if (s->num_splits == 0 && q.max_e > 0 && q.max_e * q.G <= kDecRows * kDecMaxRowBlocks) {
        // Decode-shaped.  nsplit bounds the workgroups that may share a request's keys, and is what the
        // queries report: key chunks for 8 wavefronts per CU, at least 2 blocks of 32 keys each, a
        // multiple of the wavefronts of a workgroup.
        pl.row_blocks = (int32_t)q.row_blocks;
        const int64_t pairs = (int64_t)s->batch * s->num_kv_heads * pl.row_blocks;
        int64_t ns = (8LL * num_cus() + pairs - 1) / pairs;
        const int64_t cap = ((q.max_n + 31) / 32 + 1) / 2;
        if (ns > cap) ns = cap;
        ns = (ns + kDecLeastWaves - 1) / kDecLeastWaves * kDecLeastWaves;
        if (ns > kDecMaxChunks) ns = kDecMaxChunks;
        if (ns < kDecLeastWaves) ns = kDecLeastWaves;
        pl.nsplit = (int32_t)ns;
        pl.decode = true;
        double us;
        choose_decode_groups(s, q.max_n, pl, &us);
        if (pl.row_blocks > 1 && q.max_n <= kSmallDecodeKeys) small_call(q, us, pl);
        return pl;
    }
    pl.q_tiles = q.work(kFullTiles).q_tiles;
    pl.max_key_tiles = q.max_key_tiles;
    if (s->num_splits >= 1) {
        pl.nsplit = s->num_splits;
        return pl;
    }
    if (q.max_e == 0) return pl;
    // The estimates for tiles of whole heads decide which rows the decode kernel's form computes, alone or next to row tiles:
    // it scales the scores, the row-tiled kernel rounds the scaled query to 16 bits.  By the estimates for today's tiles,
    // which are lower, 60 of 8022 random equal shapes that are not decode-shaped and 1487 of 10817 unequal ones would go over
    // to row tiles.
    bool beside = false; // decode-shaped requests next to others, in the decode kernel's form
    if (q.decode_rows || fits_once(q)) {
        const Plan heads = plan_of_whole_heads(q, room, true);
        if (heads.small) return heads;
        beside = q.decode_rows && heads.mixed;
    }
    const int64_t items = pl.q_tiles * s->num_kv_heads;
    const bool by_items = q.equal || q.by_request || items < 2 * num_cus();
    const bool few = by_items && items <= num_cus() && q.work(kHalfTiles).q_tiles * s->num_kv_heads <= num_cus(); // so that half tiles fit the CUs at once
    double us = 0.0;
    auto one_number = [&] { // of key ranges for all requests, or small
        if (by_items) q.equal ? choose_equal_splits(q, kFullTiles, room, pl, &us) : choose_splits(q, kFullTiles, room, pl, &us);
        if (few) {
            Plan half;
            double half_us;
            q.equal ? choose_equal_splits(q, kHalfTiles, room, half, &half_us) : choose_splits(q, kHalfTiles, room, half, &half_us);
            if (half_us + kHalfUs < us) {
                pl = half;
                us = half_us + kHalfUs;
            }
        }
        if (small_call(q, us, pl)) {
            pl.nsplit = 1;
            pl.tail_units = 0;
        }
    };
    const bool settled = beside && !fits_once(q); // request by request, whatever the estimates say
    if (!settled) one_number();
    if (!q.by_request) return pl;
    Plan mixed, half;
    double mixed_us, half_us;
    bool any = plan_mixed(q, room, kFullTiles, mixed, &mixed_us);
    if (few && plan_mixed(q, room, kHalfTiles, half, &half_us) && (!any || half_us + kHalfUs < mixed_us)) {
        any = true;
        mixed = half;
        mixed_us = half_us + kHalfUs;
    }
    if (any && ((beside && !pl.small) || mixed_us + kMixedUs < us)) {
        if (order) q.write_order(order);
        return mixed;
    }
    if (settled) one_number();
    return pl;
}

// Whether XCDs that share a KV head take a contiguous range of its items each (see work_item): for equal requests, if
// no range takes more than 6 % longer than the mean.  Then the XCDs stream different keys; dealt out, all the same
// ones.  20 requests, P = 0, E = 1511, 8/2 heads 121 us, dealt out 130; 9, P = 5548, E = 817 170 and 168; but with a
// range 15 % over the mean (3 requests, P = 0, E = 5067, 16/4 heads) 347, dealt out 296.
constexpr double kContiguousExcess = 1.06;
bool contiguous_ranges(const cp_shape *s, const Plan &pl, int64_t items, int xcds)
{
    if (items <= 0 || pl.mixed || pl.tail_units > 0 || !equal_lengths(s)) return false;
    const int G = s->num_q_heads / s->num_kv_heads, E = s->h_extend_lens[0];
    const int64_t nt = row_tiles(E, G, pl.tile_shift), per = (items + xcds - 1) / xcds;
    const double prefix = (double)((s->h_prefix_lens[0] + kBN - 1) / kBN);
    double load = 0.0, most = 0.0, all = 0.0;
    int64_t left = per;
    for (int r = 0; r < s->batch; ++r)
        for (int64_t t = nt - 1; t >= 0; --t) {
            const double tiles = prefix + (double)((std::min<int64_t>(E, (((t + 1) << pl.tile_shift) + G - 1) / G) + kBN - 1) / kBN);
            const double us = kItemUs + kTileUs * tiles / pl.nsplit;
            for (int64_t n = pl.nsplit; n > 0;) {
                const int64_t take = std::min(n, left);
                load += (double)take * us;
                n -= take;
                left -= take;
                if (left > 0) continue;
                most = std::max(most, load);
                all += load;
                load = 0.0;
                left = per;
            }
        }
    return std::max(most, load) * xcds <= kContiguousExcess * (all + load);
}

// Launches the merge of nsplit partial results for n_rh (row, head) pairs.
void launch_merge(const AttnParams &p, int nsplit, hipStream_t hs)
{
    const int64_t n_rh = (int64_t)p.T * p.Hq;
    if (nsplit <= kMergeFewSplits || (nsplit <= kMergeSomeSplits && n_rh >= kMergeSomeRows)) {
        const dim3 grid((unsigned)((n_rh + 7) / 8));
        if (nsplit <= 4)
            hipLaunchKernelGGL(merge_few_splits_kernel<4>, grid, dim3(256), 0, hs, p.part_o, p.part_ml, p.out, n_rh, nsplit);
        else if (nsplit > 16)
            hipLaunchKernelGGL(merge_few_splits_kernel<kMergeSomeSplits>, grid, dim3(256), 0, hs, p.part_o, p.part_ml,
                               p.out, n_rh, nsplit);
        else if (nsplit > kMergeFewSplits)
            hipLaunchKernelGGL(merge_few_splits_kernel<16>, grid, dim3(256), 0, hs, p.part_o, p.part_ml, p.out, n_rh, nsplit);
        else
            hipLaunchKernelGGL(merge_few_splits_kernel<kMergeFewSplits>, grid, dim3(256), 0, hs, p.part_o, p.part_ml,
                               p.out, n_rh, nsplit);
    } else {
        hipLaunchKernelGGL(merge_splits_kernel, dim3((unsigned)n_rh), dim3(32 * kMergeGroups), 0, hs, p.part_o,
                           p.part_ml, p.out, n_rh, nsplit);
    }
}

size_t workspace_for(const cp_shape *s, const Plan &pl)
{
    if (pl.mixed) return pl.part_rows > 0 ? part_bytes((size_t)pl.part_rows, s->num_q_heads) : 0;
    if (pl.nsplit <= 1) return 0;
    if (pl.tail_units > 0) return part_bytes((size_t)pl.tail_units * (size_t)pl.nsplit * kBM, s->num_kv_heads);
    return part_bytes((size_t)pl.nsplit * (size_t)s->total_extend, s->num_q_heads);
}
// plan_of_whole_heads for any call.
Plan old_plan(Requests &q, size_t room = SIZE_MAX)
{
    if (q.s->num_splits >= 1 || q.max_e * q.G <= kDecRows * kDecMaxRowBlocks) return make_plan(q, room); // it has no row tiles, or no choice
    return plan_of_whole_heads(q, room, false);
}
// What the launches touch of it: of a decode-shaped call the partial results of the workgroups that share a
// request's keys, at most nsplit, none where one workgroup has them all.
size_t scratch_used(const cp_shape *s, const Plan &pl)
{
    if (!pl.decode) return workspace_for(s, pl);
    return pl.dec_groups > 1 ? part_bytes((size_t)pl.dec_groups * (size_t)s->total_extend, s->num_q_heads) : 0;
}

// Whether a call with `room` bytes of scratch and the plan pl made for them is refused: the plan needs more, or
// the call is not decode-shaped, brings less than its best plan wants and also less than key ranges of
// at least 8 tiles, for two workgroups per CU, take, or than a split request by request does.  Plans
// without partial results exist for it, but would run several times slower than the call can, without a word.
bool too_little_scratch(Requests &q, const Plan &pl, size_t room)
{
    const cp_shape *const s = q.s;
    if (scratch_used(s, pl) > room) return true;
    if (pl.decode || s->num_splits >= 1) return false;
    // The line lies where it lay when row tiles held whole heads.
    const int64_t items = q.work(kWholeHeads).q_tiles * s->num_kv_heads, want = 2LL * num_cus();
    int64_t ns = items > 0 && items < want ? (want + items - 1) / items : 1;
    ns = std::min<int64_t>({ns, q.max_key_tiles / 8, kMaxSplits});
    if (ns <= 1 || part_bytes((size_t)ns * (size_t)s->total_extend, s->num_q_heads) <= room) return false;
    if (workspace_for(s, old_plan(q)) <= room) return false;
    Plan mixed;
    double us;
    return !q.by_request || !plan_mixed(q, SIZE_MAX, kWholeHeads, mixed, &us) || workspace_for(s, mixed) > room;
}

// The plan of a call with `room` bytes of scratch: the best one if that is enough for it, otherwise the best that fits;
// false if the call is refused.
bool plan_for(Requests &q, size_t room, Plan &pl, uint8_t *order)
{
    pl = make_plan(q, SIZE_MAX, order);
    if (scratch_used(q.s, pl) <= room) return true;
    pl = make_plan(q, room, order);
    return !too_little_scratch(q, pl, room);
}

inline bool aligned_to(const void *p, uintptr_t a) { return reinterpret_cast<uintptr_t>(p) % a == 0; }

// Device address of a file-scope __device__ array on the current device, looked up once per
// device (every device holds its own copy at its own address).
constexpr int kMaxDevices = 64;
struct SymbolCache {
    std::mutex lock;
    void *addr[kMaxDevices] = {};
};
template <typename Lookup>
void *device_address(SymbolCache &cache, Lookup lookup)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> guard(cache.lock);
    if (!cache.addr[dev]) {
        void *ptr = nullptr;
        if (lookup(&ptr) != hipSuccess) return nullptr;
        cache.addr[dev] = ptr;
    }
    return cache.addr[dev];
}
void *check_report_address()
{
    static SymbolCache cache;
    return device_address(cache, [](void **ptr) { return hipGetSymbolAddress(ptr, HIP_SYMBOL(g_check_report)); });
}

std::atomic<int> g_debug_validate{
#ifdef CP_DEBUG_VALIDATE
    1
#else
    -1 // not decided yet: the environment variable CP_DEBUG_VALIDATE is read on first use
#endif
};
bool debug_validate_on()
{
    int v = g_debug_validate.load(std::memory_order_relaxed);
    if (v < 0) {
        const char *e = getenv("CP_DEBUG_VALIDATE");
        v = (e && e[0] && e[0] != '0') ? 1 : 0;
        g_debug_validate.store(v, std::memory_order_relaxed);
    }
    return v == 1;
}

// The check itself: lengths are compared on the host after one copy, table entries on the
// device.  Waits for `stream` (this is the one place where the library synchronises).
int check_tables(const int32_t *block_table, const int32_t *prefix_lens, const int32_t *extend_lens,
                 hipStream_t hs, const cp_shape *s, int32_t *info)
{
    if (info) info[0] = info[1] = info[2] = -1;
    const int B = s->batch;
    std::vector<int32_t> dev_p((size_t)B), dev_e((size_t)B);
    if (hipMemcpyAsync(dev_p.data(), prefix_lens, (size_t)B * 4, hipMemcpyDeviceToHost, hs) != hipSuccess ||
        hipMemcpyAsync(dev_e.data(), extend_lens, (size_t)B * 4, hipMemcpyDeviceToHost, hs) != hipSuccess ||
        hipStreamSynchronize(hs) != hipSuccess)
        return CP_ERR_LAUNCH;
    for (int r = 0; r < B; ++r)
        if (dev_p[r] != s->h_prefix_lens[r] || dev_e[r] != s->h_extend_lens[r]) {
            if (info) {
                info[0] = r;
                info[1] = dev_p[r];
                info[2] = dev_e[r];
            }
            return CP_ERR_LENGTHS;
        }
    auto *report = static_cast<unsigned long long *>(check_report_address());
    if (!report) return CP_ERR_LAUNCH;
    const unsigned long long clear = ~0ull;
    if (hipMemcpyAsync(report, &clear, sizeof(clear), hipMemcpyHostToDevice, hs) != hipSuccess) return CP_ERR_LAUNCH;
    const int blocks_x = std::max(1, std::min(64, (s->max_pages_per_req + kCheckThreads - 1) / kCheckThreads));
    for (int r0 = 0; r0 < B; r0 += 65535) { // grid.y limit
        const int nb = std::min(65535, B - r0);
        hipLaunchKernelGGL(check_tables_kernel, dim3((unsigned)blocks_x, (unsigned)nb), dim3(kCheckThreads), 0, hs,
                           block_table + (int64_t)r0 * s->max_pages_per_req, prefix_lens + r0, extend_lens + r0, nb,
                           s->max_pages_per_req, s->num_pages, report);
        if (hipGetLastError() != hipSuccess) return CP_ERR_LAUNCH;
        unsigned long long got = 0;
        if (hipMemcpyAsync(&got, report, sizeof(got), hipMemcpyDeviceToHost, hs) != hipSuccess ||
            hipStreamSynchronize(hs) != hipSuccess)
            return CP_ERR_LAUNCH;
        if (got != ~0ull) {
            const bool bad_page = (got >> 62) != 0;
            const int r = r0 + (int)((got >> 31) & 0x7fffffffu), slot = (int)(got & 0x7fffffffu);
            int32_t entry = -1;
            if (bad_page && (hipMemcpyAsync(&entry, block_table + (int64_t)r * s->max_pages_per_req + slot, 4,
                                            hipMemcpyDeviceToHost, hs) != hipSuccess ||
                             hipStreamSynchronize(hs) != hipSuccess))
                return CP_ERR_LAUNCH;
            if (info) {
                info[0] = r;
                info[1] = bad_page ? slot : dev_p[r];
                info[2] = bad_page ? entry : dev_e[r];
            }
            return bad_page ? CP_ERR_TABLE : CP_ERR_LENGTHS;
        }
    }
    return CP_OK;
}

} // namespace

// Split-K / decode partial results of cp_extend_attention_noalloc: one array per device, held
// until the process ends.  Nothing in it has to start at zero (every partial that the merge
// reads is written by the launch before it), so it is never cleared; calls that overlap on one
// device share it and race.
#define CP_NOALLOC_SCRATCH_BYTES (64u << 20)
static __device__ __align__(256) unsigned char scratch[CP_NOALLOC_SCRATCH_BYTES];

namespace {
void *scratch_address()
{
    static SymbolCache cache;
    return device_address(cache, [](void **ptr) { return hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch)); });
}
} // namespace

extern "C" {

const char *cp_status_string(int status)
{
    switch (status) {
    case CP_OK: return "ok";
    case CP_ERR_NULL: return "a required pointer is NULL";
    case CP_ERR_SHAPE: return "unsupported or inconsistent shape";
    case CP_ERR_WORKSPACE:
        return "workspace missing, too small or misaligned (cp_extend_attention_noalloc: the shape needs more "
               "than the library's own scratch)";
    case CP_ERR_LAUNCH: return "HIP launch error";
    case CP_ERR_ALIGN: return "a device pointer is not aligned as required";
    case CP_ERR_TABLE: return "block_table holds a page id outside [0, num_pages)";
    case CP_ERR_LENGTHS: return "device prefix_lens / extend_lens differ from the host copies";
    default: return "unknown status";
    }
}

int32_t cp_num_splits(const cp_shape *shape)
{
    if (validate(shape) != CP_OK) return 0;
    Requests q(shape);
    return make_plan(q).nsplit;
}

int32_t cp_plan_kind(const cp_shape *shape)
{
    if (validate(shape) != CP_OK) return CP_PLAN_INVALID;
    Requests q(shape);
    const Plan pl = make_plan(q);
    if (pl.decode || pl.small) return CP_PLAN_DECODE;
    return pl.nsplit > 1 ? CP_PLAN_ROW_TILED_SPLIT : CP_PLAN_ROW_TILED;
}

int32_t cp_plan_tile_rows(const cp_shape *shape)
{
    if (validate(shape) != CP_OK || shape->total_extend == 0) return 0;
    Requests q(shape);
    const Plan pl = make_plan(q);
    return pl.decode || pl.small ? 0 : 1 << pl.tile_shift;
}

size_t cp_workspace_bytes(const cp_shape *shape)
{
    if (validate(shape) != CP_OK) return 0;
    Requests q(shape);
    return workspace_for(shape, make_plan(q));
}

} // extern "C"

namespace {
// Everything behind cp_extend_attention: argument checks, plan, launches.  `workspace` is
// whatever scratch the entry point brings: the caller's buffer or the library's own array.  `lengths` are those of
// the shape, which the entry point has validated.  `planned`: the plan for the scratch where the entry point has made and
// checked one, with its order in p.
int run_attention(const void *q, const void *k_new, const void *v_new, const void *kv_pages,
                  const int32_t *block_table, const int32_t *prefix_lens, const int32_t *extend_lens, void *out,
                  void *stream, Requests &lengths, void *workspace, size_t workspace_bytes, MixedParams &p,
                  const Plan *planned)
{
    const cp_shape *const shape = lengths.s;
    if (!block_table || !prefix_lens || !extend_lens) return CP_ERR_NULL;
    if (shape->total_extend == 0) return CP_OK;
    if (!q || !k_new || !v_new || !kv_pages || !out) return CP_ERR_NULL;
    if (!aligned_to(q, 16) || !aligned_to(k_new, 16) || !aligned_to(v_new, 16) || !aligned_to(kv_pages, 16) ||
        !aligned_to(out, 16) || !aligned_to(block_table, 4) || !aligned_to(prefix_lens, 4) ||
        !aligned_to(extend_lens, 4))
        return CP_ERR_ALIGN;
    if (debug_validate_on()) {
        const int chk = check_tables(block_table, prefix_lens, extend_lens, static_cast<hipStream_t>(stream), shape,
                                     nullptr);
        if (chk != CP_OK) return chk;
    }
    const size_t room = workspace ? workspace_bytes : 0;
    Plan pl;
    if (planned) pl = *planned;
    else if (!plan_for(lengths, room, pl, p.order)) return CP_ERR_WORKSPACE;
    if (workspace && !aligned_to(workspace, 256)) {
        // The caller's mistake where row tiles of whole heads asked for scratch, which is where this has been one.  Calls that
        // ask for some only with today's tiles run with such a buffer as without one.
        const Plan heads = old_plan(lengths, room);
        if (scratch_used(shape, heads) > 0) return CP_ERR_WORKSPACE;
        if (scratch_used(shape, pl) > 0) pl = make_plan(lengths, 0, p.order);
    }
    const size_t need = scratch_used(shape, pl);
    const int64_t per_head = pl.mixed ? pl.row_items + (pl.dec_units + kWaves - 1) / kWaves :
                             pl.tail_units > 0 ? pl.q_tiles + pl.tail_units * (int64_t)(pl.nsplit - 1) : pl.q_tiles * pl.nsplit;
    const int64_t total = per_head * shape->num_kv_heads;
    if (total > INT32_MAX / 2) return CP_ERR_SHAPE;
    const int64_t dec_units = (int64_t)shape->batch * shape->num_kv_heads * pl.nsplit * pl.row_blocks;
    if (pl.decode && dec_units > INT32_MAX / 2) return CP_ERR_SHAPE;

    p.q = static_cast<const uint16_t *>(q);
    p.k_new = static_cast<const uint16_t *>(k_new);
    p.v_new = static_cast<const uint16_t *>(v_new);
    p.kv_pages = static_cast<const uint16_t *>(kv_pages);
    p.block_table = block_table;
    p.prefix_lens = prefix_lens;
    p.extend_lens = extend_lens;
    p.out = static_cast<uint16_t *>(out);
    p.part_o = nullptr;
    p.part_ml = nullptr;
    p.batch = shape->batch;
    p.Hq = shape->num_q_heads;
    p.Hkv = shape->num_kv_heads;
    p.G = shape->num_q_heads / shape->num_kv_heads;
    p.max_pages = shape->max_pages_per_req;
    p.T = shape->total_extend;
    p.nsplit = pl.nsplit;
    p.tail_units = pl.tail_units;
    p.tile_shift = pl.tile_shift;
    p.whole_units = pl.tail_units > 0 ? (int32_t)pl.q_tiles - pl.tail_units : 0;
    p.dec_row_blocks = pl.row_blocks;
    p.items_per_head = (int32_t)per_head;
    p.total_items = (int32_t)total;
    p.xcds_per_head = p.Hkv < kXcds && kXcds % p.Hkv == 0 ? kXcds / p.Hkv : 1;
    const bool ranges = p.xcds_per_head > 1 && contiguous_ranges(shape, pl, per_head, p.xcds_per_head);
    if (ranges) p.xcds_per_head = 1;
    p.alternate = !ranges && per_head * p.Hkv <= kAlternateRounds * (int64_t)num_cus() && lengths.equal;
    p.items_per_xcd = (int32_t)(p.xcds_per_head > 1 ? (per_head + p.xcds_per_head - 1) / p.xcds_per_head
                                                    : (total + kXcds - 1) / kXcds);
    p.scale_log2 = shape->softmax_scale * 1.4426950408889634f;

    p.g_magic = (lengths.max_e * p.G + kBM + 1) * p.G <= INT64_C(0x100000000) ? 0xffffffffu / (uint32_t)p.G : 0u;

    p.seg_tiles = pl.seg_tiles;
    p.dec_blocks = pl.dec_blocks;
    if (pl.mixed) p.dec_share = (((uint64_t)(per_head - pl.row_items) << 32) + (uint64_t)per_head - 1) / (uint64_t)per_head;

    hipStream_t hs = static_cast<hipStream_t>(stream);
    if (need > 0) {
        const size_t parts = pl.mixed ? (size_t)pl.part_rows : (size_t)(pl.decode ? pl.dec_groups : pl.nsplit) * (size_t)p.T;
        const size_t rows = pl.tail_units > 0 ? (size_t)pl.tail_units * (size_t)pl.nsplit * kBM * (size_t)p.Hkv : parts * (size_t)p.Hq;
        p.part_o = static_cast<float *>(workspace);
        p.part_ml = reinterpret_cast<float *>(static_cast<char *>(workspace) + ((rows * kD * sizeof(float) + 255) / 256) * 256);
    }
    if (pl.decode || pl.small) {
        p.nsplit = pl.dec_groups;
        const int share = pl.small ? 1 : pl.dec_share;
        const dim3 groups((unsigned)((int64_t)p.batch * p.Hkv * pl.dec_groups * ((pl.row_blocks + share - 1) / share)));
        const AttnParams &a = p;
        if (pl.small) hipLaunchKernelGGL((decode_attn_kernel<8, 1>), groups, dim3(512), 0, hs, a);
        else if (share == 1) hipLaunchKernelGGL((decode_attn_kernel<4, 1>), groups, dim3(256), 0, hs, a);
        else hipLaunchKernelGGL((decode_attn_kernel<4, 2>), groups, dim3(256), 0, hs, a);
        if (hipGetLastError() != hipSuccess) return CP_ERR_LAUNCH;
        if (pl.dec_groups > 1) launch_merge(p, pl.dec_groups, hs);
        return hipGetLastError() == hipSuccess ? CP_OK : CP_ERR_LAUNCH;
    }
    if (!allow_large_lds()) return CP_ERR_LAUNCH;
    const dim3 grid((unsigned)(p.items_per_xcd * kXcds)), block(kThreads);
    if (pl.mixed) {
        hipLaunchKernelGGL(extend_attn_kernel<kMixed>, grid, block, kMixedLdsBytes, hs, p);
        if (pl.merge_rows > 0) {
            if (hipGetLastError() != hipSuccess) return CP_ERR_LAUNCH;
            const int64_t blocks = pl.merge_rows * ((p.Hq + kMergeHeads - 1) / kMergeHeads);
            hipLaunchKernelGGL(merge_mixed_kernel, dim3((unsigned)blocks), dim3(32 * kMergeHeads), 0, hs, p);
        }
    } else if (pl.nsplit > 1) {
        hipLaunchKernelGGL(extend_attn_kernel<kSplit>, grid, block, kLdsBytes, hs, static_cast<const AttnParams &>(p));
        if (hipGetLastError() != hipSuccess) return CP_ERR_LAUNCH;
        if (pl.tail_units == 0) launch_merge(p, pl.nsplit, hs);
        else {
            const dim3 blocks((unsigned)(pl.tail_units * p.Hkv * (kBM / 8)));
            const AttnParams &a = p;
            if (pl.nsplit <= 4) hipLaunchKernelGGL(merge_tail_kernel<4>, blocks, dim3(256), 0, hs, a);
            else if (pl.nsplit <= 8) hipLaunchKernelGGL(merge_tail_kernel<8>, blocks, dim3(256), 0, hs, a);
            else hipLaunchKernelGGL(merge_tail_kernel<kMaxTailSplits>, blocks, dim3(256), 0, hs, a);
        }
    } else {
        hipLaunchKernelGGL(extend_attn_kernel<kWhole>, grid, block, kLdsBytes, hs, static_cast<const AttnParams &>(p));
    }
    if (hipGetLastError() != hipSuccess) return CP_ERR_LAUNCH;
    return CP_OK;
}
} // namespace

extern "C" {

int cp_extend_attention(const void *q, const void *k_new, const void *v_new, const void *kv_pages,
                        const int32_t *block_table, const int32_t *prefix_lens,
                        const int32_t *extend_lens, void *out, void *stream, const cp_shape *shape,
                        void *workspace, size_t workspace_bytes)
{
    const int st = validate(shape);
    if (st != CP_OK) return st;
    MixedParams p;
    Requests lengths(shape);
    return run_attention(q, k_new, v_new, kv_pages, block_table, prefix_lens, extend_lens, out, stream, lengths,
                         workspace, workspace_bytes, p, nullptr);
}

size_t cp_noalloc_scratch_bytes(void) { return CP_NOALLOC_SCRATCH_BYTES; }

int cp_extend_attention_noalloc(const void *q, const void *k_new, const void *v_new, const void *kv_pages,
                                const int32_t *block_table, const int32_t *prefix_lens,
                                const int32_t *extend_lens, void *out, void *stream, const cp_shape *shape)
{
    const int st = validate(shape);
    if (st != CP_OK) return st;
    // sizes beyond the library's own array are refused here, before anything is looked up or launched
    MixedParams p;
    Requests lengths(shape);
    Plan pl;
    if (!plan_for(lengths, CP_NOALLOC_SCRATCH_BYTES, pl, p.order)) return CP_ERR_WORKSPACE;
    void *ptr = scratch_address(); // the array's address on the current device, never the array's name
    if (!ptr) return CP_ERR_LAUNCH;
    return run_attention(q, k_new, v_new, kv_pages, block_table, prefix_lens, extend_lens, out, stream, lengths, ptr,
                         CP_NOALLOC_SCRATCH_BYTES, p, &pl);
}

int cp_write_kv(const void *k_new, const void *v_new, void *kv_pages, const int32_t *block_table,
                const int32_t *prefix_lens, const int32_t *extend_lens, void *stream,
                const cp_shape *shape)
{
    const int st = validate(shape);
    if (st != CP_OK) return st;
    if (!block_table || !prefix_lens || !extend_lens) return CP_ERR_NULL;
    if (shape->total_extend == 0) return CP_OK;
    if (!k_new || !v_new || !kv_pages) return CP_ERR_NULL;
    if (!aligned_to(k_new, 16) || !aligned_to(v_new, 16) || !aligned_to(kv_pages, 16) ||
        !aligned_to(block_table, 4) || !aligned_to(prefix_lens, 4) || !aligned_to(extend_lens, 4))
        return CP_ERR_ALIGN;
    if (debug_validate_on()) {
        const int chk = check_tables(block_table, prefix_lens, extend_lens, static_cast<hipStream_t>(stream), shape,
                                     nullptr);
        if (chk != CP_OK) return chk;
    }
    const int T = shape->total_extend;
    const int64_t blocks = (int64_t)((T + kWriteRows - 1) / kWriteRows) * ((shape->num_kv_heads + kWriteHeads - 1) / kWriteHeads);
    if (blocks > INT32_MAX) return CP_ERR_SHAPE;
    hipLaunchKernelGGL(write_kv_kernel, dim3((unsigned)blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const uint16_t *>(k_new), static_cast<const uint16_t *>(v_new),
                       static_cast<uint16_t *>(kv_pages), block_table, prefix_lens, extend_lens,
                       shape->batch, shape->num_kv_heads, shape->max_pages_per_req, T);
    if (hipGetLastError() != hipSuccess) return CP_ERR_LAUNCH;
    return CP_OK;
}

int cp_check_tables(const int32_t *block_table, const int32_t *prefix_lens, const int32_t *extend_lens,
                    void *stream, const cp_shape *shape, int32_t *info)
{
    const int st = validate(shape);
    if (st != CP_OK) return st;
    if (!block_table || !prefix_lens || !extend_lens) return CP_ERR_NULL;
    if (!aligned_to(block_table, 4) || !aligned_to(prefix_lens, 4) || !aligned_to(extend_lens, 4)) return CP_ERR_ALIGN;
    return check_tables(block_table, prefix_lens, extend_lens, static_cast<hipStream_t>(stream), shape, info);
}

void cp_set_debug_validate(int on) { g_debug_validate.store(on ? 1 : 0, std::memory_order_relaxed); }

} // extern "C"
