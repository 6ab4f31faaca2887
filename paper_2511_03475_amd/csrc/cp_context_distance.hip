// Pairwise context distance (paper, Section 4.1, Eq. 1) for gfx950.
//
// A tile is kRows row contexts against 256 column contexts, one column per thread.  The tile's row
// ids go into a dictionary in LDS: id -> one byte per row, 0 where the row lacks the id, else
// 0x80 | its position in the row.  A column then looks up each of its ids ONCE for all rows of the
// tile, turns the bytes of four of its positions around so that a word holds one row's four bytes,
// and two byte-wise sums of absolute differences per word add up what Eq. 1 needs of the row: the
// masked one the position gaps, the other 128 x (ids shared) + (positions).  A pair of positions
// thus costs about one vector instruction where comparing the ids costs two, and a pair of
// contexts of 16 ids some 45 in place of 512.
//
// What bounds it: the stores of the matrix, next vector instructions.  The matrix is symmetric, so
// only tiles on and above the diagonal blocks of 256 are computed, and a tile is written twice: by
// its rows from the registers, and by its columns after a turn through LDS.  Measured for 8192
// contexts of 15 ids, stride 16: 60 us (4.5 TB/s of stores; 40 us without them, a plain fill takes
// 39), against 1130 us for comparing every pair of positions; 200 to 1000 contexts 9-10 us, a
// launch, against 197; 16384 contexts 249 us against 4240; stride 32, 8192 contexts 110 against 4040.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cp_context_distance.h"

namespace {

constexpr int kThreads = 256;   // columns per tile
constexpr int kEntries = 512;   // (row, position) entries of a tile's dictionary
// Dictionary slots: buckets of four words, one 16-byte read.  The hash is a multiplication by an odd
// number, which loses nothing: its top 10 bits choose the bucket, the other 22 tell the ids of a
// bucket apart, and the 10 bits that the shift leaves free hold the entry of the id.
constexpr int kBuckets = 1024;
constexpr uint32_t kHash = 0x9E3779B1u;
constexpr uint32_t kEmpty = 0xFFFFFFFFu;   // its entry bits lie above kEntries: never taken for a hit
constexpr uint32_t kEntryMask = 1023u;

template <int kMax>
__global__ __launch_bounds__(kThreads, 4) void context_distance_kernel(const int32_t *__restrict__ contexts,
                                                                   const int32_t *__restrict__ lens,
                                                                   int n, int stride, float alpha,
                                                                   float *__restrict__ dist, int wide_rows)
{
    constexpr int kRows = kEntries / kMax;   // 32 rows of up to 16 ids, 16 of up to 32
    constexpr int kWords = kRows / 4;        // of an entry's bytes
    // the dictionary; once every column has looked its ids up, the place where the tile is transposed
    __shared__ uint4 s_mem[kBuckets + (kEntries + 1) * kWords / 4];
    uint4 *const s_slot = s_mem, *const s_bytes = s_mem + kBuckets; // the last entry stays zero: id absent
    static_assert(sizeof(float) * kRows * kThreads <= sizeof(s_mem), "a tile fits where the dictionary was");
    __shared__ uint32_t s_over_hash[kEntries];               // ids whose bucket was full
    __shared__ uint32_t s_over_entry[kEntries];
    // length of a row and its reciprocal (infinite for 0), as bits: neither is negative, so they
    // compare like whole numbers, which spares the canonicalising of fmaxf / fminf
    __shared__ uint2 s_len[kRows];
    __shared__ uint32_t s_over;

    const int tid = threadIdx.x;
    const int i0 = blockIdx.y * kRows;
    // Workgroups go round the XCDs by their number, so without a shift from tile to tile one XCD
    // would get the columns at the left, which few tiles need, and another those at the right.
    const int g = (blockIdx.x + blockIdx.y) % gridDim.x; // group of kThreads columns
    const int diag = i0 / kThreads;                      // the group that these rows are in
    if (g < diag) return;

    // ---- dictionary of the rows i0 .. i0 + kRows - 1
    for (int s = tid; s < kBuckets; s += kThreads) s_slot[s] = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
    for (int s = tid; s < (kEntries + 1) * kWords / 4; s += kThreads) s_bytes[s] = make_uint4(0, 0, 0, 0);
    if (tid < kRows) {
        const float l = i0 + tid < n ? (float)lens[i0 + tid] : 0.f;
        s_len[tid] = make_uint2(__float_as_uint(l), __float_as_uint(l > 0.f ? 1.f / l : __builtin_inff()));
    }
    if (tid == 0) s_over = 0;
    __syncthreads();
#pragma unroll
    for (int e = tid; e < kEntries; e += kThreads) {
        const int row = e / kMax, pos = e % kMax, i = i0 + row;
        if (i >= n || pos >= stride || pos >= lens[i]) continue;
        const uint32_t h = (uint32_t)contexts[(int64_t)i * stride + pos] * kHash;
        uint32_t *slot = reinterpret_cast<uint32_t *>(&s_slot[h >> 22]);
        const uint32_t rest = h << 10;
        uint32_t entry = kEntries;
        for (int k = 0; k < 4 && entry == kEntries; ++k) {
            const uint32_t old = atomicCAS(slot + k, kEmpty, rest | (uint32_t)e);
            if (old == kEmpty) entry = e;
            else if ((old ^ rest) < (uint32_t)kEntries) entry = old ^ rest;
        }
        if (entry == kEntries) { // bucket full: the entry stands for this row alone
            const uint32_t at = atomicAdd(&s_over, 1u);
            s_over_hash[at] = h;
            s_over_entry[at] = e;
            entry = e;
        }
        reinterpret_cast<uint8_t *>(s_bytes)[entry * kRows + row] = (uint8_t)(0x80 | pos);
    }
    __syncthreads();
    const int over = __builtin_amdgcn_readfirstlane(s_over);

    const int j = g * kThreads + tid;
    const bool col_ok = j < n;
    const int jc = col_ok ? j : n - 1;
    const int len_j = lens[jc];
    // low half: sum of the position gaps; high half (kMax 16): 128 x shared + sum of positions,
    // which stays below 128 because the positions of a row are distinct: 0 + 1 + .. + 15 = 120
    uint32_t acc[kRows], cnt[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) acc[r] = cnt[r] = 0;
#pragma unroll
    for (int q = 0; q < kMax / 4; ++q) {
        if (4 * q >= stride) break;      // uniform
        const int4 ids = *reinterpret_cast<const int4 *>(contexts + (int64_t)jc * stride + 4 * q);
        const int id[4] = {ids.x, ids.y, ids.z, ids.w};
        uint32_t w[4][kWords];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t h = (uint32_t)id[b] * kHash;
            const uint4 s = s_slot[h >> 22];
            const uint32_t rest = h << 10;
            uint32_t entry = min(min(s.x ^ rest, s.y ^ rest), min(s.z ^ rest, s.w ^ rest));
            entry = 4 * q + b < len_j ? min(entry, (uint32_t)kEntries) : (uint32_t)kEntries;
#pragma unroll
            for (int k = 0; k < kWords / 4; ++k) {
                const uint4 v = s_bytes[entry * (kWords / 4) + k];
                w[b][4 * k] = v.x;
                w[b][4 * k + 1] = v.y;
                w[b][4 * k + 2] = v.z;
                w[b][4 * k + 3] = v.w;
            }
        }
        const uint32_t here = 0x80808080u | (0x03020100u + 0x04040404u * q); // these four positions
#pragma unroll
        for (int k = 0; k < kWords; ++k) {
            // four rows: their bytes of the four positions side by side
            const uint32_t lo01 = __builtin_amdgcn_perm(w[1][k], w[0][k], 0x05010400);
            const uint32_t hi01 = __builtin_amdgcn_perm(w[1][k], w[0][k], 0x07030602);
            const uint32_t lo23 = __builtin_amdgcn_perm(w[3][k], w[2][k], 0x05010400);
            const uint32_t hi23 = __builtin_amdgcn_perm(w[3][k], w[2][k], 0x07030602);
            const uint32_t row[4] = {__builtin_amdgcn_perm(lo23, lo01, 0x05040100), __builtin_amdgcn_perm(lo23, lo01, 0x07060302),
                                     __builtin_amdgcn_perm(hi23, hi01, 0x05040100), __builtin_amdgcn_perm(hi23, hi01, 0x07060302)};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                acc[4 * k + r] = __builtin_amdgcn_msad_u8(here, row[r], acc[4 * k + r]);
                if constexpr (kMax <= 16) acc[4 * k + r] = __builtin_amdgcn_sad_hi_u8(row[r], 0, acc[4 * k + r]);
                else cnt[4 * k + r] += __builtin_popcount(row[r] & 0x80808080u);
            }
        }
    }

    // rare: ids whose bucket was full, one row and position each
    for (int t = 0; t < over; ++t) {
        const uint32_t h = s_over_hash[t], entry = s_over_entry[t], pos = entry % kMax;
        uint32_t gap = 0, hit = 0;
        for (int b = 0; b < min(len_j, stride); ++b) // the length comes from the device, unchecked
            if ((uint32_t)contexts[(int64_t)jc * stride + b] * kHash == h) {
                gap = (uint32_t)abs(b - (int)pos);
                hit = 1;
            }
#pragma unroll
        for (int r = 0; r < kRows; ++r)
            if ((uint32_t)r == entry / kMax) {
                acc[r] += kMax <= 16 ? gap + ((hit * (0x80 + pos)) << 16) : gap;
                cnt[r] += hit;
            }
    }

    const uint32_t fl_j = __float_as_uint((float)len_j);
    const uint32_t inv_j = __float_as_uint(len_j > 0 ? 1.f / (float)len_j : __builtin_inff());
    float d[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const uint2 row = s_len[r];
        const float gap = (float)(kMax <= 16 ? acc[r] & 0xffu : acc[r]);
        const float shared = (float)(kMax <= 16 ? acc[r] >> 23 : cnt[r]);
        // shared / longest and gap / shared, correctly rounded: a product with the reciprocal and one
        // correction (holds for every shared <= 32 and gap < 1024, also if v_rcp_f32 is an ulp off)
        const float longest = __uint_as_float(max(row.x, fl_j)), inv_longest = __uint_as_float(min(row.y, inv_j));
        float part = shared * inv_longest;
        part = fmaf(fmaf(-part, longest, shared), inv_longest, part);
        const float inv_shared = __builtin_amdgcn_rcpf(shared);
        float mean = gap * inv_shared;
        mean = fmaf(fmaf(-mean, shared, gap), inv_shared, mean);
        d[r] = shared > 0.f ? fmaf(alpha, mean, 1.f - part) : (longest > 0.f ? 1.f : 0.f);
    }
    if (col_ok) {
        float *row = dist + (int64_t)i0 * n + (int64_t)g * kThreads; // uniform
        if (i0 + kRows <= n) {
#pragma unroll
            for (int r = 0; r < kRows; ++r, row += n) row[tid] = d[r];
        } else {
#pragma unroll
            for (int r = 0; r < kRows; ++r)
                if (i0 + r < n) row[(int64_t)r * n + tid] = d[r];
        }
    }
    if (g == diag) return; // uniform: both halves of a diagonal block are computed

    // The same values as pieces of rows g * kThreads ..: a column holds 128 bytes of its row, and
    // written from the registers each 16 of them would be a request of its own to the L2 (measured:
    // 84 us for n = 8192, against 58 without these rows at all).  So every wavefront
    // turns its 64 columns around in LDS: chunk k of column c lies at k ^ (c % kChunks).
    constexpr int kChunks = kRows / 4;
    __syncthreads();
    float4 *const mine = reinterpret_cast<float4 *>(s_mem) + (tid & ~63) * kChunks;
    const int lane = tid & 63;
#pragma unroll
    for (int k = 0; k < kChunks; ++k)
        mine[lane * kChunks + (k ^ (lane % kChunks))] = make_float4(d[4 * k], d[4 * k + 1], d[4 * k + 2], d[4 * k + 3]);
    const int j0 = g * kThreads + (tid & ~63);
    if (wide_rows && i0 + kRows <= n) {
#pragma unroll
        for (int s = 0; s < kChunks; ++s) {
            const int c = s * (64 / kChunks) + lane / kChunks, k = lane % kChunks;
            const float4 v = mine[c * kChunks + (k ^ (c % kChunks))];
            if (j0 + c < n) *reinterpret_cast<float4 *>(dist + (int64_t)(j0 + c) * n + i0 + 4 * k) = v;
        }
    } else {
        const float *const words = reinterpret_cast<const float *>(mine);
        for (int s = 0; s < kRows; ++s) {
            const int c = s * (64 / kRows) + lane / kRows, r = lane % kRows;
            const float v = words[c * kRows + 4 * ((r / 4) ^ (c % kChunks)) + r % 4];
            if (j0 + c < n && i0 + r < n) dist[(int64_t)(j0 + c) * n + i0 + r] = v;
        }
    }
}

template <int kMax>
void launch(const int32_t *contexts, const int32_t *lens, int n, int stride, float alpha, float *dist, hipStream_t hs)
{
    constexpr int kRows = kEntries / kMax;
    const int tiles = (n + kRows - 1) / kRows, groups = (n + kThreads - 1) / kThreads;
    // pieces of mirrored rows can be written 16 bytes at a time
    const int wide_rows = n % 4 == 0 && reinterpret_cast<uintptr_t>(dist) % 16 == 0;
    hipLaunchKernelGGL(context_distance_kernel<kMax>, dim3((unsigned)groups, (unsigned)tiles), dim3(kThreads), 0, hs,
                       contexts, lens, n, stride, alpha, dist, wide_rows);
}

} // namespace

extern "C" int cp_context_distance(const int32_t *contexts, const int32_t *lens, int32_t n,
                                   int32_t stride, float alpha, float *dist, void *stream)
{
    if (n < 0 || n > 65536 || stride < 1 || stride > 32 || stride % 4 != 0) return -2;
    if (!(alpha >= 0.f) || !(alpha < 3.0e38f)) return -2;
    if (n == 0) return 0;
    if (!contexts || !lens || !dist) return -1;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    if (stride <= 16) launch<16>(contexts, lens, n, stride, alpha, dist, hs);
    else launch<32>(contexts, lens, n, stride, alpha, dist, hs);
    return hipGetLastError() == hipSuccess ? 0 : -4;
}
