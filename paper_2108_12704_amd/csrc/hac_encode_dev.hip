// GPU-side encoder: builds a HAC or sHAC blob (arXiv 2108.12704 Sect. IV-B / IV-C) from a matrix
// that already lives in device memory, byte for byte the blob hac_encode / shac_encode would build
// on the host.
//
// The steps of the host encoder, split between device and host:
//   1. device  the one pass over W: per 32 rows of a column a word with a bit per non-zero, the
//              non-zeros themselves packed column by column (where they are few), and a histogram
//              of the distinct fp32 values (a hash table keyed by bit pattern, privatised in LDS
//              per block); the occupied slots of the table are gathered into a list;
//   2. host    alphabet in value order, Huffman lengths, canonical code, decode tables, and a
//              small hash table from a value's bit pattern to its codeword;
//   3. device  non-zeros and stream bits of every (row segment, column) from the words and the
//              packed values; with Rice-coded row gaps also the gap bits for every parameter
//              k = 0..15; then, per column, running sums over its segments and their totals;
//   4. host    chunk size, prefix sums over the columns (first stream bit, CSC position, first
//              chunk of every column), section offsets, header;
//   5. device  one thread per (row segment, column) writes the codewords (and row-index fields or
//              gap codewords) of its non-zeros, and the chunk entries.
// W is far larger than everything else, so it is read once.  A word costs 1/32 of what it stands for
// and a packed list is as long as the non-zeros, so steps 3 and 5 move a few per cent of W's bytes
// on a pruned layer; where more than an eighth of a 32 x 64 tile is non-zero its values are not
// packed but fetched from W again, by then mostly whole cache lines.
// 25088 x 4096, 2 % non-zero: the three passes over W that this replaces took 0.25 + 0.36 + 0.40 ms.
// What crosses the bus is of the size of the alphabet and of the number of columns, never of the
// matrix.  The call synchronises the stream twice before its final wait (steps 2 and 4 need the
// device's results).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "hac_hostlib.h"

namespace {

using namespace hac_internal;

constexpr uint32_t kHashSlots = 1u << 17;          // distinct values <= 65536 keep the load below 1/2
constexpr uint32_t kSegRowsMax = 256, kSegRowsMin = 32;   // multiples of 32: a segment is whole words
constexpr uint32_t kSegWordsMax = kSegRowsMax / 32;
constexpr uint64_t kMaxRows = 65535ull * 1024;
constexpr uint32_t kTileCols = 64, kTileRows = 32;        // what a wavefront reads at a time in step 1
constexpr uint32_t kQuota = 4;                            // packed values per column of a tile: an eighth of it
constexpr uint32_t kNotPacked = 0xffffu;
constexpr uint32_t kScanWaves = 8, kScanQueue = 1024, kScanBlocks = 1024;   // 40 KB of LDS a block: four on a CU
constexpr uint32_t kCodeSlotsLds = 2048;                  // code tables up to this size (24 KB) are copied to LDS

// Rows per segment: 256 on a large matrix, fewer on a small one, so that there are about 512 K
// (segment, column) threads (a thread's work is a chain of short trips to memory).
__host__ inline uint32_t seg_rows_for(uint64_t n, uint64_t m)
{
    const uint64_t want = (n * m + 524287) / 524288;
    uint32_t r = kSegRowsMin;
    while (r < kSegRowsMax && r < want) r <<= 1;
    return r;
}
constexpr uint32_t kLocalSlots = 1024;
constexpr uint32_t kFlagNonFinite = 1u, kFlagTableFull = 2u;

__host__ __device__ inline uint32_t mix32(uint32_t k)
{
    k ^= k >> 16; k *= 0x7feb352du; k ^= k >> 15; k *= 0x846ca68bu; k ^= k >> 16;
    return k;
}

__global__ void fill_zero_kernel(uint32_t* p, uint64_t count)
{
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (; i < count; i += stride) p[i] = 0u;
}

__device__ void table_add(uint32_t* keys, uint32_t* cnts, uint32_t* flags, uint32_t key, uint32_t add)
{
    uint32_t h = mix32(key) & (kHashSlots - 1);
    for (uint32_t probe = 0; probe < kHashSlots; ++probe) {
        const uint32_t old = atomicCAS(&keys[h], 0u, key);
        if (old == 0u || old == key) { atomicAdd(&cnts[h], add); return; }
        h = (h + 1) & (kHashSlots - 1);
    }
    atomicOr(flags, kFlagTableFull);
}

// Step 1.  A wavefront takes tiles of 32 rows x 64 columns, all 32 loads of a tile in flight at once;
// lane l owns column l, so the bit of every row falls into the lane's own word.  A prefix sum of the
// lanes' counts gives every lane its place in the tile's list; the list is put together in LDS, from
// where the wavefront counts it (64 values at a time, whatever the density) and copies it out.  Tiles
// are dealt over a grid that fits the chip once, so that a block merges its histogram only once.
// The words and the room per tile need no atomics; what bounds it is reading W.
// mask, off: [rows / 32][m]; values: [rows / 32][m][kQuota], a tile's columns' room taken as one list.
__global__ void __launch_bounds__(64 * kScanWaves)
enc_scan_kernel(const float* __restrict__ W, uint32_t n, uint32_t m, uint64_t ldw, uint32_t col_groups, uint32_t tiles,
                uint32_t* __restrict__ mask, uint16_t* __restrict__ off, uint32_t* __restrict__ values,
                uint32_t* keys, uint32_t* cnts, uint32_t* flags)
{
    __shared__ uint32_t lk[kLocalSlots], lc[kLocalSlots], queue[kScanWaves][kScanQueue];
    for (uint32_t i = threadIdx.x; i < kLocalSlots; i += 64 * kScanWaves) { lk[i] = 0u; lc[i] = 0u; }
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t* q = queue[wave];
    bool non_finite = false;
    auto count_value = [&](uint32_t key) {
        if ((key & 0x7f800000u) == 0x7f800000u) { non_finite = true; return; }
        uint32_t h = mix32(key) & (kLocalSlots - 1);
        for (uint32_t probe = 0; probe < 64; ++probe) {
            uint32_t cur = __hip_atomic_load(&lk[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (cur == 0u) cur = atomicCAS(&lk[h], 0u, key);
            if (cur == 0u || cur == key) { atomicAdd(&lc[h], 1u); return; }
            h = (h + 1) & (kLocalSlots - 1);
        }
        table_add(keys, cnts, flags, key, 1u);                       // the block's table is crowded
    };
    for (uint32_t tile = blockIdx.x * kScanWaves + wave; tile < tiles; tile += gridDim.x * kScanWaves) {
        const uint32_t w = tile / col_groups, j = (tile - w * col_groups) * kTileCols + lane, r0 = w * kTileRows;
        const float* col = W + (uint64_t)r0 * ldw + (j < m ? j : m - 1);
        const uint32_t rows = n - r0 < kTileRows ? n - r0 : kTileRows;
        float v[kTileRows];
        if (rows == kTileRows) {
#pragma unroll
            for (uint32_t u = 0; u < kTileRows; ++u) v[u] = col[u * ldw];
        } else {
#pragma unroll
            for (uint32_t u = 0; u < kTileRows; ++u) v[u] = u < rows ? col[u * ldw] : 0.0f;
        }
        uint32_t word = 0;
#pragma unroll
        for (uint32_t u = 0; u < kTileRows; ++u) word |= (v[u] != 0.0f ? 1u : 0u) << u;   // +0.0 and -0.0 are the null entry
        if (j >= m) word = 0;
        const uint32_t cnt = __popc(word);
        uint32_t incl = cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) { const uint32_t t = __shfl_up(incl, d, 64); if ((int)lane >= d) incl += t; }
        const uint32_t total = __builtin_amdgcn_readfirstlane(__shfl(incl, 63, 64));
        const uint32_t j0 = j - lane;
        const bool packed = total <= kQuota * (m - j0 < kTileCols ? m - j0 : kTileCols);
        if (j < m) {
            mask[(uint64_t)w * m + j] = word;
            off[(uint64_t)w * m + j] = (uint16_t)(packed ? incl - cnt : kNotPacked);
        }
        if (total <= kScanQueue) {
            uint32_t at = incl - cnt;
#pragma unroll
            for (uint32_t u = 0; u < kTileRows; ++u)
                if (word >> u & 1u) q[at++] = __float_as_uint(v[u]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (uint32_t i = lane; i < total; i += 64) {
                const uint32_t key = q[i];
                if (packed) values[((uint64_t)w * m + j0) * kQuota + i] = key;
                count_value(key);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // read before the next tile's list is written
            __builtin_amdgcn_wave_barrier();
        } else {                                                     // half of the tile or more: most lanes have work in every row
#pragma unroll
            for (uint32_t u = 0; u < kTileRows; ++u)
                if (word >> u & 1u) count_value(__float_as_uint(v[u]));
        }
    }
    if (non_finite) atomicOr(flags, kFlagNonFinite);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kLocalSlots; i += 64 * kScanWaves)
        if (lk[i]) table_add(keys, cnts, flags, lk[i], lc[i]);
}

// What step 1 leaves behind, and the code: three arrays of `slots` words (a power of two, at most half
// full): a value's bit pattern (0: empty), its codeword, its length.
struct Survivors {
    const float* W; uint32_t n, m; uint64_t ldw;
    const uint32_t* mask; const uint16_t* off; const uint32_t* values;
    const uint32_t* table; uint32_t slots;
    uint32_t col_blocks, seg_rows;
};

// the code table in LDS when it is small (LDS_TABLE), behind a barrier of the whole block
template <bool LDS_TABLE>
__device__ __forceinline__ const uint32_t* code_table(const Survivors& s, uint32_t* lds)
{
    if (!LDS_TABLE) return s.table;
    for (uint32_t i = threadIdx.x; i < 3 * s.slots; i += 256) lds[i] = s.table[i];
    __syncthreads();
    return lds;
}

__device__ __forceinline__ uint32_t slot_of(const uint32_t* __restrict__ table, uint32_t slots, uint32_t key)
{
    uint32_t h = mix32(key) & (slots - 1);
    for (uint32_t probe = 0; probe < slots && table[h] != key; ++probe) h = (h + 1) & (slots - 1);
    return h;                                                        // the key is there: step 1 saw it
}

// The row after the last non-zero of column j above row r0 (a multiple of 32), 0 if there is none.  Only threads whose
// segment holds a non-zero may ask: the walks of a column then end at each other's segments and add up to its n / 32
// words.  Four words are requested together (200 000 x 64, first and last row only: whole call 1880 -> 740 us).
__device__ __forceinline__ uint32_t row_after_previous(const Survivors& s, uint32_t j, uint32_t r0)
{
    for (uint32_t w = r0 / 32; w > 0; w = w > 4 ? w - 4 : 0u) {
        const uint32_t* p = s.mask + (uint64_t)(w - 1) * s.m + j;
        uint32_t word[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) { word[u] = *p; if (w > u + 1) p -= s.m; }   // (past the top: the top word again)
        if (!(word[0] | word[1] | word[2] | word[3])) continue;                       // (one wait for all four)
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u)
            if (word[u]) return 32 * (w > u ? w - u : 1u) - __clz((int)word[u]);
    }
    return 0;
}

// A thread's segment of a column: its words wait in LDS (each thread reads back only its own), so that the
// lanes of a wavefront step through their words independently and it runs as long as the lane with the
// most non-zeros in the whole segment, not the sum of the words' longest lanes.
struct SegWords { uint32_t mask[kSegWordsMax][256]; uint16_t off[kSegWordsMax][256]; };

__device__ __forceinline__ uint32_t load_segment(const Survivors& s, SegWords& sw, uint32_t j, uint32_t r0, uint32_t r1)
{
    const uint32_t w0 = r0 / 32, words = (r1 - r0 + 31) / 32;
    uint32_t total = 0;
#pragma unroll
    for (uint32_t w = 0; w < kSegWordsMax; ++w) {
        if (w < words) {
            const uint64_t at = (uint64_t)(w0 + w) * s.m + j;
            const uint32_t word = s.mask[at];
            sw.mask[w][threadIdx.x] = word;
            sw.off[w][threadIdx.x] = s.off[at];
            total += __popc(word);
        }
    }
    return total;
}

// f(row, bit pattern) for the segment's `total` non-zeros, in order
template <class F>
__device__ __forceinline__ void for_survivors(const Survivors& s, const SegWords& sw, uint32_t j, uint32_t r0, uint32_t total, F f)
{
    const uint32_t t = threadIdx.x;
    uint32_t w = 0, word = sw.mask[0][t], at = sw.off[0][t];
    const uint32_t* list = s.values + ((uint64_t)(r0 / 32) * s.m + (j - j % kTileCols)) * kQuota;   // of the segment's first tile
    for (uint32_t i = 0; i < total; ++i) {
        while (word == 0) { ++w; word = sw.mask[w][t]; at = sw.off[w][t]; }
        const uint32_t r = r0 + 32 * w + (uint32_t)__builtin_ctz(word);
        word &= word - 1;
        uint32_t key;
        if (at != kNotPacked) key = list[(uint64_t)w * s.m * kQuota + at++];
        else key = __float_as_uint(s.W[(uint64_t)r * s.ldw + j]);
        f(r, key);
    }
}

__device__ __forceinline__ uint32_t rice_len(uint32_t d, uint32_t k)
{
    const uint32_t q = d >> k;
    return q < kRiceEscape ? q + 1 + k : kRiceEscape + 1 + 32;
}

// Step 3.  seg_bits: code bits and, in HAC, the zeros' codewords.  gap_bits (Rice-coded gaps only, else
// nullptr): [k][segment][column] bits of the gap codewords for k = 0..15; gap_total: their 16 sums
// over the matrix (added up in the block first: the sums are 16 addresses for the whole chip).
template <bool LDS_TABLE>
__global__ void __launch_bounds__(256)
enc_bits_kernel(Survivors s, uint32_t zlen, uint32_t* __restrict__ seg_nnz, uint32_t* __restrict__ seg_bits,
                uint32_t* __restrict__ gap_bits, unsigned long long* gap_total, uint64_t seg_cols)
{
    extern __shared__ uint32_t table_lds[];
    __shared__ SegWords sw;
    __shared__ unsigned long long sums[kRiceKMax + 1];
    if (threadIdx.x <= kRiceKMax) sums[threadIdx.x] = 0;
    const uint32_t* table = code_table<LDS_TABLE>(s, table_lds);
    const uint32_t seg = blockIdx.x / s.col_blocks, j = (blockIdx.x - seg * s.col_blocks) * 256 + threadIdx.x;
    const uint32_t r0 = seg * s.seg_rows, r1 = r0 + s.seg_rows < s.n ? r0 + s.seg_rows : s.n;
    const uint64_t at = (uint64_t)seg * s.m + j;
    uint32_t g[kRiceKMax + 1];
#pragma unroll
    for (uint32_t k = 0; k <= kRiceKMax; ++k) g[k] = 0;
    if (j < s.m) {
        uint32_t bits = 0;
        const uint32_t total = load_segment(s, sw, j, r0, r1);
        uint32_t next = gap_bits && total ? row_after_previous(s, j, r0) : 0u;   // the row the next gap counts from
        for_survivors(s, sw, j, r0, total, [&](uint32_t r, uint32_t key) {
            bits += table[2 * s.slots + slot_of(table, s.slots, key)];
            if (gap_bits) {
                const uint32_t d = r - next;
#pragma unroll
                for (uint32_t k = 0; k <= kRiceKMax; ++k) g[k] += rice_len(d, k);
                next = r + 1;
            }
        });
        seg_nnz[at] = total;
        seg_bits[at] = bits + (r1 - r0 - total) * zlen;
    }
    if (!gap_bits) return;
    if (!LDS_TABLE) __syncthreads();                                  // the sums are zeroed
#pragma unroll
    for (uint32_t k = 0; k <= kRiceKMax; ++k) {
        if (j < s.m) gap_bits[(uint64_t)k * seg_cols + at] = g[k];
        unsigned long long t = g[k];                                  // lanes past m hold 0
        for (int d = 32; d >= 1; d >>= 1) t += __shfl_down(t, d, 64);
        if ((threadIdx.x & 63) == 0 && t) atomicAdd(&sums[k], t);
    }
    __syncthreads();
    if (threadIdx.x <= kRiceKMax && sums[threadIdx.x]) atomicAdd(&gap_total[threadIdx.x], sums[threadIdx.x]);
}

// Words of a thread's own run of bits, which it writes from front to back into cleared memory.  Only the
// run's first and last word are shared with other threads; every word between is stored whole.
struct BitRun {
    uint32_t* words;
    uint32_t first, cur, acc;
    __device__ __forceinline__ void begin(uint32_t* p, uint64_t bit) { words = p; first = cur = (uint32_t)(bit >> 5); acc = 0; }
    __device__ __forceinline__ void flush(bool last)
    {
        if (!acc) return;
        if (last || cur == first) atomicOr(&words[cur], acc); else words[cur] = acc;
    }
    // `len` bits of `code` (right-justified), MSB first, at bit `bit`; 1 <= len <= 32
    __device__ __forceinline__ void put(uint64_t bit, uint32_t code, uint32_t len)
    {
        const uint32_t w = (uint32_t)(bit >> 5), off = (uint32_t)(bit & 31);
        const uint64_t v = (uint64_t)code << (64 - len - off);
        if (w != cur) { flush(false); cur = w; acc = 0; }
        acc |= (uint32_t)(v >> 32);
        if (off + len > 32) { flush(false); cur = w + 1; acc = (uint32_t)v; }
    }
};

struct EmitArgs {
    const uint32_t* seg_bit0; const uint32_t* seg_pos0;                 // within the column
    const uint32_t* col_bit; const uint32_t* col_pos; const uint32_t* col_chunk;
    uint32_t* stream; void* ent; uint32_t* ri;
    uint32_t shac, zcode, zlen, chunk, ent_bits, row_bits, ri_bits;
    uint32_t rice, rice_k;                                              // sHAC with Rice-coded gaps in the stream
};

// Step 5.  Codewords pass through a word in a register (BitRun): with an atomic OR per codeword and
// row-index field this was the longest of the passes.
template <bool LDS_TABLE>
__global__ void __launch_bounds__(256) enc_emit_kernel(Survivors s, EmitArgs a)
{
    extern __shared__ uint32_t table_lds[];
    __shared__ SegWords sw;
    const uint32_t* table = code_table<LDS_TABLE>(s, table_lds);
    const uint32_t seg = blockIdx.x / s.col_blocks, j = (blockIdx.x - seg * s.col_blocks) * 256 + threadIdx.x;
    if (j >= s.m) return;
    const uint32_t r0 = seg * s.seg_rows, r1 = r0 + s.seg_rows < s.n ? r0 + s.seg_rows : s.n;
    const uint64_t at = (uint64_t)seg * s.m + j;
    const uint32_t total = load_segment(s, sw, j, r0, r1);
    if (total == 0 && (a.shac || a.zcode == 0)) return;                 // its zeros are what the cleared stream holds
    const uint32_t cbit0 = a.col_bit[j], cpos0 = a.col_pos[j], cchunk0 = a.col_chunk[j];
    const uint32_t chunk = hac_internal::chunk_of_column(a.chunk, a.col_pos[j + 1] - cpos0);   // of this column
    uint32_t bit = cbit0 + a.seg_bit0[at], q = a.seg_pos0[at];          // q: position within the column
    // (only the chunk entries of HAC and of Rice-coded gaps, and those gaps, start from the non-zero before)
    uint32_t next_row = r0, prow = total && (!a.shac || a.rice) && q ? row_after_previous(s, j, r0) : 0u;
    uint32_t in_chunk = q % chunk, next_chunk = cchunk0 + (q + chunk - 1) / chunk;
    BitRun out, rows;
    out.begin(a.stream, bit);
    rows.begin(a.ri, a.ri ? (uint64_t)(cpos0 + q) * a.ri_bits : 0u);
    auto zeros_up_to = [&](uint32_t r) {                                // HAC: the codewords of rows next_row .. r - 1
        if (a.zcode == 0) { bit += (r - next_row) * a.zlen; return; }
        for (; next_row < r; ++next_row) { out.put(bit, a.zcode, a.zlen); bit += a.zlen; }
    };
    for_survivors(s, sw, j, r0, total, [&](uint32_t r, uint32_t key) {
        const uint32_t slot = slot_of(table, s.slots, key);
        const uint32_t code = table[s.slots + slot], len = table[2 * s.slots + slot];
        if (in_chunk == 0) {
            // HAC and Rice-coded gaps start a chunk right behind the non-zero before it; for HAC that is
            // as many zero codewords back as there are rows since
            uint32_t rel = bit - cbit0;
            if (!a.shac) rel -= (next_row - prow) * a.zlen;
            if (a.shac && !a.rice) {
                if (a.ent_bits == 16) static_cast<uint16_t*>(a.ent)[next_chunk] = (uint16_t)rel;
                else static_cast<uint32_t*>(a.ent)[next_chunk] = rel;
            } else if (a.ent_bits == 32) {
                static_cast<uint32_t*>(a.ent)[next_chunk] = (rel << a.row_bits) | prow;
            } else {
                static_cast<uint32_t*>(a.ent)[2 * (uint64_t)next_chunk] = prow;
                static_cast<uint32_t*>(a.ent)[2 * (uint64_t)next_chunk + 1] = rel;
            }
            ++next_chunk;
        }
        if (++in_chunk == chunk) in_chunk = 0;
        if (!a.shac) zeros_up_to(r);
        if (a.rice) {
            const uint32_t d = r - prow, k = a.rice_k, qq = d >> k;
            if (qq < kRiceEscape) {
                out.put((uint64_t)bit + qq, (1u << k) | (d & ((1u << k) - 1u)), k + 1);
                bit += qq + 1 + k;
            } else {
                out.put((uint64_t)bit + kRiceEscape, 1u, 1);
                out.put((uint64_t)bit + kRiceEscape + 1, d, 32);
                bit += kRiceEscape + 1 + 32;
            }
        }
        out.put(bit, code, len);
        bit += len;
        next_row = prow = r + 1;
        if (a.ri) rows.put((uint64_t)(cpos0 + q) * a.ri_bits, r, a.ri_bits);
        ++q;
    });
    if (!a.shac) zeros_up_to(r1);
    out.flush(true);
    if (a.ri) rows.flush(true);
}

// step 1, second part: the occupied slots of the table as a list of (key, count), in no
// particular order (the host sorts by value); *n_list counts them, entries past `cap` are dropped
// (the host then sees n_list > cap and gives up: more than 65536 distinct values)
__global__ void __launch_bounds__(256)
enc_gather_kernel(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ cnts, uint32_t* list, uint32_t cap, uint32_t* n_list)
{
    const uint32_t h = blockIdx.x * 256 + threadIdx.x;
    if (h >= kHashSlots) return;
    const uint32_t key = keys[h];
    if (!key) return;
    const uint32_t i = atomicAdd(n_list, 1u);
    if (i < cap) { list[2 * (uint64_t)i] = key; list[2 * (uint64_t)i + 1] = cnts[h]; }
}

// Step 3, second part: running sums over the segments of every column (in place: what stands above a
// segment in its column) and the column's totals.  16 columns x 16 ranges of segments per block: a tall
// and narrow matrix has hundreds of segments per column and few columns.
// gap_bits: all 16 parameters; the one with the fewest bits counts, the smaller on ties (as on the host).
__global__ void __launch_bounds__(256)
enc_col_scan_kernel(uint32_t m, uint32_t S, uint32_t* __restrict__ seg_nnz, uint32_t* __restrict__ seg_bits,
                    const uint32_t* __restrict__ gap_bits, const unsigned long long* __restrict__ gap_total, uint64_t seg_cols,
                    uint32_t* __restrict__ col_nnz, unsigned long long* __restrict__ col_bits)
{
    __shared__ uint32_t part_nnz[16][17];
    __shared__ unsigned long long part_bits[16][17];
    const uint32_t c = threadIdx.x & 15, g = threadIdx.x >> 4, j = blockIdx.x * 16 + c;
    if (gap_bits) {
        uint32_t best = 0;
        for (uint32_t k = 1; k <= kRiceKMax; ++k) if (gap_total[k] < gap_total[best]) best = k;
        gap_bits += best * seg_cols;
    }
    const uint32_t per = (S + 15) / 16, s0 = g * per < S ? g * per : S, s1 = s0 + per < S ? s0 + per : S;
    uint32_t nnz = 0;
    unsigned long long bits = 0;
    if (j < m) {
#pragma unroll 4
        for (uint32_t s = s0; s < s1; ++s) {
            const uint64_t at = (uint64_t)s * m + j;
            nnz += seg_nnz[at];
            bits += (unsigned long long)seg_bits[at] + (gap_bits ? gap_bits[at] : 0u);
        }
    }
    part_nnz[g][c] = nnz; part_bits[g][c] = bits;
    __syncthreads();
    if (j >= m) return;
    nnz = 0; bits = 0;
    for (uint32_t o = 0; o < g; ++o) { nnz += part_nnz[o][c]; bits += part_bits[o][c]; }
    if (g == 15) { col_nnz[j] = nnz + part_nnz[15][c]; col_bits[j] = bits + part_bits[15][c]; }
#pragma unroll 4
    for (uint32_t s = s0; s < s1; ++s) {
        const uint64_t at = (uint64_t)s * m + j;
        const uint32_t cn = seg_nnz[at], cb = seg_bits[at] + (gap_bits ? gap_bits[at] : 0u);
        seg_nnz[at] = nnz; seg_bits[at] = (uint32_t)bits;
        nnz += cn; bits += cb;
    }
}

constexpr uint32_t kListCap = 65536 + 64;          // one more than the largest alphabet is enough to see "too many"

struct WsLayout {
    size_t keys, cnts, flags, list, mask, off, values, seg_nnz, seg_bits, gap_bits, table, col_bits, col_nnz, total;
};

WsLayout ws_layout(uint64_t n, uint64_t m)
{
    const uint64_t seg_rows = seg_rows_for(n, m), S = (n + seg_rows - 1) / seg_rows;
    const uint64_t words = (n + 31) / 32;
    WsLayout L;
    size_t c = 0;
    auto take = [&](size_t bytes) { const size_t o = c; c = (c + bytes + 255) / 256 * 256; return o; };
    L.keys = take(4ull * kHashSlots); L.cnts = take(4ull * kHashSlots); L.flags = take(256);
    L.list = take(8ull * kListCap);                                 // behind the flags: one copy to the host
    L.mask = take(4 * words * m); L.off = take(2 * words * m); L.values = take(4ull * kQuota * words * m);
    L.seg_nnz = take(4 * S * m); L.seg_bits = take(4 * S * m);
    L.gap_bits = take(4 * S * m * (kRiceKMax + 1));                  // used with Rice-coded gaps only
    L.table = take(12ull * kHashSlots);
    L.col_bits = take(8 * m); L.col_nnz = take(4 * m);               // side by side: one copy to the host
    L.total = c;
    return L;
}

int hip_fail(hipError_t e) { hac_internal::set_last_hip_error((int)e); return HAC_EHIP; }

} // namespace

namespace {

// `place` is called once, when the header is complete: it returns the blob's memory or nullptr.
template <class Place>
int encode_on_device(uint32_t format, const float* d_W, int64_t n, int64_t m, int64_t ldw, const hac_opts_t* opts,
                     hac_desc_t* desc, void* d_ws, size_t ws_bytes, hac_stream_t stream_, Place place)
{
    if (!d_W || !desc || !d_ws) return HAC_EINVAL;
    if (format != HAC_FORMAT_HAC && format != HAC_FORMAT_SHAC) return HAC_EINVAL;
    if (n < 1 || m < 1 || ldw < m) return HAC_EINVAL;
    if (n > 0x7fffffffll || m > 0x7fffffffll) return HAC_ERANGE;
    if ((uint64_t)n > kMaxRows) return HAC_ERANGE;
    int rc = check_opts(opts);
    if (rc) return rc;
    if (opts && opts->chunk_rows) return HAC_EINVAL;                   // the row index is built by the host encoders only
    const bool shac = format == HAC_FORMAT_SHAC;
    const bool rice = opts && opts->ri_coding == HAC_RI_RICE;
    if (rice && (!shac || opts->ri_bits)) return HAC_EINVAL;          // as the host encoders
    const uint32_t need_bits = std::max<uint32_t>(ceil_log2((uint64_t)n), 1);
    uint32_t ri_bits = 0;
    if (shac && !rice) {
        ri_bits = opts && opts->ri_bits ? opts->ri_bits : need_bits;
        if (ri_bits < need_bits || ri_bits > 32) return HAC_EINVAL;
    }
    if (reinterpret_cast<uintptr_t>(d_ws) % 256) return HAC_EINVAL;
    const WsLayout L = ws_layout((uint64_t)n, (uint64_t)m);
    if (ws_bytes < L.total) return HAC_EWORKSPACE;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    hac_internal::set_last_hip_error(0);
    uint8_t* ws = static_cast<uint8_t*>(d_ws);
    auto dptr = [&](size_t off) { return reinterpret_cast<uint32_t*>(ws + off); };
    const uint32_t seg_rows = seg_rows_for((uint64_t)n, (uint64_t)m);
    const uint32_t S = (uint32_t)(((uint64_t)n + seg_rows - 1) / seg_rows);
    const uint64_t SM = (uint64_t)S * (uint64_t)m;
    Survivors sv;
    sv.W = d_W; sv.n = (uint32_t)n; sv.m = (uint32_t)m; sv.ldw = (uint64_t)ldw;
    sv.mask = dptr(L.mask); sv.off = reinterpret_cast<uint16_t*>(ws + L.off); sv.values = dptr(L.values);
    sv.table = dptr(L.table);
    sv.col_blocks = (uint32_t)(((uint64_t)m + 255) / 256);
    sv.seg_rows = seg_rows;
    const uint32_t col_groups = (uint32_t)(((uint64_t)m + kTileCols - 1) / kTileCols);
    const uint64_t tiles = ((uint64_t)n + kTileRows - 1) / kTileRows * col_groups;
    if (tiles > 0x7fffffffull || (uint64_t)sv.col_blocks * S > 0x7fffffffull) return HAC_ERANGE;   // terabytes of W
    const dim3 seg_grid(sv.col_blocks * S);
    hipError_t e;
    try {
        // ---- step 1 ----
        uint32_t* d_flags = dptr(L.flags);                           // [0] flags, [1] length of the list, +64 bytes: gap totals
        hipLaunchKernelGGL(fill_zero_kernel, dim3(512), dim3(256), 0, stream, dptr(L.keys), (uint64_t)(L.list - L.keys) / 4);
        const uint64_t scan_blocks = std::min<uint64_t>((tiles + kScanWaves - 1) / kScanWaves, kScanBlocks);
        hipLaunchKernelGGL(enc_scan_kernel, dim3((uint32_t)scan_blocks), dim3(64 * kScanWaves), 0, stream, d_W, (uint32_t)n, (uint32_t)m,
                           (uint64_t)ldw, col_groups, (uint32_t)tiles, dptr(L.mask), reinterpret_cast<uint16_t*>(ws + L.off),
                           dptr(L.values), dptr(L.keys), dptr(L.cnts), d_flags);
        hipLaunchKernelGGL(enc_gather_kernel, dim3(kHashSlots / 256), dim3(256), 0, stream, dptr(L.keys), dptr(L.cnts),
                           dptr(L.list), kListCap, d_flags + 1);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e);
        // flags, the length of the list and its first entries (they sit side by side), then the rest of
        // the list; a small alphabet arrives with the first copy
        constexpr uint32_t kFirst = 1024, kHead = 64;                // words
        std::vector<uint32_t> head(kHead + 2 * (size_t)kFirst);
        if ((e = hipMemcpyAsync(head.data(), d_flags, 4 * head.size(), hipMemcpyDeviceToHost, stream)) != hipSuccess) return hip_fail(e);
        if ((e = hipStreamSynchronize(stream)) != hipSuccess) return hip_fail(e);
        const uint32_t flags = head[0], n_list = head[1];
        if (flags & kFlagNonFinite) return HAC_EINVAL;
        if (flags & kFlagTableFull) return HAC_ERANGE;
        if (n_list > 65536) return HAC_ERANGE;
        if (n_list > kFirst) {
            head.resize(kHead + 2 * (size_t)n_list);
            if ((e = hipMemcpyAsync(head.data(), d_flags, 4 * head.size(), hipMemcpyDeviceToHost, stream)) != hipSuccess) return hip_fail(e);
            if ((e = hipStreamSynchronize(stream)) != hipSuccess) return hip_fail(e);
        }
        const uint32_t* list = head.data() + kHead;

        // ---- step 2 ----
        struct Val { float v; uint32_t key; uint64_t f; };
        std::vector<Val> vals(n_list);
        uint64_t nnz = 0;
        for (uint32_t i = 0; i < n_list; ++i) {
            vals[i].key = list[2 * (size_t)i]; vals[i].f = list[2 * (size_t)i + 1];
            std::memcpy(&vals[i].v, &vals[i].key, 4);
            nnz += vals[i].f;
        }
        if (nnz > 0xfffffff0ull) return HAC_ERANGE;
        std::sort(vals.begin(), vals.end(), [](const Val& a, const Val& b) { return a.v < b.v; });
        const uint64_t zeros = (uint64_t)n * (uint64_t)m - nnz;
        const bool has_zero = !shac && zeros > 0;
        const uint32_t shift = has_zero ? 1u : 0u;
        std::vector<float> codebook;
        std::vector<uint64_t> freq;
        if (has_zero) { codebook.push_back(0.0f); freq.push_back(zeros); }
        for (const Val& x : vals) { codebook.push_back(x.v); freq.push_back(x.f); }
        std::vector<uint8_t> len; uint32_t lmax = 0;
        if (!huffman_lengths(freq, len, lmax)) return HAC_ERANGE;
        CodeTables t; canonical_codes(len, t);
        uint64_t total_bits = 0;
        for (size_t i = 0; i < freq.size(); ++i) total_bits += freq[i] * len[i];
        if (total_bits > 0xfffffff0ull) return HAC_ERANGE;
        const uint32_t lut_bits = pick_lut_bits(opts, lmax);
        if (lut_bits < 1 || lut_bits > 12) return HAC_EINVAL;
        std::vector<uint32_t> lut; build_lut(len, t, lut_bits, lut);
        const uint32_t zlen = has_zero ? len[0] : 0, zcode = has_zero ? t.code[0] : 0;

        // bit pattern -> codeword, at most a quarter full (half for the largest alphabets)
        uint32_t slots = 64;
        while (slots < 4 * (uint64_t)n_list && slots < kHashSlots) slots <<= 1;
        std::vector<uint32_t> table(3 * (size_t)slots, 0);
        for (size_t i = 0; i < vals.size(); ++i) {
            uint32_t h = mix32(vals[i].key) & (slots - 1);
            while (table[h]) h = (h + 1) & (slots - 1);
            table[h] = vals[i].key; table[slots + h] = t.code[i + shift]; table[2 * (size_t)slots + h] = len[i + shift];
        }
        if ((e = hipMemcpyAsync(dptr(L.table), table.data(), 4 * table.size(), hipMemcpyHostToDevice, stream)) != hipSuccess) return hip_fail(e);
        sv.slots = slots;
        const bool lds_table = slots <= kCodeSlotsLds;
        const size_t table_lds = lds_table ? 12 * (size_t)slots : 0;

        // ---- step 3 ----
        unsigned long long* d_gap_total = reinterpret_cast<unsigned long long*>(ws + L.flags + 64);   // zeroed with the flags
        uint32_t* d_gap_bits = rice ? dptr(L.gap_bits) : static_cast<uint32_t*>(nullptr);
        hipLaunchKernelGGL(lds_table ? enc_bits_kernel<true> : enc_bits_kernel<false>, seg_grid, dim3(256), table_lds, stream, sv, zlen,
                           dptr(L.seg_nnz), dptr(L.seg_bits), d_gap_bits, d_gap_total, SM);
        unsigned long long* d_col_bits = reinterpret_cast<unsigned long long*>(ws + L.col_bits);
        hipLaunchKernelGGL(enc_col_scan_kernel, dim3((uint32_t)(((uint64_t)m + 15) / 16)), dim3(256), 0, stream, (uint32_t)m, S,
                           dptr(L.seg_nnz), dptr(L.seg_bits), static_cast<const uint32_t*>(d_gap_bits),
                           static_cast<const unsigned long long*>(d_gap_total), SM, dptr(L.col_nnz), d_col_bits);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e);
        unsigned long long gap_total[kRiceKMax + 1] = { 0 };
        if (rice && (e = hipMemcpyAsync(gap_total, d_gap_total, sizeof gap_total, hipMemcpyDeviceToHost, stream)) != hipSuccess) return hip_fail(e);
        std::vector<uint8_t> col_sums(L.col_nnz - L.col_bits + 4 * (size_t)m);
        if ((e = hipMemcpyAsync(col_sums.data(), d_col_bits, col_sums.size(), hipMemcpyDeviceToHost, stream)) != hipSuccess) return hip_fail(e);
        if ((e = hipStreamSynchronize(stream)) != hipSuccess) return hip_fail(e);
        const unsigned long long* col_bits = reinterpret_cast<const unsigned long long*>(col_sums.data());
        const uint32_t* col_nnz = reinterpret_cast<const uint32_t*>(col_sums.data() + (L.col_nnz - L.col_bits));
        // the Rice parameter: fewest gap bits, the smaller k on ties
        uint32_t rice_k = 0; uint64_t gap_bits = 0;
        if (rice) {
            for (uint32_t k = 1; k <= kRiceKMax; ++k) if (gap_total[k] < gap_total[rice_k]) rice_k = k;
            gap_bits = gap_total[rice_k];
            total_bits += gap_bits;
            if (total_bits > 0xfffffff0ull) return HAC_ERANGE;
        }

        // ---- step 4 ----
        uint64_t max_col_nnz = 0, max_col_bits = 0;
        for (int64_t j = 0; j < m; ++j) {
            max_col_nnz = std::max<uint64_t>(max_col_nnz, col_nnz[(size_t)j]);
            max_col_bits = std::max<uint64_t>(max_col_bits, col_bits[(size_t)j]);
        }
        const uint32_t Cn = pick_chunk(opts, max_col_nnz);
        // the three per-column arrays sit side by side in the blob (256-byte aligned sections): one
        // host buffer with the same spacing, one copy
        const size_t col_stride = (4 * ((size_t)m + 1) + 255) / 256 * 256 / 4;       // words from one array to the next
        std::vector<uint32_t> col_arrays(3 * col_stride, 0);
        uint32_t* col_chunk = col_arrays.data();
        uint32_t* col_pos = col_chunk + col_stride;
        uint32_t* col_bit = col_pos + col_stride;
        uint64_t bit = 0, pos = 0, chunks = 0;
        for (int64_t j = 0; j < m; ++j) {
            col_bit[(size_t)j] = (uint32_t)bit; col_pos[(size_t)j] = (uint32_t)pos; col_chunk[(size_t)j] = (uint32_t)chunks;
            bit += col_bits[(size_t)j]; pos += col_nnz[(size_t)j];
            const uint32_t cj = chunk_of_column(Cn, col_nnz[(size_t)j]);
            chunks += (col_nnz[(size_t)j] + cj - 1) / cj;
        }
        col_bit[(size_t)m] = (uint32_t)bit; col_pos[(size_t)m] = (uint32_t)pos; col_chunk[(size_t)m] = (uint32_t)chunks;
        if (bit != total_bits || pos != nnz) return HAC_EFORMAT;
        if (chunks > 0xfffffff0ull) return HAC_ERANGE;

        hac_desc_t d;
        std::memset(&d, 0, sizeof d);
        d.magic = kMagic; d.version = kVersion; d.format = format; d.header_bytes = 256;
        d.n = (uint64_t)n; d.m = (uint64_t)m; d.nnz = nnz; d.total_bits = total_bits; d.n_words = (total_bits + 31) / 32;
        d.k_sym = (uint32_t)codebook.size(); d.lmax = lmax; d.lut_bits = lut_bits;
        d.chunk = Cn; d.n_chunks = chunks; d.max_col_bits = max_col_bits; d.max_col_nnz = max_col_nnz;
        if (rice) {
            const uint32_t brel_bits = std::max<uint32_t>(ceil_log2(max_col_bits + 1), 1);
            d.ent_bits = need_bits + brel_bits <= 32 ? 32 : 64;
            d.row_bits = d.ent_bits == 32 ? need_bits : 0;
            d.ri_coding = HAC_RI_RICE; d.rice_k = rice_k; d.gap_bits = gap_bits;
        } else if (shac) {
            d.ri_bits = ri_bits;
            d.ent_bits = max_col_bits < 65536 ? 16 : 32;
            if (nnz * (uint64_t)ri_bits > 0xfffffff0ull * 32ull) return HAC_ERANGE;
        } else {
            d.has_zero = has_zero ? 1 : 0;
            d.zero_len = (has_zero && zcode == 0) ? zlen : 0;
            const uint32_t brel_bits = std::max<uint32_t>(ceil_log2(max_col_bits + 1), 1);
            d.ent_bits = need_bits + brel_bits <= 32 ? 32 : 64;
            d.row_bits = d.ent_bits == 32 ? need_bits : 0;
        }
        place_sections(d);
        *desc = d;
        void* d_blob = place((size_t)d.blob_bytes);
        if (!d_blob) return HAC_EWORKSPACE;                                         // desc->blob_bytes says how much
        if (reinterpret_cast<uintptr_t>(d_blob) % 256) return HAC_EINVAL;

        // head of the blob (header, tables, per-column arrays) is assembled here and copied over
        const size_t head_bytes = (size_t)d.off_stream;
        std::vector<uint8_t> blob_head(head_bytes, 0);
        std::memcpy(blob_head.data(), &d, sizeof d);
        write_tables(blob_head.data(), d, codebook, len, t, lut);
        uint8_t* blob = static_cast<uint8_t*>(d_blob);
        hipLaunchKernelGGL(fill_zero_kernel, dim3(1024), dim3(256), 0, stream, reinterpret_cast<uint32_t*>(blob + d.off_stream),
                           (uint64_t)(d.blob_bytes - d.off_stream) / 4);
        if ((e = hipMemcpyAsync(blob, blob_head.data(), head_bytes, hipMemcpyHostToDevice, stream)) != hipSuccess) return hip_fail(e);
        if (d.off_col_pos - d.off_col_chunk != 4 * col_stride || d.off_col_bit - d.off_col_pos != 4 * col_stride) return HAC_EFORMAT;
        if ((e = hipMemcpyAsync(blob + d.off_col_chunk, col_chunk, 4 * (2 * col_stride + (size_t)m + 1), hipMemcpyHostToDevice, stream)) != hipSuccess) return hip_fail(e);

        // ---- step 5 ----
        EmitArgs a;
        a.seg_bit0 = dptr(L.seg_bits); a.seg_pos0 = dptr(L.seg_nnz);
        a.col_bit = reinterpret_cast<const uint32_t*>(blob + d.off_col_bit);
        a.col_pos = reinterpret_cast<const uint32_t*>(blob + d.off_col_pos);
        a.col_chunk = reinterpret_cast<const uint32_t*>(blob + d.off_col_chunk);
        a.stream = reinterpret_cast<uint32_t*>(blob + d.off_stream);
        a.ent = blob + d.off_chunk_ent;
        a.ri = (shac && !rice) ? reinterpret_cast<uint32_t*>(blob + d.off_ri) : nullptr;
        a.rice = rice ? 1u : 0u; a.rice_k = rice_k;
        a.shac = shac ? 1u : 0u; a.zcode = zcode; a.zlen = zlen;
        a.chunk = Cn; a.ent_bits = d.ent_bits; a.row_bits = d.row_bits; a.ri_bits = ri_bits;
        hipLaunchKernelGGL(lds_table ? enc_emit_kernel<true> : enc_emit_kernel<false>, seg_grid, dim3(256), table_lds, stream, sv, a);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e);
        // the host vectors above feed asynchronous copies: they must outlive them
        if ((e = hipStreamSynchronize(stream)) != hipSuccess) return hip_fail(e);
        return HAC_OK;
    } catch (const std::bad_alloc&) {
        return HAC_ENOMEM;
    }
}

} // namespace

extern "C" size_t hac_encode_dev_workspace_bytes(int64_t n, int64_t m)
{
    if (n < 1 || m < 1 || n > 0x7fffffffll || m > 0x7fffffffll) return 0;
    return ws_layout((uint64_t)n, (uint64_t)m).total;
}

extern "C" int hac_encode_dev(uint32_t format, const float* d_W, int64_t n, int64_t m, int64_t ldw,
                              const hac_opts_t* opts, void* d_blob, size_t blob_capacity, hac_desc_t* desc,
                              void* d_ws, size_t ws_bytes, hac_stream_t stream)
{
    if (d_blob && reinterpret_cast<uintptr_t>(d_blob) % 256) return HAC_EINVAL;
    return encode_on_device(format, d_W, n, m, ldw, opts, desc, d_ws, ws_bytes, stream,
                            [&](size_t bytes) { return blob_capacity >= bytes ? d_blob : nullptr; });
}

extern "C" int hac_encode_dev_alloc(uint32_t format, const float* d_W, int64_t n, int64_t m, int64_t ldw,
                                    const hac_opts_t* opts, hac_alloc_t alloc, void* alloc_ctx, hac_desc_t* desc,
                                    void* d_ws, size_t ws_bytes, hac_stream_t stream)
{
    if (!alloc) return HAC_EINVAL;
    return encode_on_device(format, d_W, n, m, ldw, opts, desc, d_ws, ws_bytes, stream,
                            [&](size_t bytes) { return alloc(bytes, alloc_ctx); });
}
