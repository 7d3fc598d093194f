// GPU-side encoder: builds a HAC or sHAC blob (arXiv 2108.12704 Sect. IV-B / IV-C) from a matrix
// that already lives in device memory, byte for byte the blob hac_encode / shac_encode would build
// on the host.
//
// The steps of the host encoder:
//   1. the one pass over W: per 32 rows of a column a word with a bit per non-zero, the
//      non-zeros themselves packed column by column (where they are few), and a histogram
//      of the distinct fp32 values (a hash table keyed by bit pattern, privatised in LDS
//      per block, and a list of its occupied slots);
//   2. alphabet in value order, Huffman lengths, canonical code, decode tables, and a
//      small hash table from a value's bit pattern to its codeword: one block, up to kDevSymbols
//      values; a larger alphabet comes to the host, which then does this step;
//   3. non-zeros and stream bits of every (row segment, column) from the words and the
//      packed values; with Rice-coded row gaps also the gap bits for every parameter
//      k = 0..15; then, per column, running sums over its segments and their totals;
//   4. chunk size and prefix sums over the columns (first stream bit, CSC position, first
//      chunk of every column); the host learns the counts, places the sections and asks for the
//      blob's memory;
//   5. header, tables and column arrays are copied into the blob and the rest of it cleared; one
//      thread per (row segment, column) writes the codewords (and row-index fields or
//      gap codewords) of its non-zeros, and the chunk entries.
// W is far larger than everything else, so it is read once.  A word costs 1/32 of what it stands for
// and a packed list is as long as the non-zeros, so steps 3 and 5 move a few per cent of W's bytes
// on a pruned layer; where more than an eighth of a 32 x 64 tile is non-zero its values are not
// packed but fetched from W again, by then mostly whole cache lines.
// 25088 x 4096, 2 % non-zero: the three passes over W that this replaces took 0.25 + 0.36 + 0.40 ms.
// The host waits once before step 5, for a few counts that the device writes into pinned memory, and
// once at the end; steps 1 to 4 are launched one after the other without it.  With steps 2 and 4 on the host, which
// took the histogram and the columns' sums over the bus and sent tables and column arrays back (three waits, six copies),
// a call on a small matrix took 114 us (700 x 90; 89 now) where its kernels run for 50.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "hac_hostlib.h"

namespace {

using namespace hac_internal;

constexpr uint32_t kHashSlots = 1u << 17;          // distinct values <= 65536 keep the load below 1/2
constexpr uint32_t kSegRowsMax = 512, kSegRowsMin = 32;   // multiples of 32: a segment is whole words
constexpr uint64_t kMaxRows = 65535ull * 1024;
constexpr uint32_t kTileCols = 64, kTileRows = 32;        // what a wavefront reads at a time in step 1
constexpr uint32_t kQuota = 4;                            // packed values per column of a tile: an eighth of it
constexpr uint32_t kNotPacked = 0xffffu;
constexpr uint32_t kScanWaves = 8, kScanQueue = 1024, kScanBlocks = 512;   // two blocks a CU: their registers fill it
constexpr uint64_t kCachedEntries = 64u << 20;            // 256 MB of W, the size of the memory-side cache
constexpr uint32_t kCodeSlotsLds = 2048;                  // code tables up to this size (24 KB) are copied to LDS

// Rows per segment: 512 on a large matrix, fewer on a small one, so that there are about 256 K
// (segment, column) threads.  What bounds the emission is the atomics on the words that two segments share (1.3 million with
// segments of 256 rows at 25088 x 4096, 2 %; half the segments, half of them) and lanes that wait for the one with the most non-zeros
// (12.5 turns for 5.1 non-zeros a lane, 17 for 10); whole calls with 512 K threads -> 256 K -> 128 K: that layer 245 -> 226 -> 245 us,
// 12000 x 2000, 10 % 209 -> 183 -> 195, 4096 x 4096, 40 % 298 -> 287 -> 324.
__host__ inline uint32_t seg_rows_for(uint64_t n, uint64_t m)
{
    const uint64_t want = (n * m + 262143) / 262144;
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

// The histogram of the whole matrix: keys and counts, and the slots in use in the order in which they were taken, as many
// as step 2 takes on the device; flags[1] counts them until there are more (an alphabet of 40000 would add to that one word
// 40000 times).
constexpr uint32_t kDevSymbols = 512;              // non-zero values of an alphabet whose code is built on the device
struct Histogram { uint32_t* keys; uint32_t* cnts; uint32_t* used; uint32_t* flags; };

__device__ void table_add(const Histogram& t, uint32_t key, uint32_t add)
{
    uint32_t h = mix32(key) & (kHashSlots - 1);
    for (uint32_t probe = 0; probe < kHashSlots; ++probe) {
        const uint32_t old = atomicCAS(&t.keys[h], 0u, key);
        if (old == 0u && __hip_atomic_load(&t.flags[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= kDevSymbols) {
            const uint32_t i = atomicAdd(&t.flags[1], 1u);
            if (i < kDevSymbols) t.used[i] = h;
        }
        if (old == 0u || old == key) { atomicAdd(&t.cnts[h], add); return; }
        h = (h + 1) & (kHashSlots - 1);
    }
    atomicOr(t.flags, kFlagTableFull);
}

// Step 1.  A wavefront takes tiles of 32 rows x 64 columns, all 32 loads of a tile in flight at once;
// lane l owns column l, so the bit of every row falls into the lane's own word.  A prefix sum of the
// lanes' counts gives every lane its place in the tile's list; the list is put together in LDS, from
// where the wavefront counts it (64 values at a time, whatever the density) and copies it out.  Tiles
// are dealt over a grid that fits the chip once, so that a block merges its histogram only once (4096 x 4096, 40 %, with twice as
// many blocks 286 us for the whole call, 274 so; a W that comes from memory is read more evenly by twice as many: 220.5 and 218.5).
// The words and the room per tile need no atomics; what bounds it is reading W.
// ONCE: W does not stay in any cache until the emission may ask for some of it again, and is read past them (25088 x 4096, 411 MB:
// 227 -> 218 us for the whole call; but 4096 x 4096, 40 %, 286 -> 292).
// mask, off: [rows / 32][m]; values: [rows / 32][m][kQuota], a tile's columns' room taken as one list.
template <bool ONCE>
__global__ void __launch_bounds__(64 * kScanWaves)
enc_scan_kernel(const float* __restrict__ W, uint32_t n, uint32_t m, uint64_t ldw, uint32_t col_groups, uint32_t tiles,
                uint32_t* __restrict__ mask, uint16_t* __restrict__ off, uint32_t* __restrict__ values, Histogram table)
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
        table_add(table, key, 1u);                       // the block's table is crowded
    };
    for (uint32_t tile = blockIdx.x * kScanWaves + wave; tile < tiles; tile += gridDim.x * kScanWaves) {
        const uint32_t w = tile / col_groups, j = (tile - w * col_groups) * kTileCols + lane, r0 = w * kTileRows;
        const float* col = W + (uint64_t)r0 * ldw + (j < m ? j : m - 1);
        const uint32_t rows = n - r0 < kTileRows ? n - r0 : kTileRows;
        float v[kTileRows];
        if (rows == kTileRows) {
#pragma unroll
            for (uint32_t u = 0; u < kTileRows; ++u) v[u] = ONCE ? __builtin_nontemporal_load(col + u * ldw) : col[u * ldw];
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
    if (non_finite) atomicOr(table.flags, kFlagNonFinite);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kLocalSlots; i += 64 * kScanWaves)
        if (lk[i]) table_add(table, lk[i], lc[i]);
}

// ---------------------------------------------------------------------------
// step 2
// ---------------------------------------------------------------------------
constexpr uint32_t kDevSlots = 2 * kDevSymbols;    // its code table: at most half full
constexpr uint32_t kCodeThreads = kDevSymbols + 64;   // of the block that builds it: a thread a symbol; idle wavefronts cost the others time
constexpr uint32_t kPairUp = 64;                   // symbols from which all merges of a turn are made at once

enum : uint32_t { kCodeOk, kCodeNonFinite, kCodeRange, kCodeOnHost };
struct EncCode {
    uint32_t status, values, k_sym, lmax, lut_bits, has_zero, zcode, zlen, slots;
    uint64_t nnz, bits;                            // of the codewords of all symbols
};
// What the host waits for: the code and step 4's sums.
struct EncResult {
    EncCode code;
    uint32_t chunk, rice_k;
    uint64_t max_col_nnz, max_col_bits, col_bits, col_nnz, chunks, gap_bits;
};
// tables of the blob, as step 2 leaves them in the workspace (words)
struct DevTables { uint32_t codebook[kDevSymbols + 4], codelen[(kDevSymbols + 4) / 4], canon[100], symsort[kDevSymbols + 4], lut[4096]; };

// of the sorted w[from .. to): how many are less than `than`
__device__ __forceinline__ uint32_t count_below(const uint32_t* w, uint32_t from, uint32_t to, uint32_t than)
{
    uint32_t lo = from, hi = to;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (w[mid] < than) lo = mid + 1; else hi = mid;
    }
    return lo - from;
}

// One block.  Symbols are numbered by counting smaller ones.  Huffman's merging: leaves in order of (count, symbol) and merged
// nodes in the order of their making are two queues whose heads are the smallest left, the leaf first where they are
// equal, which is the order that the host's heap gives (weight, then node number).  Two ways:
//   one thread walks the queues, 0.2 us a merge, each a chain of reads from LDS (one wavefront with the heads of the queues in scalar
//   registers, a chain of 50 instructions and no wait: 0.23 us);
//   from kPairUp symbols on the block pairs off, in order and at once, everything that weighs up to s, the two smallest
//   together: no node made from now on weighs less, and one of the same weight comes behind all there are.  8 to 22 turns of about 1 us
//   for 16 to 256 values by k-means or equal bins (s grows like Fibonacci's numbers at least).
// The kernel takes 13 us for 32 values in equal bins and 22 for 200 by k-means (one thread: 49).
__global__ void __launch_bounds__(kCodeThreads)
enc_code_kernel(Histogram h, uint64_t entries, uint32_t shac, uint32_t lut_opt, uint32_t* __restrict__ table, DevTables* __restrict__ out, EncCode* __restrict__ code)
{
    constexpr uint32_t K = kDevSymbols + 1;
    __shared__ unsigned long long sum;
    __shared__ __align__(16) uint32_t freq[K + 3];
    __shared__ uint32_t leaf[kCodeThreads], node[kCodeThreads], merged[2 * K], upto[2][2], last_is_node;
    __shared__ __align__(16) uint32_t order[(kDevSymbols + 3) / 4 * 4];
    __shared__ __align__(16) uint32_t lens[(K + 3) / 4];
    __shared__ uint32_t key_of[K], leaf_sym[K], parent[2 * K], sort[K], codes[K], count[33], first_code[33], first_index[33];
    __shared__ uint32_t wave_count[kCodeThreads / 64][33];
    __shared__ uint32_t tkey[kDevSlots], tcode[kDevSlots], tlen[kDevSlots];
    __shared__ uint32_t bad;
    const uint32_t t = threadIdx.x;
    const uint32_t flags = h.flags[0], nv = h.flags[1];
    if (flags || nv > kDevSymbols || entries >= 0xffffffffull) {           // (weights of 32 bits here)
        if (t == 0) {
            code->status = flags & kFlagNonFinite ? kCodeNonFinite : flags ? kCodeRange : kCodeOnHost;
        }
        return;
    }
    uint8_t* len = reinterpret_cast<uint8_t*>(lens);
    uint32_t key = 0, cnt = 0;
    if (t < nv) { const uint32_t s = h.used[t]; key = h.keys[s]; cnt = h.cnts[s]; }
    if (t == 0) { sum = 0; bad = 0; }
    if (t < 33) count[t] = 0;
    node[t] = ~0u;
    const uint32_t ordered = key ^ (key >> 31 ? 0xffffffffu : 0x80000000u);     // unsigned order = order of the floats
    if (t < (kDevSymbols + 3) / 4 * 4) order[t] = t < nv ? ordered : 0xffffffffu;   // (that is a NaN's: larger than any value here)
    __syncthreads();
    auto add_up = [&](unsigned long long v) {                              // of the block's threads, to `sum`
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
        if ((t & 63u) == 0 && v) atomicAdd(&sum, v);
    };
    add_up(cnt);
    uint32_t rank = 0;
    if (t < nv)
        for (uint32_t i = 0; i < nv; i += 4) {
            const uint4 o = *reinterpret_cast<const uint4*>(&order[i]);
            rank += (o.x < ordered ? 1u : 0u) + (o.y < ordered ? 1u : 0u) + (o.z < ordered ? 1u : 0u) + (o.w < ordered ? 1u : 0u);
        }
    __syncthreads();
    const uint64_t nnz = sum;
    const uint32_t shift = !shac && entries > nnz ? 1u : 0u, k = nv + shift;
    if (t >= k && t < K + 3) freq[t] = ~0u;
    if (t < nv) { freq[rank + shift] = cnt; key_of[rank + shift] = key; }
    if (t == 0 && shift) { freq[0] = (uint32_t)(entries - nnz); key_of[0] = 0u; }
    __syncthreads();
    if (t < k) {
        const uint32_t f = freq[t];
        uint32_t r = 0;
        for (uint32_t i = 0; i < k; i += 4) {                             // (past k: ~0, which no count reaches)
            const uint4 g = *reinterpret_cast<const uint4*>(&freq[i]);
            r += (g.x < f + (i < t ? 1u : 0u) ? 1u : 0u) + (g.y < f + (i + 1 < t ? 1u : 0u) ? 1u : 0u) +
                 (g.z < f + (i + 2 < t ? 1u : 0u) ? 1u : 0u) + (g.w < f + (i + 3 < t ? 1u : 0u) ? 1u : 0u);
        }
        leaf[r] = f; leaf_sym[r] = t;
    }
    if (t >= k) leaf[t] = ~0u;
    if (t == 0) sum = 0;
    __syncthreads();
    if (k >= kPairUp) {
        // thread t holds leaf t and node t, and the weights behind them
        uint32_t li = 0, ni = 0, wl = ~0u, wl_next = ~0u, wn = ~0u, wn_next = ~0u;
        if (t < k) { wl = leaf[t]; wl_next = leaf[t + 1]; }
        if (t == 0) upto[0][0] = upto[0][1] = 0;
        __syncthreads();
        for (uint32_t made = 0, turn = 0; made + 1 < k; ++turn) {
            const uint32_t l0 = leaf[li], l1 = leaf[li + 1], n0 = node[ni], n1 = node[ni + 1];
            const uint32_t s = l0 <= n0 ? l0 + (l1 <= n0 ? l1 : n0) : n0 + (l0 <= n1 ? l0 : n1);
            uint32_t (&n_upto)[2] = upto[turn & 1u];
            const bool in_l = t >= li && t < k && wl <= s, in_n = t >= ni && t < made && wn <= s;
            if (in_l && (t + 1 == k || wl_next > s)) n_upto[0] = t + 1 - li;
            if (in_n && (t + 1 == made || wn_next > s)) n_upto[1] = t + 1 - ni;
            if (t == 0) upto[~turn & 1u][0] = upto[~turn & 1u][1] = 0;
            __syncthreads();
            const uint32_t nl = n_upto[0], nn = n_upto[1], pairs = (nl + nn) / 2, odd = (nl + nn) & 1u;
            if (in_l) {
                const uint32_t at = t - li + count_below(node, ni, ni + nn, wl);
                merged[at] = wl;
                if (at < 2 * pairs) parent[t] = made + at / 2; else last_is_node = 0;
            }
            if (in_n) {
                const uint32_t at = t - ni + count_below(leaf, li, li + nl, wn + 1);
                merged[at] = wn;
                if (at < 2 * pairs) parent[K + t] = made + at / 2; else last_is_node = 1;
            }
            __syncthreads();
            const uint32_t stays = odd ? 1u + last_is_node : 0u;           // the last one, if it has no partner
            if (t + 1 >= made && t < made + pairs) {
                const uint32_t q = t + 1 - made;                           // pair of the node behind this thread's
                if (q) { wn = merged[2 * q - 2] + merged[2 * q - 1]; node[t] = wn; }
                wn_next = q < pairs ? merged[2 * q] + merged[2 * q + 1] : ~0u;
            }
            li += nl - (stays == 1 ? 1u : 0u);
            ni += nn - (stays == 2 ? 1u : 0u);
            made += pairs;
            __syncthreads();
        }
    } else if (t == 0) {
        uint32_t li = 0, ni = 0;
        for (uint32_t made = 0; made + 1 < k; ++made) {
            const uint32_t l0 = leaf[li], l1 = leaf[li + 1], n0 = node[ni], n1 = node[ni + 1];   // (~0 past the end)
            const bool a = l0 <= n0;                                       // the first is a leaf
            const uint32_t lx = a ? l1 : l0, nx = a ? n0 : n1;
            const bool b = lx <= nx;
            node[made] = (a ? l0 : n0) + (b ? lx : nx);
            parent[a ? li : K + ni] = made;
            li += a ? 1u : 0u; ni += a ? 0u : 1u;
            parent[b ? li : K + ni] = made;
            li += b ? 1u : 0u; ni += b ? 0u : 1u;
        }
    }
    __syncthreads();
    unsigned long long my_bits = 0;
    if (t < k) {
        uint32_t l = 1;
        if (k > 1)
            for (uint32_t p = parent[t]; p + 2 != k && l <= 32; p = parent[K + p]) ++l;
        if (l > 32) { bad = 1; l = 32; }
        len[leaf_sym[t]] = (uint8_t)l;
        atomicAdd(&count[l], 1u);
        my_bits = (unsigned long long)leaf[t] * l;
    }
    add_up(my_bits);
    __syncthreads();
    uint32_t lmax = 32;
    while (lmax && !count[lmax]) --lmax;
    if (t == 0) {
        uint64_t c = 0;
        uint32_t idx = 0;
        first_code[0] = first_index[0] = 0;
        for (uint32_t l = 1; l <= 32; ++l) {
            c <<= 1;
            first_code[l] = (uint32_t)c; first_index[l] = idx;
            c += count[l]; idx += count[l];
        }
    }
    uint32_t slots = 64;
    while (slots < 4 * nv && slots < kDevSlots) slots <<= 1;
    for (uint32_t i = t; i < slots; i += kCodeThreads) tkey[i] = 0;
    __syncthreads();
    // a symbol's place among those of its length: lanes below in the wavefront, then the wavefronts before
    const uint32_t my_len = t < k ? len[t] : 0u;
    uint32_t below = 0;
    for (uint32_t l = 1; l <= lmax; ++l) {
        const uint64_t same = __ballot(my_len == l);
        if (my_len == l) below = (uint32_t)__popcll(same & ((1ull << (t & 63u)) - 1u));
        if ((t & 63u) == 0) wave_count[t >> 6][l] = (uint32_t)__popcll(same);
    }
    __syncthreads();
    if (t < k) {
        const uint32_t l = my_len;
        uint32_t r = below;
        for (uint32_t w = 0; w < t >> 6; ++w) r += wave_count[w][l];
        codes[t] = first_code[l] + r;
        sort[first_index[l] + r] = t;
        if (t >= shift) {
            const uint32_t key2 = key_of[t];
            uint32_t s = mix32(key2) & (slots - 1);
            while (atomicCAS(&tkey[s], 0u, key2) != 0u) s = (s + 1) & (slots - 1);   // (half of the slots stay empty)
            tcode[s] = codes[t]; tlen[s] = l;
        }
    }
    __syncthreads();
    for (uint32_t i = t; i < slots; i += kCodeThreads) {
        const bool any = tkey[i] != 0u;
        table[i] = tkey[i]; table[slots + i] = any ? tcode[i] : 0u; table[2 * slots + i] = any ? tlen[i] : 0u;
    }
    const uint32_t T = lut_opt ? lut_opt : lmax < 1 ? 1u : lmax < 10 ? lmax : 10u;
    for (uint32_t e = t; e < (1u << T); e += kCodeThreads) {
        uint32_t v = 0;
        for (uint32_t l = 1; l <= T && l <= lmax; ++l) {
            const uint32_t r = (e >> (T - l)) - first_code[l];
            if (r < count[l]) { v = sort[first_index[l] + r] << 6 | l; break; }
        }
        out->lut[e] = v;
    }
    if (t < k) { out->codebook[t] = key_of[t]; out->symsort[t] = sort[t]; }
    if (t < (kDevSymbols + 4) / 4) {
        uint32_t w = 0;
        for (uint32_t i = 0; i < 4; ++i) if (4 * t + i < k) w |= (uint32_t)len[4 * t + i] << (8 * i);
        out->codelen[t] = w;
    }
    if (t < 33) { out->canon[t] = first_code[t]; out->canon[33 + t] = count[t]; out->canon[66 + t] = first_index[t]; }
    if (t == 0) {
        EncCode c = {};
        c.status = bad || nnz > 0xfffffff0ull || sum > 0xfffffff0ull ? kCodeRange : kCodeOk;
        c.values = nv; c.k_sym = k; c.lmax = lmax; c.lut_bits = T;
        c.has_zero = shift; c.zcode = shift ? codes[0] : 0u; c.zlen = shift ? len[0] : 0u; c.slots = slots;
        c.nnz = nnz; c.bits = sum;
        *code = c;
    }
}

// An alphabet for the host: the occupied slots of the histogram as a list of (key, count) in no particular order (the host sorts by
// value), by all threads of a grid.  flags[2] counts them; those past kListCap are dropped: more than 65536 values are refused.
// `near`: the first kBoxPairs of them once more, in pinned memory (or nullptr).
constexpr uint32_t kListCap = 65536 + 64;
constexpr uint32_t kBoxPairs = 4096;
struct PairList { uint32_t* list; uint32_t* near; };

__device__ __forceinline__ void list_pairs(const Histogram& h, const PairList& to)
{
    const uint32_t threads = gridDim.x * blockDim.x;
    for (uint32_t s0 = blockIdx.x * blockDim.x + threadIdx.x; s0 < kHashSlots; s0 += 16 * threads) {
        uint32_t keys[16];                             // requested together: a small matrix has few threads for its 131072 slots
#pragma unroll
        for (uint32_t u = 0; u < 16; ++u) { const uint64_t s = s0 + (uint64_t)u * threads; keys[u] = h.keys[s < kHashSlots ? s : kHashSlots - 1]; }
#pragma unroll
        for (uint32_t u = 0; u < 16; ++u) {
            const uint64_t s = s0 + (uint64_t)u * threads;
            if (!keys[u] || s >= kHashSlots) continue;
            const uint32_t i = atomicAdd(&h.flags[2], 1u), cnt = h.cnts[s];
            if (i < kListCap) { to.list[2 * (uint64_t)i] = keys[u]; to.list[2 * (uint64_t)i + 1] = cnt; }
            if (i < kBoxPairs && to.near) { to.near[2 * i] = keys[u]; to.near[2 * i + 1] = cnt; }
        }
    }
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

// the same without the codewords: bit patterns, then lengths
template <bool LDS_TABLE>
__device__ __forceinline__ const uint32_t* length_table(const Survivors& s, uint32_t* lds)
{
    if (!LDS_TABLE) return s.table;
    for (uint32_t i = threadIdx.x; i < 2 * s.slots; i += 256) lds[i] = s.table[i < s.slots ? i : i + s.slots];
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
struct SegWords {
    uint32_t* mask_; uint16_t* off_;
    __device__ __forceinline__ uint32_t& mask(uint32_t w) const { return mask_[256 * w + threadIdx.x]; }
    __device__ __forceinline__ uint16_t& off(uint32_t w) const { return off_[256 * w + threadIdx.x]; }
};
__host__ __device__ inline uint32_t seg_words_lds(uint32_t seg_rows) { return (seg_rows / 32) * (256 + 128); }   // in words of 32 bits
// a block's LDS: its segments' words, then the code table
__device__ __forceinline__ SegWords seg_words(uint32_t* lds, uint32_t seg_rows)
{
    return SegWords{ lds, reinterpret_cast<uint16_t*>(lds + (seg_rows / 32) * 256) };
}

__device__ __forceinline__ uint32_t load_segment(const Survivors& s, const SegWords& sw, uint32_t j, uint32_t r0, uint32_t r1)
{
    const uint32_t words = (r1 - r0 + 31) / 32;
    const uint64_t at = (uint64_t)(r0 / 32) * s.m + j;
    uint32_t total = 0;
    for (uint32_t w0 = 0; w0 < words; w0 += 8) {                      // eight words' loads in flight; past the end: the last word again
        uint32_t word[8], off[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            const uint64_t a = at + (uint64_t)(w0 + u < words ? w0 + u : words - 1) * s.m;
            word[u] = s.mask[a]; off[u] = s.off[a];
        }
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u)
            if (w0 + u < words) { sw.mask(w0 + u) = word[u]; sw.off(w0 + u) = (uint16_t)off[u]; total += __popc(word[u]); }
    }
    return total;
}

// f(row, bit pattern) for the segment's `total` non-zeros, in order.  The patterns of four are requested together: one trip to
// memory per non-zero was half of what the passes of steps 3 and 5 took.
template <class F>
__device__ __forceinline__ void for_survivors(const Survivors& s, const SegWords& sw, uint32_t j, uint32_t r0, uint32_t total, F f)
{
    uint32_t w = 0, word = sw.mask(0), at = sw.off(0);
    const uint32_t* list = s.values + ((uint64_t)(r0 / 32) * s.m + (j - j % kTileCols)) * kQuota;   // of the segment's first tile
    for (uint32_t i = 0; i < total; i += 4) {
        uint32_t r[4], key[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) {
            if (i + u < total) {
                while (word == 0) { ++w; word = sw.mask(w); at = sw.off(w); }
                r[u] = r0 + 32 * w + (uint32_t)__builtin_ctz(word);
                word &= word - 1;
                const uint32_t* from = at != kNotPacked ? list + (uint64_t)w * s.m * kQuota + at
                                                        : reinterpret_cast<const uint32_t*>(s.W) + (uint64_t)r[u] * s.ldw + j;
                at += at != kNotPacked ? 1u : 0u;
                key[u] = *from;
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u)
            if (i + u < total) f(r[u], key[u]);
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
// Where the code has to come from the host, its alphabet is listed instead.
template <bool LDS_TABLE>
__global__ void __launch_bounds__(256)
enc_bits_kernel(Survivors s, const EncCode* __restrict__ code, Histogram hist, PairList pairs, uint32_t* __restrict__ seg_nnz, uint32_t* __restrict__ seg_bits,
                uint32_t* __restrict__ gap_bits, unsigned long long* gap_total, uint64_t seg_cols)
{
    extern __shared__ uint32_t lds[];
    const SegWords sw = seg_words(lds, s.seg_rows);
    __shared__ unsigned long long sums[kRiceKMax + 1];
    const uint32_t seg = blockIdx.x / s.col_blocks, j = (blockIdx.x - seg * s.col_blocks) * 256 + threadIdx.x;
    const uint32_t r0 = seg * s.seg_rows, r1 = r0 + s.seg_rows < s.n ? r0 + s.seg_rows : s.n;
    const uint64_t at = (uint64_t)seg * s.m + j;
    const uint32_t total = j < s.m ? load_segment(s, sw, j, r0, r1) : 0u;      // (needs nothing of the code: on its way first)
    if (code->status != kCodeOk) {
        if (code->status == kCodeOnHost) list_pairs(hist, pairs);
        return;
    }
    const uint32_t zlen = code->zlen;
    s.slots = code->slots;
    if (threadIdx.x <= kRiceKMax) sums[threadIdx.x] = 0;
    const uint32_t* table = length_table<LDS_TABLE>(s, lds + seg_words_lds(s.seg_rows));
    const uint32_t* lengths = table + (LDS_TABLE ? 1u : 2u) * s.slots;
    uint32_t g[kRiceKMax + 1];
#pragma unroll
    for (uint32_t k = 0; k <= kRiceKMax; ++k) g[k] = 0;
    if (j < s.m) {
        uint32_t bits = 0;
        uint32_t next = gap_bits && total ? row_after_previous(s, j, r0) : 0u;   // the row the next gap counts from
        for_survivors(s, sw, j, r0, total, [&](uint32_t r, uint32_t key) {
            bits += lengths[slot_of(table, s.slots, key)];
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
    extern __shared__ uint32_t lds[];
    const SegWords sw = seg_words(lds, s.seg_rows);
    const uint32_t* table = code_table<LDS_TABLE>(s, lds + seg_words_lds(s.seg_rows));
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

// the parameter with the fewest gap bits, the smaller on ties (as on the host)
__device__ __forceinline__ uint32_t best_rice_k(const unsigned long long* __restrict__ gap_total)
{
    uint32_t best = 0;
#pragma unroll
    for (uint32_t k = 1; k <= kRiceKMax; ++k) if (gap_total[k] < gap_total[best]) best = k;
    return best;
}

// Step 3, second part: running sums over the segments of every column (in place: what stands above a
// segment in its column) and the column's totals.  16 columns x 16 ranges of segments per block: a tall
// and narrow matrix has hundreds of segments per column and few columns.
// gap_bits: all 16 parameters; the best one counts.
__global__ void __launch_bounds__(256)
enc_col_scan_kernel(const EncCode* __restrict__ code, uint32_t m, uint32_t S, uint32_t* __restrict__ seg_nnz, uint32_t* __restrict__ seg_bits,
                    const uint32_t* __restrict__ gap_bits, const unsigned long long* __restrict__ gap_total, uint64_t seg_cols,
                    uint32_t* __restrict__ col_nnz, unsigned long long* __restrict__ col_bits)
{
    __shared__ uint32_t part_nnz[16][17];
    __shared__ unsigned long long part_bits[16][17];
    const uint32_t c = threadIdx.x & 15, g = threadIdx.x >> 4, j = blockIdx.x * 16 + c;
    if (code->status != kCodeOk) return;
    if (gap_bits) gap_bits += best_rice_k(gap_total) * seg_cols;
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

// Step 4.  One block: the longest column gives the chunk size, then running sums over the columns, four neighbouring ones per thread and a
// strip of 4 blockDim.x at a time (few columns: fewer wavefronts, which wait for each other).  What bounds it is the chain of trips to memory, so a
// strip's columns are requested while the one before is added up; matrices of one strip are read once.  (A range of columns per thread
// instead, a line of memory for every column and lane: 64 x 500 000 3120 us for the whole call, 640 so; 64 x 4096 87 and 81.)
// col_arrays: first chunk, CSC position and first stream bit of every column and one past it, `stride` words apart; what lies behind a multiple of
// four past the last column is the sums once more.  The counts go to *result and, where the host waits for them in pinned memory, to *mailbox.
struct ColumnQuad { uint32_t nnz[4]; unsigned long long bits[4]; };

// (the arrays have room for whole quads; columns past m count as empty)
__device__ __forceinline__ ColumnQuad load_quad(const uint32_t* __restrict__ col_nnz, const unsigned long long* __restrict__ col_bits, uint32_t j, uint32_t m)
{
    ColumnQuad q = {};
    if (j >= m) return q;
    const uint4 c = *reinterpret_cast<const uint4*>(col_nnz + j);
    const ulonglong2 b0 = *reinterpret_cast<const ulonglong2*>(col_bits + j), b1 = *reinterpret_cast<const ulonglong2*>(col_bits + j + 2);
    const uint32_t left = m - j;
    q.nnz[0] = c.x; q.nnz[1] = left > 1 ? c.y : 0u; q.nnz[2] = left > 2 ? c.z : 0u; q.nnz[3] = left > 3 ? c.w : 0u;
    q.bits[0] = b0.x; q.bits[1] = left > 1 ? b0.y : 0ull; q.bits[2] = left > 2 ? b1.x : 0ull; q.bits[3] = left > 3 ? b1.y : 0ull;
    return q;
}

__global__ void __launch_bounds__(1024)
enc_columns_kernel(const EncCode* __restrict__ code, uint32_t m, const uint32_t* __restrict__ col_nnz, const unsigned long long* __restrict__ col_bits,
                   const uint32_t* __restrict__ flags, uint32_t chunk_opt, const unsigned long long* __restrict__ gap_total, uint32_t* __restrict__ col_arrays, uint64_t stride,
                   EncResult* __restrict__ result, EncResult* mailbox)
{
    __shared__ unsigned long long wave_bits[2][16];
    __shared__ uint32_t wave_nnz[2][16], wave_chunks[2][16];
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6, waves = blockDim.x / 64, strip = 4 * blockDim.x;
    const uint32_t status = code->status;
    uint32_t most = 0, chunk = 0, k = 0;
    unsigned long long longest = 0, all_nnz = 0, all_chunks = 0, all_bits = 0, gap_bits = 0;
    if (status == kCodeOk) {                                                // (uniform)
        const ColumnQuad first = load_quad(col_nnz, col_bits, 4 * t, m);
        ColumnQuad q = first;
        for (uint64_t j0 = 0; j0 < m; j0 += strip) {
            const uint64_t next = j0 + strip + 4 * t;
            const ColumnQuad ahead = load_quad(col_nnz, col_bits, next < m ? (uint32_t)next : m, m);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                most = q.nnz[u] > most ? q.nnz[u] : most;
                longest = q.bits[u] > longest ? q.bits[u] : longest;
            }
            q = ahead;
        }
        for (int d = 32; d >= 1; d >>= 1) {
            const uint32_t o = __shfl_xor(most, d, 64);
            const unsigned long long p = __shfl_xor(longest, d, 64);
            most = o > most ? o : most; longest = p > longest ? p : longest;
        }
        if (lane == 0) { wave_nnz[1][wave] = most; wave_bits[1][wave] = longest; }
        __syncthreads();
        for (uint32_t w = 0; w < waves; ++w) {
            most = wave_nnz[1][w] > most ? wave_nnz[1][w] : most; longest = wave_bits[1][w] > longest ? wave_bits[1][w] : longest;
        }
        chunk = hac_internal::chunk_for(chunk_opt, most);
        q = first;
        uint32_t side = 0;                                                  // of the wavefronts' sums: one barrier a strip
        for (uint64_t j0 = 0; j0 < m; j0 += strip, side ^= 1u) {
            const uint64_t j = j0 + 4 * t, next = j + strip;
            const ColumnQuad ahead = load_quad(col_nnz, col_bits, next < m ? (uint32_t)next : m, m);
            uint32_t chunks[4], nnz = 0, ch = 0;
            unsigned long long bits = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t cj = hac_internal::chunk_of_column(chunk, q.nnz[u]);
                chunks[u] = (q.nnz[u] + cj - 1) / cj;
                nnz += q.nnz[u]; ch += chunks[u]; bits += q.bits[u];
            }
            // this thread's place among all: sums of the threads before it in its wavefront, and of the wavefronts before
            uint32_t in = nnz, ic = ch;
            unsigned long long ib = bits;
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t a = __shfl_up(in, d, 64), b = __shfl_up(ic, d, 64);
                const unsigned long long c = __shfl_up(ib, d, 64);
                if ((int)lane >= d) { in += a; ic += b; ib += c; }
            }
            if (lane == 63) { wave_nnz[side][wave] = in; wave_chunks[side][wave] = ic; wave_bits[side][wave] = ib; }
            __syncthreads();
            unsigned long long pos = all_nnz + in - nnz, at = all_chunks + ic - ch, bit = all_bits + ib - bits;
            for (uint32_t w = 0; w < waves; ++w) {
                const uint32_t wn = wave_nnz[side][w], wc = wave_chunks[side][w];
                const unsigned long long wb = wave_bits[side][w];
                if (w < wave) { pos += wn; at += wc; bit += wb; }
                all_nnz += wn; all_chunks += wc; all_bits += wb;
            }
            if (j < m) {
                uint32_t o[3][4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    o[0][u] = (uint32_t)at; o[1][u] = (uint32_t)pos; o[2][u] = (uint32_t)bit;
                    at += chunks[u]; pos += q.nnz[u]; bit += q.bits[u];
                }
#pragma unroll
                for (int s = 0; s < 3; ++s) *reinterpret_cast<uint4*>(col_arrays + s * stride + j) = make_uint4(o[s][0], o[s][1], o[s][2], o[s][3]);
            }
            q = ahead;
        }
        if (gap_total) { k = best_rice_k(gap_total); gap_bits = gap_total[k]; }
    }
    if (t != 0) return;
    if (status == kCodeOk) { col_arrays[m] = (uint32_t)all_chunks; col_arrays[stride + m] = (uint32_t)all_nnz; col_arrays[2 * stride + m] = (uint32_t)all_bits; }
    for (EncResult* r : { result, mailbox }) {
        if (!r) continue;
        r->code = *code;
        if (status == kCodeOnHost) r->code.values = flags[2];
        r->chunk = chunk; r->rice_k = k;
        r->max_col_nnz = most; r->max_col_bits = longest;
        r->col_bits = all_bits; r->col_nnz = all_nnz; r->chunks = all_chunks; r->gap_bits = gap_bits;
    }
}

// Step 5, first part: the blob as the codewords find it.  `tables`: step 2's (nullptr: the host copies header and tables itself).
__global__ void __launch_bounds__(256)
enc_head_kernel(hac_desc_t d, const DevTables* __restrict__ tables, const uint32_t* __restrict__ col_arrays, uint32_t* __restrict__ blob)
{
    const uint64_t i0 = blockIdx.x * 256 + threadIdx.x, step = (uint64_t)gridDim.x * 256;
    const uint64_t cols = d.off_col_chunk / 4, ents = d.off_chunk_ent / 4, stride = (d.off_col_pos - d.off_col_chunk) / 4;
    if (tables) {
        auto section = [&](uint64_t off, uint64_t end, const uint32_t* from, uint32_t words) {   // the words of one, zeros behind them
            for (uint64_t i = i0; i < (end - off) / 4; i += step) blob[off / 4 + i] = i < words ? from[i] : 0u;
        };
        section(0, d.off_codebook, reinterpret_cast<const uint32_t*>(&d), (uint32_t)sizeof(hac_desc_t) / 4);
        section(d.off_codebook, d.off_codelen, tables->codebook, d.k_sym);
        section(d.off_codelen, d.off_canon, tables->codelen, (d.k_sym + 3) / 4);
        section(d.off_canon, d.off_symsort, tables->canon, 99);
        section(d.off_symsort, d.off_lut, tables->symsort, d.k_sym);
        section(d.off_lut, d.off_stream, tables->lut, 1u << d.lut_bits);
    }
    for (uint64_t i = i0; i < ents - cols; i += step) blob[cols + i] = i % stride <= d.m ? col_arrays[i] : 0u;   // (three of them, laid out alike)
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
    uint4* b4 = reinterpret_cast<uint4*>(blob);
    for (uint64_t i = d.off_stream / 16 + i0; i < cols / 4; i += step) b4[i] = zero;
    for (uint64_t i = ents / 4 + i0; i < d.blob_bytes / 16; i += step) b4[i] = zero;
}

struct WsLayout {
    size_t keys, cnts, flags, used, list, mask, off, values, seg_nnz, seg_bits, gap_bits, table, col_bits, col_nnz, code, result, tables, col_arrays, total;
    size_t col_stride;                                               // words from one of the column arrays to the next, as in a blob
};

WsLayout ws_layout(uint64_t n, uint64_t m)
{
    const uint64_t seg_rows = seg_rows_for(n, m), S = (n + seg_rows - 1) / seg_rows;
    const uint64_t words = (n + 31) / 32;
    WsLayout L;
    size_t c = 0;
    auto take = [&](size_t bytes) { const size_t o = c; c = (c + bytes + 255) / 256 * 256; return o; };
    L.keys = take(4ull * kHashSlots); L.cnts = take(4ull * kHashSlots); L.flags = take(256);
    L.used = take(4ull * kDevSymbols);
    L.list = take(8ull * kListCap);
    L.mask = take(4 * words * m); L.off = take(2 * words * m); L.values = take(4ull * kQuota * words * m);
    L.seg_nnz = take(4 * S * m); L.seg_bits = take(4 * S * m);
    L.gap_bits = take(4 * S * m * (kRiceKMax + 1));                  // used with Rice-coded gaps only
    L.table = take(12ull * kHashSlots);
    L.col_bits = take(8 * m); L.col_nnz = take(4 * m);
    L.code = take(sizeof(EncCode)); L.result = take(sizeof(EncResult)); L.tables = take(sizeof(DevTables));
    L.col_stride = (4 * ((size_t)m + 1) + 255) / 256 * 256 / 4;
    L.col_arrays = take(12 * L.col_stride);
    L.total = c;
    return L;
}

int hip_fail(hipError_t e) { hac_internal::set_last_hip_error((int)e); return HAC_EHIP; }

// Pinned memory that the device leaves a call's counts in, and a list of up to kBoxPairs values: kBoxes of them for the process (512 KB),
// allocated with the first call (one costs more than the call) and lent to a call until it has read them.  get() is nullptr where
// none is free, or none can be had: what the host needs is then copied.  From sent() on kernels of the call's stream may write to the box: it
// goes back only once the stream has been waited for, by the call (arrived()) or, where an error ended that early, by the destructor, and never if that
// wait fails.
constexpr int kBoxes = 16;
struct Box { EncResult result; uint32_t pairs[2 * kBoxPairs]; };
class Mailbox {
    struct Pool { std::mutex lock; Box* base = nullptr; bool asked = false; uint32_t taken = 0; };
    static Pool& pool() { static Pool* p = new Pool; return *p; }   // (never taken down: a call may run while the process ends)
    int i = -1;
    Box* p = nullptr;
    hipStream_t stream;
    bool written = false;                              // or about to be
public:
    explicit Mailbox(hipStream_t s) : stream(s)
    {
        Pool& q = pool();
        std::lock_guard<std::mutex> hold(q.lock);
        if (!q.asked) {
            q.asked = true;
            void* mem = nullptr;
            if (hipHostMalloc(&mem, sizeof(Box) * kBoxes, hipHostMallocPortable) == hipSuccess) q.base = static_cast<Box*>(mem);
            else (void)hipGetLastError();
        }
        if (!q.base) return;
        for (int k = 0; k < kBoxes && i < 0; ++k) if (!(q.taken >> k & 1u)) i = k;
        if (i >= 0) { q.taken |= 1u << i; p = q.base + i; }
    }
    ~Mailbox()
    {
        if (i < 0 || (written && hipStreamSynchronize(stream) != hipSuccess)) return;
        Pool& q = pool();
        std::lock_guard<std::mutex> hold(q.lock);
        q.taken &= ~(1u << i);
    }
    Mailbox(const Mailbox&) = delete;
    Mailbox& operator=(const Mailbox&) = delete;
    Box* get() const { return p; }
    void sent() { written = true; }
    void arrived() { written = false; }
};

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
    const Histogram hist = { dptr(L.keys), dptr(L.cnts), dptr(L.used), dptr(L.flags) };   // (gap totals 64 bytes behind the flags, zeroed with them)
    unsigned long long* d_gap_total = rice ? reinterpret_cast<unsigned long long*>(ws + L.flags + 64) : static_cast<unsigned long long*>(nullptr);
    uint32_t* d_gap_bits = rice ? dptr(L.gap_bits) : static_cast<uint32_t*>(nullptr);
    unsigned long long* d_col_bits = reinterpret_cast<unsigned long long*>(ws + L.col_bits);
    EncCode* d_code = reinterpret_cast<EncCode*>(ws + L.code);
    EncResult* d_result = reinterpret_cast<EncResult*>(ws + L.result);
    DevTables* d_tables = reinterpret_cast<DevTables*>(ws + L.tables);
    const size_t words_lds = 4 * (size_t)seg_words_lds(seg_rows);
    // (code tables up to kCodeSlotsLds are read from LDS)
    auto table_bytes = [](uint32_t slots) { return slots <= kCodeSlotsLds ? 12 * (size_t)slots : (size_t)0; };
    hipError_t e;
    // steps 3 and 4 with a code of at most `slots` slots, and the wait for their sums
    std::vector<uint32_t> list;                        // of a code that the host has to build
    auto sums = [&](uint32_t slots, EncResult& r) -> hipError_t {
        Mailbox mail(stream);
        Box* const box = mail.get();
        mail.sent();
        const PairList to = { dptr(L.list), box ? box->pairs : nullptr };
        const size_t lds = table_bytes(slots) / 3 * 2;
        hipLaunchKernelGGL(lds ? enc_bits_kernel<true> : enc_bits_kernel<false>, seg_grid, dim3(256), words_lds + lds, stream, sv, d_code, hist, to,
                           dptr(L.seg_nnz), dptr(L.seg_bits), d_gap_bits, d_gap_total, SM);
        hipLaunchKernelGGL(enc_col_scan_kernel, dim3((uint32_t)(((uint64_t)m + 15) / 16)), dim3(256), 0, stream, d_code, (uint32_t)m, S,
                           dptr(L.seg_nnz), dptr(L.seg_bits), static_cast<const uint32_t*>(d_gap_bits),
                           static_cast<const unsigned long long*>(d_gap_total), SM, dptr(L.col_nnz), d_col_bits);
        hipLaunchKernelGGL(enc_columns_kernel, dim3(1), dim3(m <= 1024 ? 256 : 1024), 0, stream, d_code, (uint32_t)m, dptr(L.col_nnz), d_col_bits,
                           dptr(L.flags), opts ? opts->chunk_nnz : 0u, static_cast<const unsigned long long*>(d_gap_total), dptr(L.col_arrays),
                           (uint64_t)L.col_stride, d_result, box ? &box->result : nullptr);
        hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
        if (!box && (err = hipMemcpyAsync(&r, d_result, sizeof r, hipMemcpyDeviceToHost, stream)) != hipSuccess) return err;
        if ((err = hipStreamSynchronize(stream)) != hipSuccess) return err;
        mail.arrived();
        if (box) r = box->result;
        if (r.code.status != kCodeOnHost || r.code.values > 65536) return hipSuccess;
        list.resize(2 * (size_t)r.code.values);
        if (box && r.code.values <= kBoxPairs) std::memcpy(list.data(), box->pairs, 4 * list.size());
        else if ((err = hipMemcpyAsync(list.data(), to.list, 4 * list.size(), hipMemcpyDeviceToHost, stream)) == hipSuccess) err = hipStreamSynchronize(stream);
        return err;
    };
    try {
        // ---- steps 1 to 4 ----
        hipLaunchKernelGGL(fill_zero_kernel, dim3(512), dim3(256), 0, stream, dptr(L.keys), (uint64_t)(L.used - L.keys) / 4);
        const bool once = (uint64_t)n * (uint64_t)m > kCachedEntries;
        const uint64_t scan_blocks = std::min<uint64_t>((tiles + kScanWaves - 1) / kScanWaves, once ? 2 * kScanBlocks : kScanBlocks);
        hipLaunchKernelGGL(once ? enc_scan_kernel<true> : enc_scan_kernel<false>, dim3((uint32_t)scan_blocks), dim3(64 * kScanWaves), 0, stream, d_W, (uint32_t)n, (uint32_t)m,
                           (uint64_t)ldw, col_groups, (uint32_t)tiles, dptr(L.mask), reinterpret_cast<uint16_t*>(ws + L.off),
                           dptr(L.values), hist);
        hipLaunchKernelGGL(enc_code_kernel, dim3(1), dim3(kCodeThreads), 0, stream, hist, (uint64_t)n * (uint64_t)m, shac ? 1u : 0u,
                           opts ? opts->lut_bits : 0u, dptr(L.table), d_tables, d_code);
        EncResult r;
        if ((e = sums(kDevSlots, r)) != hipSuccess) return hip_fail(e);
        if (r.code.status == kCodeNonFinite) return HAC_EINVAL;
        if (r.code.status == kCodeRange) return HAC_ERANGE;

        // ---- step 2 for a large alphabet ----
        const bool on_host = r.code.status == kCodeOnHost;
        std::vector<float> codebook;
        std::vector<uint8_t> len;
        std::vector<uint32_t> lut, table;
        CodeTables t;
        EncCode c = {};
        if (on_host) {
            const uint32_t nv = r.code.values;
            if (nv > 65536) return HAC_ERANGE;
            struct Val { float v; uint32_t key; uint64_t f; };
            std::vector<Val> vals(nv);
            for (uint32_t i = 0; i < nv; ++i) {
                vals[i].key = list[2 * (size_t)i]; vals[i].f = list[2 * (size_t)i + 1];
                std::memcpy(&vals[i].v, &vals[i].key, 4);
                c.nnz += vals[i].f;
            }
            if (c.nnz > 0xfffffff0ull) return HAC_ERANGE;
            std::sort(vals.begin(), vals.end(), [](const Val& a, const Val& b) { return a.v < b.v; });
            const uint64_t zeros = (uint64_t)n * (uint64_t)m - c.nnz;
            c.has_zero = !shac && zeros > 0 ? 1u : 0u;
            std::vector<uint64_t> freq;
            if (c.has_zero) { codebook.push_back(0.0f); freq.push_back(zeros); }
            for (const Val& x : vals) { codebook.push_back(x.v); freq.push_back(x.f); }
            if (!huffman_lengths(freq, len, c.lmax)) return HAC_ERANGE;
            canonical_codes(len, t);
            for (size_t i = 0; i < freq.size(); ++i) c.bits += freq[i] * len[i];
            if (c.bits > 0xfffffff0ull) return HAC_ERANGE;
            c.k_sym = (uint32_t)codebook.size(); c.lut_bits = pick_lut_bits(opts, c.lmax);
            build_lut(len, t, c.lut_bits, lut);
            c.zlen = c.has_zero ? len[0] : 0; c.zcode = c.has_zero ? t.code[0] : 0;
            c.status = kCodeOk; c.values = nv;
            // bit pattern -> codeword, at most a quarter full (half for the largest alphabets)
            c.slots = 64;
            while (c.slots < 4 * (uint64_t)nv && c.slots < kHashSlots) c.slots <<= 1;
            table.assign(3 * (size_t)c.slots, 0);
            for (size_t i = 0; i < vals.size(); ++i) {
                uint32_t h = mix32(vals[i].key) & (c.slots - 1);
                while (table[h]) h = (h + 1) & (c.slots - 1);
                table[h] = vals[i].key; table[c.slots + h] = t.code[i + c.has_zero]; table[2 * (size_t)c.slots + h] = len[i + c.has_zero];
            }
            if ((e = hipMemcpyAsync(dptr(L.table), table.data(), 4 * table.size(), hipMemcpyHostToDevice, stream)) != hipSuccess) return hip_fail(e);
            if ((e = hipMemcpyAsync(d_code, &c, sizeof c, hipMemcpyHostToDevice, stream)) != hipSuccess) return hip_fail(e);
            if ((e = sums(c.slots, r)) != hipSuccess) return hip_fail(e);
        }
        c = r.code;
        sv.slots = c.slots;
        const uint64_t total_bits = c.bits + r.gap_bits, nnz = c.nnz;
        if (total_bits > 0xfffffff0ull) return HAC_ERANGE;
        if (r.col_bits != total_bits || r.col_nnz != nnz) return HAC_EFORMAT;
        if (r.chunks > 0xfffffff0ull) return HAC_ERANGE;

        hac_desc_t d;
        std::memset(&d, 0, sizeof d);
        d.magic = kMagic; d.version = kVersion; d.format = format; d.header_bytes = 256;
        d.n = (uint64_t)n; d.m = (uint64_t)m; d.nnz = nnz; d.total_bits = total_bits; d.n_words = (total_bits + 31) / 32;
        d.k_sym = c.k_sym; d.lmax = c.lmax; d.lut_bits = c.lut_bits;
        d.chunk = r.chunk; d.n_chunks = r.chunks; d.max_col_bits = r.max_col_bits; d.max_col_nnz = r.max_col_nnz;
        if (rice) {
            const uint32_t brel_bits = std::max<uint32_t>(ceil_log2(r.max_col_bits + 1), 1);
            d.ent_bits = need_bits + brel_bits <= 32 ? 32 : 64;
            d.row_bits = d.ent_bits == 32 ? need_bits : 0;
            d.ri_coding = HAC_RI_RICE; d.rice_k = r.rice_k; d.gap_bits = r.gap_bits;
        } else if (shac) {
            d.ri_bits = ri_bits;
            d.ent_bits = r.max_col_bits < 65536 ? 16 : 32;
            if (nnz * (uint64_t)ri_bits > 0xfffffff0ull * 32ull) return HAC_ERANGE;
        } else {
            d.has_zero = c.has_zero;
            d.zero_len = (c.has_zero && c.zcode == 0) ? c.zlen : 0;
            const uint32_t brel_bits = std::max<uint32_t>(ceil_log2(r.max_col_bits + 1), 1);
            d.ent_bits = need_bits + brel_bits <= 32 ? 32 : 64;
            d.row_bits = d.ent_bits == 32 ? need_bits : 0;
        }
        place_sections(d);
        *desc = d;
        void* d_blob = place((size_t)d.blob_bytes);
        if (!d_blob) return HAC_EWORKSPACE;                                         // desc->blob_bytes says how much
        if (reinterpret_cast<uintptr_t>(d_blob) % 256) return HAC_EINVAL;
        if (d.off_col_pos - d.off_col_chunk != 4 * L.col_stride || d.off_chunk_ent - d.off_col_chunk != 12 * L.col_stride) return HAC_EFORMAT;

        // ---- step 5 ----
        uint8_t* blob = static_cast<uint8_t*>(d_blob);
        hipLaunchKernelGGL(enc_head_kernel, dim3(1024), dim3(256), 0, stream, d, static_cast<const DevTables*>(on_host ? nullptr : d_tables),
                           static_cast<const uint32_t*>(dptr(L.col_arrays)), reinterpret_cast<uint32_t*>(blob));
        std::vector<uint8_t> blob_head;
        if (on_host) {
            blob_head.assign((size_t)d.off_stream, 0);
            std::memcpy(blob_head.data(), &d, sizeof d);
            write_tables(blob_head.data(), d, codebook, len, t, lut);
            if ((e = hipMemcpyAsync(blob, blob_head.data(), blob_head.size(), hipMemcpyHostToDevice, stream)) != hipSuccess) return hip_fail(e);
        }
        EmitArgs a;
        a.seg_bit0 = dptr(L.seg_bits); a.seg_pos0 = dptr(L.seg_nnz);
        a.col_bit = reinterpret_cast<const uint32_t*>(blob + d.off_col_bit);
        a.col_pos = reinterpret_cast<const uint32_t*>(blob + d.off_col_pos);
        a.col_chunk = reinterpret_cast<const uint32_t*>(blob + d.off_col_chunk);
        a.stream = reinterpret_cast<uint32_t*>(blob + d.off_stream);
        a.ent = blob + d.off_chunk_ent;
        a.ri = (shac && !rice) ? reinterpret_cast<uint32_t*>(blob + d.off_ri) : nullptr;
        a.rice = rice ? 1u : 0u; a.rice_k = r.rice_k;
        a.shac = shac ? 1u : 0u; a.zcode = c.zcode; a.zlen = c.zlen;
        a.chunk = r.chunk; a.ent_bits = d.ent_bits; a.row_bits = d.row_bits; a.ri_bits = ri_bits;
        const size_t lds = table_bytes(c.slots);
        hipLaunchKernelGGL(lds ? enc_emit_kernel<true> : enc_emit_kernel<false>, seg_grid, dim3(256), words_lds + lds, stream, sv, a);
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
