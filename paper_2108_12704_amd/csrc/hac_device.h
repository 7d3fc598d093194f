// Decode primitives of libhac's kernels (gfx950): the blob as the device sees it, word sources
// (global memory or a copy staged in LDS), the decode tables in LDS, one codeword, and one lane's
// walk through a chunk of a HAC stream (arXiv 2108.12704 Sect. IV-B), an sHAC stream (Sect. IV-C)
// or an sHAC stream with Rice-coded row gaps.  Included by hac_kernels.hip only.
#ifndef HAC_DEVICE_H
#define HAC_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

constexpr int kWave = 64;
constexpr uint32_t kCodebookLdsMax = 1024;   // symbols whose values are staged in LDS

typedef __attribute__((address_space(3))) const uint32_t lds_cu32;
typedef __attribute__((address_space(3))) const float lds_cf32;

struct DevBlob {
    const float* codebook;
    const uint32_t* canon;      // first_code[33], count[33], first_index[33]
    const uint32_t* symsort;
    const uint32_t* lut;
    const uint32_t* stream;
    const uint32_t* colchunk;   // m + 1
    const uint32_t* colpos;     // m + 1 (sHAC: cb)
    const uint32_t* colbit;     // m + 1
    const void* ent;            // chunk entries
    const uint32_t* ri;         // sHAC
    uint32_t n, m, nnz, k_sym, lmax, lut_bits, has_zero, zero_len, chunk, ri_bits, ent_bits, row_bits, n_chunks;
    uint32_t rice, rice_k;      // sHAC whose row gaps are Rice-coded in front of each value's codeword
};

// (relative bit offset, first row) of chunk g
// request_entry only loads; entry_fields takes the loaded bits apart.  A kernel that has other
// loads to issue calls the two apart, so that no wait sits between its loads.
__device__ __forceinline__ uint2 request_entry(const DevBlob& d, uint32_t g)
{
    uint2 raw = make_uint2(0u, 0u);
    if (d.ent_bits == 32) raw.x = static_cast<const uint32_t*>(d.ent)[g];
    else if (d.ent_bits == 16) raw.x = static_cast<const uint16_t*>(d.ent)[g];
    else raw = static_cast<const uint2*>(d.ent)[g];
    return raw;
}

__device__ __forceinline__ void entry_fields(const DevBlob& d, const uint2& raw, uint32_t& rel, uint32_t& row)
{
    if (d.ent_bits == 32) {
        rel = raw.x >> d.row_bits;                   // sHAC: row_bits = 0
        row = raw.x & ((1u << d.row_bits) - 1u);
    } else if (d.ent_bits == 16) {
        rel = raw.x; row = 0;
    } else {
        row = raw.x; rel = raw.y;
    }
}

__device__ __forceinline__ void load_entry(const DevBlob& d, uint32_t g, uint32_t& rel, uint32_t& row)
{
    entry_fields(d, request_entry(d, g), rel, row);
}

// ---------------------------------------------------------------------------
// word sources: the blob's stream / ri words in global memory, or a copy staged
// in LDS that starts at word `wbase`
// ---------------------------------------------------------------------------
template <bool LDS, bool INLINE = true>           // INLINE: see decode_symbol
struct WordSrc {
    static constexpr bool kInline = INLINE;
    const uint32_t* w;
    uint32_t wbase;
    __device__ __forceinline__ uint32_t word(uint32_t i) const {
        if (LDS) return ((lds_cu32*)w)[i - wbase];
        return w[i];
    }
    // bits [bp, bp + 32), left-aligned
    __device__ __forceinline__ uint32_t peek32(uint32_t bp) const {
        const uint32_t wi = bp >> 5, off = bp & 31;
        const uint32_t w0 = word(wi), w1 = word(wi + 1);
        return off ? __builtin_amdgcn_alignbit(w0, w1, 32 - off) : w0;
    }
    // a `bits`-wide field (1..32) that starts at bit position bp
    __device__ __forceinline__ uint32_t field(uint64_t bp, uint32_t bits) const {
        const uint32_t wi = (uint32_t)(bp >> 5), off = (uint32_t)(bp & 31);
        const uint32_t w0 = word(wi), w1 = word(wi + 1);
        const uint32_t top = off ? __builtin_amdgcn_alignbit(w0, w1, 32 - off) : w0;
        return top >> (32 - bits);
    }
    // The staged copy only.  Bits [rel, rel + 32) with rel counted from the copy's first word and
    // handed over as rel - 1: the pair of words is then taken one word early when rel is a multiple
    // of 32, the funnel shift (which takes its amount modulo 32) by -rel = ~(rel - 1) is right in
    // every case, and nothing is selected.  At rel == 0 the word in front of the copy is read and
    // not used: every kernel keeps its tables (or other staged words) there.
    __device__ __forceinline__ uint32_t peek32_rm1(int32_t rm1) const {
        static_assert(LDS, "positions relative to the staged copy");
        lds_cu32* sw = (lds_cu32*)w;
        const int32_t q = rm1 >> 5;
        return __builtin_amdgcn_alignbit(sw[q], sw[q + 1], ~(uint32_t)rm1);
    }
    __device__ __forceinline__ uint32_t field_rel(uint32_t rel, uint32_t bits) const {
        return peek32_rm1((int32_t)rel - 1) >> (32 - bits);
    }
};

// Decode tables of one block in LDS.  Layout (uint32 words):
//   lut2[2^lut_bits][2] | bound[40] base[40] (+20 pad) | long2[k4][2]     k4 = k_sym rounded up to 4
// lut2 pairs the blob's first-level entry with the shared value of its symbol, so a short
// codeword costs one 64-bit LDS read.  A longer one is found by its length: bound[l], half of the first
// 32 bits that belong to codewords longer than l, base[l], what its first l bits have to be moved by to
// give its place in (length, symbol) order, and long2, symbol and value by that place.  long2 sits in LDS only when
// k_sym <= kCodebookLdsMax; otherwise symbols and values are read from the blob.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const u32x2 lds_cu2;

constexpr uint32_t kBounds = 40;             // entries of bound and base: lengths to 32, read four at a time

struct Tables {
    const uint2* lut2;          // LDS
    const uint32_t* bound;      // LDS; base behind it
    const uint2* long2;         // LDS when small
    bool small;                 // k_sym <= kCodebookLdsMax (uniform)
};

// codewords longer than the first-level table (none without symbols, whatever the rest of the header says)
__device__ __forceinline__ bool longer_codes(const DevBlob& d) { return d.lmax > d.lut_bits && d.k_sym != 0; }

// Code longer than the first-level table: {(symbol << 6) | length, value bits}.  Its length is the number of bounds it has passed,
// four of them read at once (all lanes the same words), then two reads.  Some lane of a wavefront is here at almost every step of a HAC
// stream: one length after the other, two reads each, made that lane's search the longest part of the step.
__device__ __forceinline__ uint2 decode_long(const Tables& t, const uint32_t* symsort, const float* codebook, uint32_t lut_bits, uint32_t lmax,
                                             uint32_t k_sym, uint32_t top)
{
    if (lmax <= lut_bits || !k_sym) return make_uint2(lmax ? lmax : 1u, 0u);    // no such code: a damaged stream; still makes progress
    lds_cu32* bound = (lds_cu32*)t.bound;
    const uint32_t half = top >> 1;
    uint32_t l = lut_bits + 1;
    for (uint32_t u = lut_bits + 1; u < lmax; u += 4) {                         // (from lmax on no bound is passed)
        const uint32_t b0 = bound[u], b1 = bound[u + 1], b2 = bound[u + 2], b3 = bound[u + 3];
        l += (half >= b0 ? 1u : 0u) + (half >= b1 ? 1u : 0u) + (half >= b2 ? 1u : 0u) + (half >= b3 ? 1u : 0u);
    }
    uint32_t at = bound[kBounds + l] + (top >> (32 - l));
    at = at < k_sym ? at : k_sym - 1u;                                          // (of a damaged stream)
    if (t.small) {
        const u32x2 e = ((lds_cu2*)t.long2)[at];
        return make_uint2(e.x << 6 | l, e.y);
    }
    const uint32_t sy = symsort[at];
    return make_uint2(sy << 6 | l, __float_as_uint(codebook[sy]));
}

__device__ __noinline__ uint2 call_decode_long(const uint32_t* bound, const uint2* long2, const uint32_t* symsort, const float* codebook, uint32_t lut_bits,
                                               uint32_t lmax, uint32_t k_sym, uint32_t top)
{
    const Tables t = { nullptr, bound, long2, k_sym <= kCodebookLdsMax };
    return decode_long(t, symsort, codebook, lut_bits, lmax, k_sym, top);
}

struct Decoded { uint32_t sym, len; float val; };

// INLINE: everywhere but where a loop waits for a word of the blob and stores several values per codeword (hac_decode_dev): the call is quicker there, with
// and without long codewords (7272 x 22, 25 % non-zero, sHAC 38.9 -> 33.6 us; 18037 x 12, 36 %, Rice-coded gaps 136 -> 127).
template <bool INLINE>
__device__ __forceinline__ Decoded decode_symbol(const DevBlob& d, const Tables& t, uint32_t top)
{
    const u32x2 raw = ((lds_cu2*)t.lut2)[top >> (32 - d.lut_bits)];
    uint2 e = make_uint2(raw.x, raw.y);
    if ((e.x & 63u) == 0) {
        if (INLINE) e = decode_long(t, d.symsort, d.codebook, d.lut_bits, d.lmax, d.k_sym, top);
        else e = call_decode_long(t.bound, t.long2, d.symsort, d.codebook, d.lut_bits, d.lmax, d.k_sym, top);
    }
    Decoded r;
    r.len = e.x & 63u; r.sym = e.x >> 6; r.val = __uint_as_float(e.y);
    return r;
}

__device__ __forceinline__ uint32_t table_words_dev(const DevBlob& d)
{
    const uint32_t k4 = (d.k_sym + 3u) & ~3u;
    return ((2u << d.lut_bits) + 100u + (d.k_sym <= kCodebookLdsMax ? 2u * k4 : 0u) + 3u) & ~3u;
}

// All threads of the block copy the tables; the caller synchronises afterwards.
//
// The copy is split in three so that every trip to memory carries as many loads as possible and a
// kernel can put its own loads beside them: request_tables issues everything that depends on
// nothing (first-level entries and, where codewords are longer than those, canonical table and symbol
// order), request_table_values the shared values of the entries and of the symbols in that order, store_tables writes LDS.
// A loop of load / store pairs would pay one trip per turn and per table instead.  Loads of the
// first kTabTurns turns of every loop are issued from clamped, valid indices on every thread;
// what a small block or a long table leaves over is copied the plain way.
constexpr int kTabTurns = 4;                        // (the asm statement in store_tables names four values)
struct TableRegs { uint32_t e[kTabTurns], v[kTabTurns]; uint32_t first, count, index, cb, sort; };

__device__ __forceinline__ TableRegs request_tables(const DevBlob& d)
{
    TableRegs r;
    const uint32_t nl = 1u << d.lut_bits;
    // What only codewords longer than the first-level table need, where there are any: requested before the others, so that the
    // number of loads behind those a later wait is for is the same on both paths (and without branches beyond this uniform one:
    // a guarded load would be moved down beside its use).
    r.first = r.count = r.index = r.sort = r.cb = 0u;
    if (longer_codes(d)) {
        const uint32_t l = threadIdx.x < 32u ? threadIdx.x : 32u;
        r.first = d.canon[l]; r.count = d.canon[33 + l]; r.index = d.canon[66 + l];
        r.sort = d.symsort[threadIdx.x < d.k_sym - 1u ? threadIdx.x : d.k_sym - 1u];
    }
#pragma unroll
    for (int k = 0; k < kTabTurns; ++k) {
        const uint32_t i = threadIdx.x + k * blockDim.x;
        r.e[k] = d.lut[i < nl ? i : nl - 1u];
        r.v[k] = 0u;
    }
    return r;
}

__device__ __forceinline__ void request_table_values(const DevBlob& d, TableRegs& r)
{
    // without symbols (an empty address map) the canonical table stands in as a valid address
    const uint32_t* cbp = d.k_sym ? reinterpret_cast<const uint32_t*>(d.codebook) : d.canon;
    if (longer_codes(d)) r.cb = cbp[r.sort < d.k_sym ? r.sort : 0u];
#pragma unroll
    for (int k = 0; k < kTabTurns; ++k) r.v[k] = cbp[(r.e[k] & 63u) ? r.e[k] >> 6 : 0u];
}

__device__ __forceinline__ Tables store_tables(const DevBlob& d, uint32_t* smem, TableRegs& r)
{
    const uint32_t nl = 1u << d.lut_bits;
    uint2* s_lut2 = reinterpret_cast<uint2*>(smem);
    uint32_t* s_bound = smem + 2 * nl;
    uint2* s_long2 = reinterpret_cast<uint2*>(s_bound + 100);
    // The values pass through an empty asm statement first: their loads then stay where they were
    // issued (the compiler would otherwise move a load down beside the guarded store that uses it,
    // behind every load issued since).
    static_assert(kTabTurns == 4, "the asm statement below names four values");
    asm volatile("" : "+v"(r.v[0]), "+v"(r.v[1]), "+v"(r.v[2]), "+v"(r.v[3]), "+v"(r.cb));
#pragma unroll
    for (int k = 0; k < kTabTurns; ++k) {
        const uint32_t i = threadIdx.x + k * blockDim.x;
        if (i < nl) s_lut2[i] = make_uint2(r.e[k], (r.e[k] & 63u) ? r.v[k] : 0u);
    }
    for (uint32_t i = threadIdx.x + kTabTurns * blockDim.x; i < nl; i += blockDim.x) {
        const uint32_t e = d.lut[i];
        s_lut2[i] = make_uint2(e, (e & 63u) ? __float_as_uint(d.codebook[e >> 6]) : 0u);
    }
    const bool longer = longer_codes(d);
    if (longer && threadIdx.x < kBounds) {                                      // (blocks have at least a wavefront)
        const uint32_t l = threadIdx.x;
        s_bound[l] = l < d.lmax && l < 32u ? (r.first + r.count) << (31u - l) : 0x80000000u;
        s_bound[kBounds + l] = r.index - r.first;
    }
    Tables t;
    t.lut2 = s_lut2; t.bound = s_bound; t.long2 = s_long2; t.small = d.k_sym <= kCodebookLdsMax;
    if (longer && t.small) {
        if (threadIdx.x < d.k_sym) s_long2[threadIdx.x] = make_uint2(r.sort, r.cb);
        for (uint32_t i = threadIdx.x + blockDim.x; i < d.k_sym; i += blockDim.x) {
            const uint32_t sy = d.symsort[i];
            s_long2[i] = make_uint2(sy, __float_as_uint(d.codebook[sy < d.k_sym ? sy : 0u]));
        }
    }
    return t;
}

__device__ __forceinline__ Tables load_tables(const DevBlob& d, uint32_t* smem)
{
    TableRegs r = request_tables(d);
    request_table_values(d, r);
    return store_tables(d, smem, r);
}

// ---------------------------------------------------------------------------
// one lane's progress through one chunk
// ---------------------------------------------------------------------------
struct ChunkState {
    uint32_t bp;      // next stream bit
    uint32_t row;     // HAC: row of the next symbol
    uint32_t wpos;    // CSC position of the next non-zero this lane will emit
    uint32_t wend;    // one past the chunk's last non-zero
};

// HAC: emit non-zeros until wpos reaches `limit` (<= wend).  Zeros only move `row`.
// When the zero symbol's codeword is the single bit 0, a run of zeros is a run of
// 0 bits and is skipped with a count-leading-zeros.
template <class Src, class Emit>
__device__ __forceinline__ void hac_advance(const DevBlob& d, const Tables& tb, const Src& src,
                                            ChunkState& st, uint32_t limit, Emit emit)
{
    const bool zfast = d.zero_len == 1;
    while (st.wpos < limit) {
        uint32_t top = src.peek32(st.bp);
        if (zfast) {
            if (top == 0) {                                            // a non-zero follows, so the run ends
                st.bp += 32; st.row += 32;
                st.wpos = st.row > d.n ? limit : st.wpos;              // ... unless the stream is damaged: end the walk
                continue;
            }
            const uint32_t z = (uint32_t)__builtin_clz(top);
            if (z) {
                st.bp += z; st.row += z;
                top = z + d.lmax <= 32 ? top << z : src.peek32(st.bp);
            }
        }
        const Decoded q = decode_symbol<Src::kInline>(d, tb, top);
        st.bp += q.len;
        if (d.has_zero && q.sym == 0) {
            st.row++;
            st.wpos = st.row > d.n ? limit : st.wpos;                  // a damaged stream: end the walk
            continue;
        }
        emit(st.wpos, st.row, q.sym, q.val);
        st.row++; st.wpos++;
    }
}

// The loops below are short chains that every lane walks alone, and what they take depends on where their instructions fall in
// the 32-byte pieces that are fetched: 17732 x 3387, 35 % non-zero, sHAC, 20 rows 376 or 389 us, 12000 x 30, 30 %, 8 rows 23.1 or 23.8,
// by what the code in front of them happened to leave.  (Padding is a few s_nop in front of a loop.)
#define ALIGN_DECODE_LOOP() asm volatile(".p2align 6")

// HAC, zero symbol = the single bit 0, words staged in LDS.  One pass of the loop per
// non-zero: 128 stream bits are fetched at once, a count-leading-zeros over the first
// 64 skips the zero run, and the codeword is taken from the same fetch.  Only a run
// of 64 or more zeros takes an extra pass (which steps over 96 bits when they are all zero:
// the lanes of a wave walk independently, and the wave runs as long as its slowest lane).
// The position is kept relative to the staged copy, less one (see WordSrc::peek32_rm1): three
// funnel shifts give the 96 bits, no 64-bit shift and no select on the bit offset.
__device__ __forceinline__ uint32_t leading_zeros_raw(uint32_t x)        // 0xffffffff for x == 0, as the instruction counts
{
    uint32_t r;
    asm("v_ffbh_u32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

template <class Emit>
__device__ __forceinline__ void hac_advance_zrun(const DevBlob& d, const Tables& tb, const WordSrc<true>& src,
                                                 ChunkState& st, uint32_t limit, Emit emit)
{
    lds_cu32* sw = (lds_cu32*)src.w;
    int32_t rm1 = (int32_t)(st.bp - (src.wbase << 5)) - 1;
    ALIGN_DECODE_LOOP();
    while (st.wpos < limit) {
        const int32_t q = rm1 >> 5;
        const uint32_t s = ~(uint32_t)rm1;
        const uint32_t w0 = sw[q], w1 = sw[q + 1], w2 = sw[q + 2], w3 = sw[q + 3];
        const uint32_t hi = __builtin_amdgcn_alignbit(w0, w1, s);
        const uint32_t mid = __builtin_amdgcn_alignbit(w1, w2, s);
        const uint32_t lo = __builtin_amdgcn_alignbit(w2, w3, s);
        if ((hi | mid) == 0) {                                             // a non-zero follows, so the run ends
            const uint32_t skip = lo ? 64u : 96u;                          // all 96 fetched bits may be zeros
            rm1 += (int32_t)skip; st.row += skip;
            st.wpos = st.row > d.n ? limit : st.wpos;                      // ... unless the stream is damaged: end the walk
            continue;
        }
        // hi == 0 counts as 0xffffffff and loses against 32 + (zeros of mid); mid == 0 with hi != 0 wraps to
        // 31, which is never below the zeros of hi
        const uint32_t zh = leading_zeros_raw(hi), zm = leading_zeros_raw(mid) + 32u;
        const uint32_t z = zh < zm ? zh : zm;
        const uint32_t x0 = z < 32u ? hi : mid, x1 = z < 32u ? mid : lo;
        const uint32_t zz = z & 31u;
        const uint32_t top = (x0 << zz) | ((x1 >> 1) >> (zz ^ 31u));
        const Decoded sy = decode_symbol<true>(d, tb, top);
        st.row += z;
        rm1 += (int32_t)(z + sy.len);
        emit(st.wpos, st.row, sy.sym, sy.val);
        st.row++; st.wpos++;
    }
    st.bp = (uint32_t)(rm1 + 1) + (src.wbase << 5);
}

// sHAC: every symbol is a non-zero.
template <class Src, class Emit>
__device__ __forceinline__ void shac_advance(const DevBlob& d, const Tables& tb, const Src& src,
                                             ChunkState& st, uint32_t limit, Emit emit)
{
    while (st.wpos < limit) {
        const Decoded q = decode_symbol<Src::kInline>(d, tb, src.peek32(st.bp));
        st.bp += q.len;
        emit(st.wpos, 0u, q.sym, q.val);
        st.wpos++;
    }
}

// The same over the staged copy.  The two words around the position and the one behind them stay in registers, the bits still
// ahead in the first counted from 31 down, so that what one codeword waits for is a funnel shift and the table's entry; the next
// word is read beside that.  (Reading both words at every codeword put a second LDS latency into the chain.)
template <class Emit>
__device__ __forceinline__ void shac_advance(const DevBlob& d, const Tables& tb, const WordSrc<true>& src,
                                             ChunkState& st, uint32_t limit, Emit emit)
{
    lds_cu32* sw = (lds_cu32*)src.w;
    const int32_t rm1 = (int32_t)(st.bp - (src.wbase << 5)) - 1;
    int32_t q = (rm1 >> 5) + 2, s = 31 - (rm1 & 31);                       // word q waits in w2
    uint32_t w0 = sw[q - 2], w1 = sw[q - 1], w2 = sw[q];
    ALIGN_DECODE_LOOP();
    while (st.wpos < limit) {
        const Decoded sy = decode_symbol<true>(d, tb, __builtin_amdgcn_alignbit(w0, w1, (uint32_t)s));
        s -= (int32_t)sy.len;
        const bool on = s < 0;                                             // into the next word
        w0 = on ? w1 : w0; w1 = on ? w2 : w1;
        q += on ? 1 : 0; s &= 31;
        w2 = sw[q];
        emit(st.wpos, 0u, sy.sym, sy.val);
        st.wpos++;
    }
    st.bp = (uint32_t)(32 * (q - 2) + 32 - s) + (src.wbase << 5);
}

// sHAC with Rice-coded row gaps: gap codeword, then the value's codeword.  Gap d with
// q = d >> k: q zeros, a one, k low bits of d; from q = 31 on: 31 zeros, a one, d in 32 bits.
// st.row is the row the next gap counts from.  Words staged in LDS: one fetch of 128 bits
// serves the unary part (count-leading-zeros), the remainder and the value's codeword.
template <class Emit>
__device__ __forceinline__ void gap_advance(const DevBlob& d, const Tables& tb, const WordSrc<true>& src,
                                            ChunkState& st, uint32_t limit, Emit emit)
{
    lds_cu32* sw = (lds_cu32*)src.w;
    const uint32_t k = d.rice_k;
    int32_t rm1 = (int32_t)(st.bp - (src.wbase << 5)) - 1;                 // as in hac_advance_zrun: funnel shifts only
    ALIGN_DECODE_LOOP();
    while (st.wpos < limit) {
        const int32_t q = rm1 >> 5;
        const uint32_t s = ~(uint32_t)rm1;
        const uint32_t w0 = sw[q], w1 = sw[q + 1], w2 = sw[q + 2], w3 = sw[q + 3];
        const uint32_t hi = __builtin_amdgcn_alignbit(w0, w1, s);
        const uint32_t mid = __builtin_amdgcn_alignbit(w1, w2, s);
        const uint32_t lo = __builtin_amdgcn_alignbit(w2, w3, s);
        const uint32_t z0 = leading_zeros_raw(hi), z = z0 < 31u ? z0 : 31u;   // a valid stream has a one within 32 bits
        uint32_t gapv, top, used;
        if (z < 31) {
            const uint32_t p0 = __builtin_amdgcn_alignbit(hi, mid, 31u - z), p1 = __builtin_amdgcn_alignbit(mid, lo, 31u - z);   // behind the one
            used = z + 1 + k;
            gapv = (z << k) | ((p0 >> 1) >> (31u - k));
            top = k ? __builtin_amdgcn_alignbit(p0, p1, 32u - k) : p0;
        } else {
            gapv = mid; top = lo; used = 64;
        }
        const Decoded sy = decode_symbol<true>(d, tb, top);
        const uint32_t row = st.row + gapv;
        rm1 += (int32_t)(used + sy.len);
        st.row = row + 1;
        emit(st.wpos, row, sy.sym, sy.val);
        st.wpos++;
    }
    st.bp = (uint32_t)(rm1 + 1) + (src.wbase << 5);
}

// The same from any word source, one field at a time (streams too long to stage, and the
// test-only decode kernel).
template <class Src, class Emit>
__device__ __forceinline__ void gap_advance_slow(const DevBlob& d, const Tables& tb, const Src& src,
                                                 ChunkState& st, uint32_t limit, Emit emit)
{
    const uint32_t k = d.rice_k;
    while (st.wpos < limit) {
        const uint32_t hi = src.peek32(st.bp);
        const uint32_t z = hi ? (uint32_t)__builtin_clz(hi) : 31u;
        st.bp += z + 1;
        uint32_t gapv;
        if (z < 31) {
            gapv = (z << k) | (k ? src.peek32(st.bp) >> (32 - k) : 0u);
            st.bp += k;
        } else {
            gapv = src.peek32(st.bp);
            st.bp += 32;
        }
        const Decoded q = decode_symbol<Src::kInline>(d, tb, src.peek32(st.bp));
        st.bp += q.len;
        const uint32_t row = st.row + gapv;
        st.row = row + 1;
        emit(st.wpos, row, q.sym, q.val);
        st.wpos++;
    }
}

// column that owns chunk g: largest j with colchunk[j] <= g (global memory search)
__device__ __forceinline__ uint32_t column_of_chunk(const DevBlob& d, uint32_t g)
{
    uint32_t lo = 0, hi = d.m;               // invariant: colchunk[lo] <= g < colchunk[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (d.colchunk[mid] <= g) lo = mid; else hi = mid;
    }
    return lo;
}

} // namespace

#endif
