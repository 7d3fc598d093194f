// Dense-tile product for an index-mapped matrix on gfx950 (MI355X):
//     Y[b][j] = sum_i X[b][i] * c[Pi[i][j]]
// (arXiv 2108.12704 Sect. III-C1: representatives in a vector c, pointers to them
// in the index map Pi; the form the paper uses for layers that are quantized but
// hardly pruned, where the product really is a dense contraction).
//
// The pointers are what is read from memory (1 or 2 bytes per weight).  What bounds the product is the
// matrix pipe: v_mfma_f32_32x32x2_f32 does 157 TFLOP/s at best, the bf16 instruction sixteen times that.
// So every fp32 operand is written as three bf16 parts, x = x1 + x2 + x3 (8 significant bits each, 24 in
// all), and six of the nine products of parts are summed in fp32 on the matrix cores: x1 w1, x1 w2, x2 w1,
// x2 w2, x1 w3, x3 w1.  The three left out are together below 2^-24 of |x w|, and one rounding of the sum per 16 products
// of parts instead of one per two makes the result closer to 64 bits than the fp32 instruction's
// (relative 2-norm error figures at plan_index_gemm).  X is split on the way to LDS, W's representatives once per block in
// the table that pointers are looked up in; every part is rounded to nearest.
// Below 2^-110 a third part has no room for the last bits, and an infinity or NaN makes the parts NaN
// (inf - inf).  A block that meets such an operand, or whose sums are not finite, computes its tile with the fp32
// instruction instead.
//
// Tiling: a block of 4 wavefronts owns 32 RT batch rows x 128 columns of Y (RT = 1..4; some blocks a row tile less, so that all CUs
// get the same) and walks K = n in steps of 32; wavefront w owns the 32 columns [32 w, 32 w + 32) of the tile and all its
// rows, as RT MFMA tiles (two sums each, 32 RT accumulator registers).  LDS holds two K steps: of X as parts, the 32 k of a row side
// by side, part by part, 208 bytes apart, so that an operand is one 128-bit read and 16 lanes' reads fall on different
// banks; of W the pointers only, turned so that a lane reads eight k of its column at once.  A column belongs to one
// wavefront, so its pointers are looked up by the lanes that multiply the values, straight into operands: writing parts of W
// to LDS and reading them back took a third of the LDS pipe's time.
// What bounds a step is the order of its instructions: two wavefronts on a SIMD do not cover what one of them waits for.  One
// barrier a step; X is split and stored for the next step, pointers for the one after next, operands are read a row tile and
// looked up half a step ahead, and every global load has a step to arrive, all of it between matrix instructions
// (sched_group_barrier; the compiler's own order, with the loads behind the products and waits before each, took 390 us
// where this one takes 348).
// Measured (MI355X), fp32 instruction -> bf16 parts, W's parts in LDS -> this kernel, whole calls: 4608 x 512 layer pruned 60 %, 12544
// rows 580 -> 354 -> 331 us (59 GFLOP; a call includes decoding the stream, about 25 us); unpruned map of that size, 784 rows
// 60.0 -> 37.9 -> 35.4 us; products alone 2048 x 2000 x 2000 112 -> 93, 12544 x 576 x 64 25.9 -> 20.5, 64 x 25088 x 1000 42 -> 35,
// 512 x 9973 x 1511 98 -> 93, 300 x 4096 x 4096 84 -> 71, 46 x 64 x 10 5.6 -> 5.6.  Same sums in the same order, same bits.
// Before row tiles were dealt evenly matrix pipes were 51 % busy at 12544 rows (44 % with W in LDS; 67 % on a CU with two blocks).
// Lane layout of v_mfma_f32_32x32x16_bf16: A operand lane l holds A[i = l % 32][k = 8 (l / 32) + 0..7], B
// operand lane l holds B[k = 8 (l / 32) + 0..7][j = l % 32], accumulator register v of lane l is
// D[(v % 4) + 8 (v / 4) + 4 (l / 32)][l % 32].
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "hac_internal.h"

namespace {

constexpr int BN = 128, BK = 32;
constexpr int PART = 2 * BK, PITCH = 3 * PART + 16;   // bytes: one part of a row's K step, one row of X in LDS
// bytes between two columns' pointers in LDS: 16 (32) lanes' 128-bit (64-bit) reads fall on different banks
template <typename IdxT> constexpr int ptr_pitch() { return sizeof(IdxT) == 1 ? BK + 8 : 2 * BK + 16; }
// two K steps of X and of pointers
template <typename IdxT> constexpr int tile_bytes(int rt) { return 2 * (32 * rt * PITCH + BN * ptr_pitch<IdxT>()); }
constexpr uint32_t kMinRT = 1, kMaxRT = 4;              // row tiles of 32 per block
constexpr uint32_t kLutLdsMax = 4096;              // representatives kept in LDS

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Pointers: four neighbouring ones of a row of the map as they are loaded (raw), eight k of one column as a lane multiplies them
// (oct).  __builtin_amdgcn_perm(hi, lo, ..) picks bytes of two words.
__device__ __forceinline__ uint32_t upper16(uint32_t hi, uint32_t lo) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }
__device__ __forceinline__ uint32_t lower16(uint32_t hi, uint32_t lo) { return __builtin_amdgcn_perm(hi, lo, 0x05040100u); }
template <typename IdxT> struct Ptr4;
template <> struct Ptr4<uint8_t> {
    typedef uint32_t raw;
    typedef uint2 oct;
    static __device__ __forceinline__ uint32_t get(raw w, int c) { return (w >> (8 * c)) & 255u; }
    static __device__ __forceinline__ uint32_t get8(oct w, int j) { return ((j & 4 ? w.y : w.x) >> (8 * (j & 3))) & 255u; }
    static __device__ __forceinline__ void ld(const uint8_t* p, uint32_t* out) {
        const uint32_t w = *reinterpret_cast<const uint32_t*>(p);
        out[0] = w & 255u; out[1] = (w >> 8) & 255u; out[2] = (w >> 16) & 255u; out[3] = w >> 24;
    }
    // rows r[0..3] of four columns -> out[c]: the four k of column c
    static __device__ __forceinline__ void turn(const raw* r, raw* out) {
        const uint32_t a = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u), b = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u);
        const uint32_t c = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u), d = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);
        out[0] = lower16(b, a); out[1] = upper16(b, a); out[2] = lower16(d, c); out[3] = upper16(d, c);
    }
};
template <> struct Ptr4<uint16_t> {
    typedef uint2 raw;
    typedef uint4 oct;
    static __device__ __forceinline__ uint32_t get(raw w, int c) { return ((c & 2 ? w.y : w.x) >> (16 * (c & 1))) & 65535u; }
    static __device__ __forceinline__ uint32_t get8(oct w, int j) {
        return ((j & 4 ? (j & 2 ? w.w : w.z) : (j & 2 ? w.y : w.x)) >> (16 * (j & 1))) & 65535u;
    }
    static __device__ __forceinline__ void ld(const uint16_t* p, uint32_t* out) {
        const uint2 w = *reinterpret_cast<const uint2*>(p);
        out[0] = w.x & 65535u; out[1] = w.x >> 16; out[2] = w.y & 65535u; out[3] = w.y >> 16;
    }
    static __device__ __forceinline__ void turn(const raw* r, raw* out) {
        out[0] = make_uint2(lower16(r[1].x, r[0].x), lower16(r[3].x, r[2].x));
        out[1] = make_uint2(upper16(r[1].x, r[0].x), upper16(r[3].x, r[2].x));
        out[2] = make_uint2(lower16(r[1].y, r[0].y), lower16(r[3].y, r[2].y));
        out[3] = make_uint2(upper16(r[1].y, r[0].y), upper16(r[3].y, r[2].y));
    }
};

// w = w1 + w2 + w3: { w1 | w2 << 16, w3 }.  Rounded to nearest (ties upwards in magnitude), so that the
// parts' signs vary and the left-out products have no bias; cut off instead where rounding could overflow.
// `cut` collects the third parts' fp32 patterns: what a bf16 has no room for is in the lower 16 bits (not
// zero below 2^-110 only).
__device__ __forceinline__ uint2 split_weight(float w, uint32_t& cut)
{
    const uint32_t up = fabsf(w) < 1e38f ? 0x8000u : 0u;
    const uint32_t h1 = (__float_as_uint(w) + up) & 0xffff0000u;
    const float r1 = w - __uint_as_float(h1);
    const uint32_t h2 = (__float_as_uint(r1) + up) & 0xffff0000u;
    const uint32_t h3 = __float_as_uint(r1 - __uint_as_float(h2));
    cut |= h3;
    return make_uint2((h1 >> 16) | h2, h3 >> 16);
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 float4u __attribute__((aligned(4)));        // global memory takes 128-bit loads at any word
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t two_bf16(f32x2 v) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2)); }   // to nearest even
__device__ __forceinline__ f32x2 two_f32(uint32_t p) { return f32x2{__uint_as_float(p << 16), __uint_as_float(p & 0xffff0000u)}; }

// the order inside a row tile's group: after each of its six matrix instructions up to `n` other vector instructions
#define ALWAYS_INLINE __attribute__((always_inline))
#define INTERLEAVE(n)                                              \
    do {                                                           \
        _Pragma("unroll") for (int z = 0; z < 6; ++z) {            \
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     \
            __builtin_amdgcn_sched_group_barrier(0x002, n, 0);     \
        }                                                          \
    } while (0)

__device__ __forceinline__ uint32_t logical_tile(uint32_t tiles_padded)
{
    // consecutive logical tiles on one XCD: the column tiles of a row tile share X rows in that L2
    const uint32_t per = tiles_padded >> 3;
    return (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
}

// (blocks per CU: 2 of three or four row tiles, 3 of two, 4 of one; their accumulators and operands in flight fill the registers)
template <typename IdxT, bool LUT_LDS, int RT>
__global__ void __launch_bounds__(256, RT >= 3 ? 2 : RT == 2 ? 3 : 4)
index_gemm_kernel(const float* __restrict__ X, uint64_t ldx, uint32_t B,
                  const IdxT* __restrict__ idx, uint64_t pitch,          // pitch in elements, a multiple of 16
                  const float* __restrict__ codebook, uint32_t k_sym, uint32_t zero_first,
                  uint32_t n, uint32_t m, float* __restrict__ Y, uint64_t ldy,
                  uint32_t tiles_n, uint32_t row_groups, uint32_t splits, uint32_t steps_per_split, float* __restrict__ part)
{
    constexpr int BM = 32 * RT;
    extern __shared__ __align__(16) float lds[];
    constexpr int PP = ptr_pitch<IdxT>(), ABYTES = BM * PITCH, BBYTES = BN * PP;
    char* As = reinterpret_cast<char*>(lds);           // two buffers of [BM] rows of PITCH bytes
    char* Ps = As + 2 * ABYTES;                        // two buffers of [BN] columns of PP bytes
    uint2* lut = reinterpret_cast<uint2*>(Ps + 2 * BBYTES);   // [k_sym + zero_first] when LUT_LDS
    // work item = (tile, K split); with more than one split a block writes its partial tile to
    // part[split][B][m] and a second kernel adds the splits in order
    const uint32_t item = logical_tile(gridDim.x);
    if (item >= row_groups * tiles_n * splits) return;
    const uint32_t tile = item / splits, split = item - tile * splits;
    const uint32_t tm = tile / tiles_n, tn = tile - tm * tiles_n;
    // row tiles of this block: RT, or RT - 1 where there are more groups than RT needs
    const uint32_t row_tiles = (B + 31) / 32;
    const uint32_t first = (uint32_t)((uint64_t)tm * row_tiles / row_groups);
    const uint32_t nr = (uint32_t)((uint64_t)(tm + 1) * row_tiles / row_groups) - first;
    const uint32_t m0 = 32 * first, n0 = tn * BN;
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const uint32_t l32 = lane & 31, half = lane >> 5;

    // pointer -> value; entry 0 is 0.0 when the pointers were written with an offset of one
    const uint32_t k_tot = k_sym + zero_first;
    auto value_of = [&](uint32_t p) ALWAYS_INLINE -> float { return (zero_first && p == 0) ? 0.0f : codebook[p - zero_first]; };
    uint32_t cut = 0;                                  // lower half not 0: some operand is more than its three parts
    typedef typename Ptr4<IdxT>::raw raw_t;
    typedef typename Ptr4<IdxT>::oct oct_t;
    auto parts_of = [&](uint32_t p) ALWAYS_INLINE -> uint2 { return LUT_LDS ? lut[p] : split_weight(value_of(p), cut); };

    // Global -> registers.  X: rows a_row + 32 r, k = 4 q .. 4 q + 3; map: rows 4 q .. 4 q + 3, columns
    // b_col .. b_col + 3 (four k of a column in one thread, so that a part of them is one 64-bit store).
    // Rows past B and columns past the pitch are read from a clamped, valid address and never stored;
    // only the last, partial K step is guarded.
    struct Stage { f32x4 ra[RT]; raw_t rb[4]; };
    const uint32_t q = t & 7, a_row = t >> 3, b_col = 4 * (t >> 3);
    const float* xrow[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const uint32_t row = m0 + a_row + 32 * r;
        xrow[r] = X + (uint64_t)(row < B ? row : B - 1) * ldx + 4 * q;
    }
    const IdxT* icol = idx + (n0 + b_col < pitch ? n0 + b_col : 0);
    Stage st;
    auto load_x_full = [&](uint32_t kt, int r) ALWAYS_INLINE {
        st.ra[r] = *reinterpret_cast<const float4u*>(xrow[r] + kt * BK);   // (rows of X start at any float)
    };
    auto load_p_full = [&](uint32_t kt, raw_t* rb) ALWAYS_INLINE {
#pragma unroll
        for (int j = 0; j < 4; ++j) rb[j] = *reinterpret_cast<const raw_t*>(icol + (uint64_t)(kt * BK + 4 * q + j) * pitch);
    };
    const uint32_t nfull = n / BK;
    auto load_x = [&](uint32_t kt, int r) ALWAYS_INLINE {
        if (kt < nfull) { load_x_full(kt, r); return; }
        const uint32_t k = kt * BK + 4 * q;
        const float* p = xrow[r] + kt * BK;
        f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
        if (k < n) v.x = p[0];
        if (k + 1 < n) v.y = p[1];
        if (k + 2 < n) v.z = p[2];
        if (k + 3 < n) v.w = p[3];
        st.ra[r] = v;
    };
    auto load_p = [&](uint32_t kt, raw_t* rb) ALWAYS_INLINE {
        if (kt < nfull) { load_p_full(kt, rb); return; }
#pragma unroll
        for (int j = 0; j < 4; ++j) {                  // (past the end: any row of the map, X is 0 there)
            const uint32_t k = kt * BK + 4 * q + j;
            rb[j] = *reinterpret_cast<const raw_t*>(icol + (uint64_t)(k < n ? k : n - 1) * pitch);
        }
    };
    // registers -> LDS, buffer `buf`
    auto store_p = [&](uint32_t buf, const raw_t* rb) ALWAYS_INLINE {
        raw_t col[4];
        Ptr4<IdxT>::turn(rb, col);
#pragma unroll
        for (int c = 0; c < 4; ++c) *reinterpret_cast<raw_t*>(Ps + buf * BBYTES + (b_col + c) * PP + 4 * sizeof(IdxT) * q) = col[c];
    };
    auto store_x = [&](uint32_t buf, int r) ALWAYS_INLINE {
        const float x[4] = {st.ra[r].x, st.ra[r].y, st.ra[r].z, st.ra[r].w};
        uint32_t p1[2], p2[2], p3[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const f32x2 v = {x[2 * j], x[2 * j + 1]};
            p1[j] = two_bf16(v);
            const f32x2 r1 = v - two_f32(p1[j]);
            p2[j] = two_bf16(r1);
            const f32x2 r2 = r1 - two_f32(p2[j]);
            p3[j] = two_bf16(r2);
            cut |= __float_as_uint(r2.x) | __float_as_uint(r2.y);
        }
        char* a = As + buf * ABYTES + (a_row + 32 * r) * PITCH + 8 * q;
        *reinterpret_cast<uint2*>(a) = make_uint2(p1[0], p1[1]);
        *reinterpret_cast<uint2*>(a + PART) = make_uint2(p2[0], p2[1]);
        *reinterpret_cast<uint2*>(a + 2 * PART) = make_uint2(p3[0], p3[1]);
    };

    // x1 w1 has a sum of its own: the instruction rounds a sum once per 16 k, and the five others, 2^-8 of it
    // and less, would each round the large sum again (one sum for all six:
    // 5.8 times the error at 4608 x 512, 12544 rows, and 1.6 times that of the fp32 instruction)
    f32x16 acc[RT], low[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = low[i][v] = 0.0f;

    // a lane's operand of 16 k: the parts of eight k of its column, looked up by the wavefront that multiplies them
    auto pointers = [&](uint32_t buf, int h) ALWAYS_INLINE -> oct_t {
        return *reinterpret_cast<const oct_t*>(Ps + buf * BBYTES + (wave * 32 + l32) * PP + (16 * h + 8 * half) * sizeof(IdxT));
    };
    auto look_up = [&](const oct_t& p, uint2* v) ALWAYS_INLINE {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = parts_of(Ptr4<IdxT>::get8(p, j));
    };
    auto pack = [&](const uint2* v, bf16x8* w) ALWAYS_INLINE {
        w[0] = __builtin_bit_cast(bf16x8, make_uint4(lower16(v[1].x, v[0].x), lower16(v[3].x, v[2].x), lower16(v[5].x, v[4].x), lower16(v[7].x, v[6].x)));
        w[1] = __builtin_bit_cast(bf16x8, make_uint4(upper16(v[1].x, v[0].x), upper16(v[3].x, v[2].x), upper16(v[5].x, v[4].x), upper16(v[7].x, v[6].x)));
        w[2] = __builtin_bit_cast(bf16x8, make_uint4(lower16(v[1].y, v[0].y), lower16(v[3].y, v[2].y), lower16(v[5].y, v[4].y), lower16(v[7].y, v[6].y)));
    };
    struct RowParts { bf16x8 x[3]; };
    auto rows = [&](uint32_t buf, int h, int i) ALWAYS_INLINE -> RowParts {
        const char* a = As + buf * ABYTES + (l32 + 32 * i) * PITCH + 16 * half + 32 * h;
        RowParts o;
#pragma unroll
        for (int p = 0; p < 3; ++p) o.x[p] = *reinterpret_cast<const bf16x8*>(a + p * PART);
        return o;
    };
    auto multiply = [&](int i, const RowParts& o, const bf16x8* w) ALWAYS_INLINE {
        low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.x[2], w[0], low[i], 0, 0, 0);
        low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.x[0], w[2], low[i], 0, 0, 0);
        low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.x[1], w[1], low[i], 0, 0, 0);
        low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.x[1], w[0], low[i], 0, 0, 0);
        low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.x[0], w[1], low[i], 0, 0, 0);
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.x[0], w[0], acc[i], 0, 0, 0);
    };

    const uint32_t all_steps = (n + BK - 1) / BK;
    const uint32_t kt0 = split * steps_per_split;
    const uint32_t ksteps = kt0 + steps_per_split < all_steps ? kt0 + steps_per_split : all_steps;   // one past the last
    // true if f holds for any thread of the block: a word per wavefront and a barrier (0.3 us less per vote than
    // __syncthreads_or); every vote has words of its own
    __shared__ uint32_t votes[2][4];
    auto block_any = [&](bool f, int which) ALWAYS_INLINE -> bool {
        const bool mine = __any(f);
        if (lane == 0) votes[which][wave] = mine ? 1u : 0u;
        __syncthreads();
        return (votes[which][0] | votes[which][1] | votes[which][2] | votes[which][3]) != 0;
    };
    // an operand was cut short, or a sum is not finite (an infinity or NaN among the operands, or an overflow)
    // (x * 0 is NaN exactly then: one instruction per sum; a comparison each took 0.2 us a block)
    auto unfit = [&]() ALWAYS_INLINE -> bool {
        float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) t[v & 3] = fmaf(acc[i][v] + low[i][v], 0.0f, t[v & 3]);
        return (cut & 0xffffu) != 0 || !((t[0] + t[1]) + (t[2] + t[3]) == 0.0f);
    };
    // a look at some of the first step's X (non-finite, or small enough to be cut) and at the table: where all of X, or a
    // representative, is like this, parts are not tried first
    auto load = [&](uint32_t kt) ALWAYS_INLINE {
#pragma unroll
        for (int r = 0; r < RT; ++r) load_x(kt, r);
        load_p(kt, st.rb);
    };
    raw_t rb1[4];                                      // pointers of the second step (of the first where there is one only)
    load_p(kt0 + 1 < ksteps ? kt0 + 1 : kt0, rb1);
    load(kt0);                                         // (in flight while the table is made)
    if (LUT_LDS)
        for (uint32_t i = t; i < k_tot; i += 256) lut[i] = split_weight(value_of(i), cut);
    bool again = (cut & 0xffffu) != 0 || n == 1;
    const float seen[4] = {st.ra[0].x, st.ra[0].y, st.ra[0].z, st.ra[0].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) again |= !(fabsf(seen[j]) <= 3.402823466e38f) || (seen[j] != 0.0f && fabsf(seen[j]) < 0x1p-110f);
    again = block_any(again, 0);                       // (a barrier: the table is complete)
    if (!again) {
        // Step kt multiplies buffer kt of X; the wavefront has its first operand of W in registers and the pointers of the second.
        // Beside the matrix instructions: X of step kt + 1 is split into the other buffer and X of kt + 2 requested, the
        // pointers of kt + 2 go to LDS and those of kt + 3 are requested, the operands of kt + 1 are looked up.  The order is
        // spelled out (a sched_barrier behind every row tile): left to itself the compiler requests at the end what the next step
        // waits for at its start and reads every operand right before its use.
        auto walk = [&](auto count) ALWAYS_INLINE {
        constexpr int NR = decltype(count)::value;
        bf16x8 w[2][3];
        oct_t p1;
        uint2 v[8];
#pragma unroll
        for (int r = 0; r < NR; ++r) store_x(0, r);
        store_p(0, st.rb);
        store_p(1, rb1);
        if (kt0 + 1 < ksteps) {
#pragma unroll
            for (int r = 0; r < NR; ++r) load_x(kt0 + 1, r);
        }
        if (kt0 + 2 < ksteps) load_p(kt0 + 2, st.rb);
        __syncthreads();
        look_up(pointers(0, 0), v);
        p1 = pointers(0, 1);
        pack(v, w[0]);
        __syncthreads();                               // the first step overwrites these pointers
        auto step = [&](uint32_t kt, auto request_x, auto request_p) ALWAYS_INLINE {
            const uint32_t buf = (kt - kt0) & 1u;
            RowParts o = rows(buf, 0, 0), next;
            look_up(p1, v);
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                next = i + 1 < NR ? rows(buf, 0, i + 1) : rows(buf, 1, 0);
                store_x(buf ^ 1u, i);
                multiply(i, o, w[0]);
                request_x(kt + 2, i);
                INTERLEAVE(7);
                __builtin_amdgcn_sched_barrier(0);
                o = next;
            }
            pack(v, w[1]);
            const oct_t p0 = pointers(buf ^ 1u, 0);
            p1 = pointers(buf ^ 1u, 1);
            store_p(buf, st.rb);                            // (of step kt + 2: this step's pointers are in registers already)
            request_p(kt + 3);
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                if (i + 1 < NR) next = rows(buf, 1, i + 1);
                if (i == (NR > 1 ? 1 : 0)) look_up(p0, v);
                if (i == NR - 1) pack(v, w[0]);
                multiply(i, o, w[1]);
                INTERLEAVE(3);
                __builtin_amdgcn_sched_barrier(0);
                o = next;
            }
            __syncthreads();
        };
        uint32_t kt = kt0;
        for (const uint32_t end = ksteps < nfull ? ksteps : nfull; kt + 3 < end; ++kt)
            step(kt, [&](uint32_t k, int r) ALWAYS_INLINE { load_x_full(k, r); }, [&](uint32_t k) ALWAYS_INLINE { load_p_full(k, st.rb); });
        for (; kt < ksteps; ++kt)
            step(kt, [&](uint32_t k, int r) ALWAYS_INLINE { if (k < ksteps) load_x(k, r); }, [&](uint32_t k) ALWAYS_INLINE { if (k < ksteps) load_p(k, st.rb); });
        };
        if (nr == RT) walk(std::integral_constant<int, RT>{});
        else if constexpr (RT > 1) walk(std::integral_constant<int, RT - 1>{});
    }
    if (!again) again = block_any(unfit(), 1);
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] += low[i][v];

    // The tile once more with the fp32 instruction (157 TFLOP/s at best) where parts will not do: the same loads, one fp32
    // value per operand in LDS.  The order of k inside a step is free as long as both operands agree:
    // instruction kk multiplies k = kk (lanes 0..31) and k = 16 + kk (lanes 32..63), so that a lane's 16
    // values of a step are four 128-bit reads.  It costs such a tile what it cost before parts were used, and
    // the steps walked until that is known.
    if (again) {
        constexpr int P32 = BK + 4;                    // floats between rows: 16 lanes' reads fall on different banks
        static_assert(4 * P32 * (BM + BN) <= 2 * (ABYTES + BBYTES), "the fp32 tiles take the place of the parts and pointers");
        float* Af = reinterpret_cast<float*>(As);
        float* Bf = Af + BM * P32;
        if (LUT_LDS)
            for (uint32_t i = t; i < k_tot; i += 256) lut[i].x = __float_as_uint(value_of(i));   // (the vote was a barrier)
        auto fp32_of = [&](uint32_t p) ALWAYS_INLINE -> float { return LUT_LDS ? __uint_as_float(lut[p].x) : value_of(p); };
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][v] = 0.0f;
        load(kt0);
        for (uint32_t kt = kt0; kt < ksteps; ++kt) {
            __syncthreads();
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float w[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) w[j] = fp32_of(Ptr4<IdxT>::get(st.rb[j], c));
                *reinterpret_cast<float4*>(Bf + (b_col + c) * P32 + 4 * q) = make_float4(w[0], w[1], w[2], w[3]);
            }
#pragma unroll
            for (int r = 0; r < RT; ++r) *reinterpret_cast<f32x4*>(Af + (a_row + 32 * r) * P32 + 4 * q) = st.ra[r];
            __syncthreads();
            if (kt + 1 < ksteps) load(kt + 1);
            const float* a = Af + l32 * P32 + 16 * half;
            const float* b = Bf + (wave * 32 + l32) * P32 + 16 * half;
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const float4 w4 = *reinterpret_cast<const float4*>(b + 4 * h);
                const float w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    const float4 x4 = *reinterpret_cast<const float4*>(a + 32 * i * P32 + 4 * h);
                    const float x[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[j], w[j], acc[i], 0, 0, 0);
                }
            }
        }
    }

    const uint32_t col = n0 + wave * 32 + l32;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const uint32_t row = m0 + i * 32 + (v & 3) + 8 * (v >> 2) + 4 * half;
            if (row < B && col < m && (uint32_t)i < nr) {
                if (splits == 1) Y[(uint64_t)row * ldy + col] = acc[i][v];
                else part[((uint64_t)split * B + row) * m + col] = acc[i][v];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Small batches (at most 32 rows of X, in groups of 8 along the grid's y): nothing much for the
// matrix cores to do; the index map is read straight through, once per group of 8 batch rows
// (from L2 after the first), and every pointer is used for the group's rows.  A block of 256
// threads owns 256 columns and a range of rows of W: thread (c, g) walks the rows g, g + 4, ...
// of the range for the four columns 4c .. 4c + 3 (one 4- or 8-byte load per row; a wavefront
// reads 256 neighbouring pointers of one row), with the range's X values in LDS (one broadcast
// read per row) and the representatives in LDS.  The four row groups of a block are added in
// LDS, the row ranges by splitk_reduce_kernel: a fixed order.
// ---------------------------------------------------------------------------
constexpr int SB_NB = 8, SB_COLS = 256, SB_GROUPS = 4;     // widest layout: 64 column lanes x 4 row groups
constexpr uint32_t kSmallMaxRows = 1024;           // rows of W per block (32 KB of X in LDS)

template <typename IdxT, bool LUT_LDS, bool WIDE>
__global__ void __launch_bounds__(256)
index_small_kernel(const float* __restrict__ X, uint64_t ldx, uint32_t B,
                   const IdxT* __restrict__ idx, uint64_t pitch,
                   const float* __restrict__ codebook, uint32_t k_sym, uint32_t zero_first,
                   uint32_t n, uint32_t m, uint32_t rows_per_split, uint32_t tiles_m, uint32_t splits,
                   uint32_t cl_log2_arg, float* __restrict__ Y, uint64_t ldy, float* __restrict__ part)
{
    const uint32_t cl_log2 = WIDE ? 6u : cl_log2_arg;              // the widest layout with compile-time shapes
    // 2^cl_log2 column lanes (4 columns each) x 256 / 2^cl_log2 row groups: 64 x 4 for a map of 129
    // columns or more, fewer lanes and more row groups for a narrow one, so that its rows are spread
    // over the block's threads instead of leaving most of them idle
    const uint32_t cl = 1u << cl_log2, cols = 4u << cl_log2, groups = 256u >> cl_log2;
    extern __shared__ float lds[];
    float* xs = lds;                                               // [rows_per_split][SB_NB]
    float* red = xs + (size_t)rows_per_split * SB_NB;              // [groups][SB_NB][cols]: 8192 floats in every layout
    float* lut = red + SB_GROUPS * SB_NB * SB_COLS;                // [k_sym + zero_first] when LUT_LDS
    const uint32_t tile = blockIdx.x % tiles_m, split = blockIdx.x / tiles_m;
    const uint32_t b0 = blockIdx.y * SB_NB;                        // this block's batch rows b0 .. b0 + 7
    const uint32_t nb = B - b0 < (uint32_t)SB_NB ? B - b0 : (uint32_t)SB_NB;
    const uint32_t c = threadIdx.x & (cl - 1), g = threadIdx.x >> cl_log2;
    const uint32_t j = tile * cols + 4 * c;                        // first of this thread's four columns
    const uint32_t r0 = split * rows_per_split;
    const uint32_t rows = r0 < n ? (n - r0 < rows_per_split ? n - r0 : rows_per_split) : 0u;
    const uint32_t k_tot = k_sym + zero_first;
    if (LUT_LDS) {
        for (uint32_t i = threadIdx.x; i < k_tot; i += 256)
            lut[i] = (zero_first && i == 0) ? 0.0f : codebook[i - zero_first];
    }
    // a thread stages whole rows: SB_NB coalesced reads (one per batch row), one contiguous store
    for (uint32_t i = threadIdx.x; i < rows; i += 256) {
        float v[SB_NB];
#pragma unroll
        for (int b = 0; b < SB_NB; ++b) v[b] = (uint32_t)b < nb ? X[(uint64_t)(b0 + b) * ldx + r0 + i] : 0.0f;
#pragma unroll
        for (int b = 0; b < SB_NB; ++b) xs[(size_t)i * SB_NB + b] = v[b];
    }
    __syncthreads();
    auto value_of = [&](uint32_t p) -> float {
        if (LUT_LDS) return lut[p];
        return (zero_first && p == 0) ? 0.0f : codebook[p - zero_first];
    };
    float acc[4][SB_NB];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int b = 0; b < SB_NB; ++b) acc[u][b] = 0.0f;
    // the pitch is a multiple of 16 and j of 4: four pointers from j on lie inside the row; those of
    // columns past m are padding (pointer 0) and their sums are never stored
    if (j < pitch) {
        const IdxT* col = idx + (uint64_t)r0 * pitch + j;
        auto row_step = [&](uint32_t i, const uint32_t* p) {
            const float* xr = xs + (size_t)i * SB_NB;
            float x[SB_NB];
#pragma unroll
            for (int b = 0; b < SB_NB; ++b) x[b] = xr[b];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float w = value_of(p[u]);
#pragma unroll
                for (int b = 0; b < SB_NB; ++b) acc[u][b] = fmaf(w, x[b], acc[u][b]);
            }
        };
        uint32_t i = g;
        // four rows at a time: their pointers are requested together, so that a thread with few
        // rows does not pay one trip to memory per row
        for (; i + 3 * groups < rows; i += 4 * groups) {
            uint32_t p[4][4];
#pragma unroll
            for (int q = 0; q < 4; ++q) Ptr4<IdxT>::ld(col + (uint64_t)(i + q * groups) * pitch, p[q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) row_step(i + q * groups, p[q]);
        }
        for (; i < rows; i += groups) {
            uint32_t p[4];
            Ptr4<IdxT>::ld(col + (uint64_t)i * pitch, p);
            row_step(i, p);
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int b = 0; b < SB_NB; ++b) red[(g * SB_NB + b) * cols + 4 * c + u] = acc[u][b];
    __syncthreads();
    // every (batch row, column) of the block: its row groups added in order, the outputs dealt to
    // the threads (256 columns x 8 rows in the widest layout, 16 x 8 with 64 row groups in the narrowest)
    for (uint32_t o = threadIdx.x; o < cols * nb; o += 256) {
        const uint32_t jl = o & (cols - 1), b = o >> (cl_log2 + 2);
        const uint32_t jc = tile * cols + jl;
        if (jc >= m) continue;
        float v = red[b * cols + jl];
        for (uint32_t q = 1; q < groups; ++q) v += red[(q * SB_NB + b) * cols + jl];
        if (splits == 1) Y[(uint64_t)(b0 + b) * ldy + jc] = v;
        else part[((uint64_t)split * B + b0 + b) * m + jc] = v;
    }
}

// Y = part[0] + part[1] + ... in that order (bitwise reproducible).
__global__ void __launch_bounds__(256)
splitk_reduce_kernel(const float* __restrict__ part, uint32_t splits, uint32_t B, uint32_t m,
                     float* __restrict__ Y, uint64_t ldy)
{
    const uint64_t total = (uint64_t)B * m;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        float v = part[i];
        uint32_t s = 1;
        for (; s + 3 < splits; s += 4) {                   // four loads in flight, added in order
            const float a = part[(uint64_t)s * total + i], b = part[(uint64_t)(s + 1) * total + i];
            const float c = part[(uint64_t)(s + 2) * total + i], d = part[(uint64_t)(s + 3) * total + i];
            v += a; v += b; v += c; v += d;
        }
        for (; s < splits; ++s) v += part[(uint64_t)s * total + i];
        const uint64_t row = i / m;
        Y[row * ldy + (i - row * m)] = v;
    }
}

} // namespace

namespace hac_internal {

static size_t index_gemm_lds_bytes(uint32_t k_tot, uint32_t idx_bits, int rt)
{
    return (size_t)(idx_bits == 8 ? tile_bytes<uint8_t>(rt) : tile_bytes<uint16_t>(rt)) + (k_tot <= kLutLdsMax ? sizeof(uint2) * k_tot : 0);
}

GemmPlan plan_index_gemm(uint32_t B, uint32_t n, uint32_t m, size_t room)
{
    GemmPlan p;
    p.us = 0.0;
    p.small = B <= 4u * SB_NB;
    if (p.small) {
        // blocks of 256 columns x a range of rows: about 512 blocks, at most 32 ranges (the pass that
        // adds them walks them one after the other) unless the rows of a range would not fit LDS
        // column lanes per row group: 64 (256 columns a block) from 129 columns on, else the power of
        // two that covers the map, at least 4 (p.rt carries its logarithm in this mode)
        uint32_t cl_log2 = 6;
        if (m <= 128) { cl_log2 = 2; while ((4u << cl_log2) < m) ++cl_log2; }
        const uint32_t tiles_m = (m + (4u << cl_log2) - 1) / (4u << cl_log2);
        const uint32_t groups = (B + SB_NB - 1) / SB_NB;
        uint32_t splits = (512 + tiles_m * groups - 1) / (tiles_m * groups);
        const uint32_t most = (n + 31) / 32, least = (n + kSmallMaxRows - 1) / kSmallMaxRows;
        if (splits > 32) splits = 32;
        if (splits > most) splits = most;
        if (splits < least) splits = least;
        if (splits < 1) splits = 1;
        p.steps_per_split = ((n + splits - 1) / splits + 3) / 4 * 4;          // rows per block
        p.splits = (n + p.steps_per_split - 1) / p.steps_per_split;
        p.steps = n; p.rt = cl_log2; p.tiles = tiles_m;
        p.part_bytes = p.splits > 1 ? (size_t)p.splits * B * m * sizeof(float) : 0;
        return p;
    }
    const uint32_t tiles_n = (m + BN - 1) / BN;
    const uint32_t steps = (n + BK - 1) / BK;
    // Row tiles per block and K splits: the pair with the shortest estimate.  A step of 32 k takes a block 0.77 + 0.26 us
    // per row tile when little else runs on its CU, and every block of a CU adds 0.22 + 0.25 us per row tile of its
    // shared pipes, counting 4 blocks of one or two row tiles, 3 of three and 2 of four.  The pass that adds the splits
    // takes 3 us and 0.4 us per MB of partial tiles, everything else 5 us.  The constants are fitted to 625 measured
    // pairs of 21 shapes (64 x 100 to 25088 x 1000, 33 to 12544 rows, 4 to 4000 work items): four in five estimates lie
    // within 8 % of the time, and the pairs they choose within 6 % of the best measured one (one shape: within 20 %).  They are those of
    // the kernel that kept W's parts in LDS: the K splits they choose set the order of the sums, which stays; for the same
    // splits the row tiles they choose are within 5 % of the best on 15 of 18 shapes (64 x 25088 x 1000 9 %).
    // Relative 2-norm error against 64 bits, fp32 instruction -> bf16 parts: one term 2.4e-8 -> 2.5e-8, two 3.4e-8 ->
    // 3.2e-8, 64 terms 1.05e-7 -> 4.0e-8, 4608 terms 1.9e-7 -> 9.9e-8 (X as after a ReLU, one K split).
    static const uint32_t kSplits[] = { 1, 2, 3, 4, 6, 8, 10, 12, 16, 20, 24, 32 };
    double best = 1e300;
    for (uint32_t rt = kMinRT; rt <= kMaxRT; ++rt) {
        const uint64_t tiles = (uint64_t)((B + 32 * rt - 1) / (32 * rt)) * tiles_n;
        const uint64_t fit = rt <= 2 ? 4 : 6 - rt;                        // blocks on a CU
        const double alone = 0.77 + 0.26 * rt, shared = 0.22 + 0.25 * rt;
        for (uint32_t splits : kSplits) {
            if (splits > 1 && (splits > steps / 4 || (uint64_t)splits * B * m * sizeof(float) > room)) break;
            const uint32_t per = (steps + splits - 1) / splits;
            const uint32_t parts = (steps + per - 1) / per;               // no empty split
            const uint64_t on_cu = (tiles * parts + 255) / 256, full = on_cu / fit, rest = on_cu - full * fit;
            double us = 5.2 + per * ((double)full * std::max(alone, shared * (double)fit) +
                                     (rest ? std::max(alone, shared * (double)rest) : 0.0));
            if (parts > 1) us += 3.0 + 1.64e-6 * (double)parts * B * m;
            // (for the choice a second launch counts 3 us more: a caller that launches as it goes waits for the host there.
            // 60 x 308 x 59: two splits 10.6 us in a graph, 14.4 called one by one; one split 12.5 and 12.3)
            const double cost = us + (parts > 1 ? 3.0 : 0.0);
            if (cost < best) { best = cost; p.us = us; p.rt = rt; p.tiles = tiles; p.splits = parts; p.steps_per_split = per; }
        }
    }
    // More groups of rows than the fewest that p.rt row tiles a block allow, some blocks with a row tile less, where that fills places
    // on the CUs that stay empty otherwise.  A step takes a CU 0.17 us for each of its blocks and 0.27 us for each of their row
    // tiles (fitted to 794 measured plans of 18 shapes); the groups have to save 3 % of that.  784 x 4608 x 512 in 12 splits, 9
    // groups -> 10: 38.3 -> 35.4 us; 12544 rows, 98 -> 128: 319 -> 317; but 2048 x 2000 x 2000, 32 -> 48 (a third block on a CU): 93 -> 104.
    // K splits, and with them the sums, stay the same.
    const uint64_t row_tiles = (B + 31) / 32, groups = p.tiles / tiles_n, per_group = (uint64_t)tiles_n * p.splits;
    const uint64_t places = 256 * (p.rt == 1 ? 4 : p.rt == 2 ? 3 : 2);
    if (p.rt > 1) {
        const uint64_t more = std::min((groups * per_group + places - 1) / places * places / per_group, row_tiles / (p.rt - 1));
        auto cu_us = [&](uint64_t g, double tiles) { return (double)((g * per_group + 255) / 256) * (0.17 + 0.27 * tiles); };
        if (more > groups && cu_us(more, (double)row_tiles / (double)more) < 0.97 * cu_us(groups, (double)p.rt)) p.tiles = tiles_n * more;
    }
    p.part_bytes = p.splits > 1 ? (size_t)p.splits * B * m * sizeof(float) : 0;
    p.steps = steps;
    return p;
}

namespace {

typedef void (*gemm_kern_t)(const float*, uint64_t, uint32_t, const void*, uint64_t, const float*, uint32_t, uint32_t,
                            uint32_t, uint32_t, float*, uint64_t, uint32_t, uint32_t, uint32_t, uint32_t, float*);

template <typename IdxT, bool LUT_LDS, int RT>
void launch_one(dim3 grid, size_t lds, hipStream_t stream, hipError_t& err,
                const float* d_X, uint64_t ldx, uint32_t B, const void* d_idx, uint64_t pitch, const float* d_codebook,
                uint32_t k_sym, uint32_t zero_first, uint32_t n, uint32_t m, float* d_Y, uint64_t ldy, uint32_t tiles_n,
                uint32_t row_groups, uint32_t splits, uint32_t steps_per_split, float* d_part)
{
    auto k = index_gemm_kernel<IdxT, LUT_LDS, RT>;
    if (lds > 63 * 1024) {                             // (the votes take some of the 64 KB a kernel gets without asking)
        err = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (err != hipSuccess) return;
    }
    hipLaunchKernelGGL(k, grid, dim3(256), lds, stream, d_X, ldx, B, static_cast<const IdxT*>(d_idx), pitch, d_codebook,
                       k_sym, zero_first, n, m, d_Y, ldy, tiles_n, row_groups, splits, steps_per_split, d_part);
    note_kernel("index_gemm_kernel<unsigned %s, %s, %d>", sizeof(IdxT) == 1 ? "char" : "short", LUT_LDS ? "true" : "false", RT);
    err = hipGetLastError();
}

template <typename IdxT, bool LUT_LDS, typename... Args>
void launch_rt(uint32_t rt, Args&&... args)
{
    switch (rt) {
    case 1: launch_one<IdxT, LUT_LDS, 1>(args...); break;
    case 2: launch_one<IdxT, LUT_LDS, 2>(args...); break;
    case 3: launch_one<IdxT, LUT_LDS, 3>(args...); break;
    default: launch_one<IdxT, LUT_LDS, 4>(args...); break;
    }
}

} // namespace

hipError_t launch_index_gemm(const GemmPlan& plan, const float* d_X, uint64_t ldx, uint32_t B, const void* d_idx, uint32_t idx_bits,
                             uint64_t pitch, const float* d_codebook, uint32_t k_sym, uint32_t zero_first,
                             uint32_t n, uint32_t m, float* d_Y, uint64_t ldy, float* d_part, hipStream_t stream)
{
    const uint32_t tiles_n = (m + BN - 1) / BN;
    if (plan.small) {
        if (plan.splits > 1 && !d_part) return hipErrorInvalidValue;
        if (idx_bits != 8 && idx_bits != 16) return hipErrorInvalidValue;
        const uint64_t blocks = plan.tiles * plan.splits;
        if (blocks > 0x7ffffff0ull) return hipErrorInvalidValue;
        const uint32_t k_tot = k_sym + zero_first;
        const bool lut_lds = k_tot <= kLutLdsMax;
        const size_t lds = sizeof(float) * ((size_t)plan.steps_per_split * SB_NB + SB_GROUPS * SB_NB * SB_COLS + (lut_lds ? k_tot : 0));
        if (lds > 160 * 1024) return hipErrorInvalidValue;           // (the plan keeps a range at kSmallMaxRows rows: 32 + 64 + 16 KB at most)
        const dim3 grid((uint32_t)blocks, (B + SB_NB - 1) / SB_NB);
        // (the rows of a range, the partial sums of the row groups and the table can exceed the 64 KB a
        // kernel gets without asking)
        hipError_t attr = hipSuccess;
        auto launch_small = [&](auto kern, auto idxp) {
            if (lds > 64 * 1024) {
                attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
                if (attr != hipSuccess) return;
            }
            hipLaunchKernelGGL(kern, grid, dim3(256), lds, stream, d_X, ldx, B,
                               idxp, pitch, d_codebook, k_sym, zero_first, n, m,
                               plan.steps_per_split, (uint32_t)plan.tiles, plan.splits, plan.rt, d_Y, ldy, d_part);
            note_kernel("index_small_kernel<unsigned %s, %s, %s>", idx_bits == 8 ? "char" : "short", lut_lds ? "true" : "false",
                        plan.rt == 6 ? "true" : "false");
        };
        const bool narrow = plan.rt == 6;
        const uint8_t* i8 = static_cast<const uint8_t*>(d_idx);
        const uint16_t* i16 = static_cast<const uint16_t*>(d_idx);
        if (idx_bits == 8) {
            if (lut_lds) { if (narrow) launch_small(index_small_kernel<uint8_t, true, true>, i8); else launch_small(index_small_kernel<uint8_t, true, false>, i8); }
            else { if (narrow) launch_small(index_small_kernel<uint8_t, false, true>, i8); else launch_small(index_small_kernel<uint8_t, false, false>, i8); }
        } else {
            if (lut_lds) { if (narrow) launch_small(index_small_kernel<uint16_t, true, true>, i16); else launch_small(index_small_kernel<uint16_t, true, false>, i16); }
            else { if (narrow) launch_small(index_small_kernel<uint16_t, false, true>, i16); else launch_small(index_small_kernel<uint16_t, false, false>, i16); }
        }
        if (attr != hipSuccess) return attr;
        hipError_t e = hipGetLastError();
        if (e != hipSuccess || plan.splits == 1) return e;
        const uint64_t total = (uint64_t)B * m;
        const uint32_t rgrid = (uint32_t)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
        hipLaunchKernelGGL(splitk_reduce_kernel, dim3(rgrid), dim3(256), 0, stream, d_part, plan.splits, B, m, d_Y, ldy);
        note_kernel("splitk_reduce_kernel");
        return hipGetLastError();
    }
    if (plan.tiles > 0x7ffffff0ull) return hipErrorInvalidValue;
    if (plan.splits > 1 && !d_part) return hipErrorInvalidValue;
    if (idx_bits != 8 && idx_bits != 16) return hipErrorInvalidValue;
    const uint32_t k_tot = k_sym + zero_first;
    const bool lut_lds = k_tot <= kLutLdsMax;
    // a long value list (from 1021 values on at four row tiles and 16-bit pointers) leaves a CU room for one block only: a row
    // tile less then, down to two
    uint32_t rt = plan.rt, row_groups = (uint32_t)(plan.tiles / tiles_n);
    while (rt > 2 && 2 * (index_gemm_lds_bytes(k_tot, idx_bits, (int)rt) + 64) > 160 * 1024) --rt;
    row_groups = std::max(row_groups, ((B + 31) / 32 + rt - 1) / rt);
    const uint64_t items64 = (uint64_t)row_groups * tiles_n * plan.splits;
    if (items64 > 0x7ffffff0ull) return hipErrorInvalidValue;
    const dim3 grid(((uint32_t)items64 + 7) / 8 * 8);
    const size_t lds = index_gemm_lds_bytes(k_tot, idx_bits, (int)rt);
    hipError_t e = hipSuccess;
    if (idx_bits == 8) {
        if (lut_lds) launch_rt<uint8_t, true>(rt, grid, lds, stream, e, d_X, ldx, B, d_idx, pitch, d_codebook, k_sym, zero_first,
                                              n, m, d_Y, ldy, tiles_n, row_groups, plan.splits, plan.steps_per_split, d_part);
        else launch_rt<uint8_t, false>(rt, grid, lds, stream, e, d_X, ldx, B, d_idx, pitch, d_codebook, k_sym, zero_first,
                                       n, m, d_Y, ldy, tiles_n, row_groups, plan.splits, plan.steps_per_split, d_part);
    } else {
        if (lut_lds) launch_rt<uint16_t, true>(rt, grid, lds, stream, e, d_X, ldx, B, d_idx, pitch, d_codebook, k_sym, zero_first,
                                               n, m, d_Y, ldy, tiles_n, row_groups, plan.splits, plan.steps_per_split, d_part);
        else launch_rt<uint16_t, false>(rt, grid, lds, stream, e, d_X, ldx, B, d_idx, pitch, d_codebook, k_sym, zero_first,
                                        n, m, d_Y, ldy, tiles_n, row_groups, plan.splits, plan.steps_per_split, d_part);
    }
    if (e != hipSuccess || plan.splits == 1) return e;
    const uint64_t total = (uint64_t)B * m;
    const uint32_t rgrid = (uint32_t)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3(rgrid), dim3(256), 0, stream, d_part, plan.splits, B, m, d_Y, ldy);
    note_kernel("splitk_reduce_kernel");
    return hipGetLastError();
}

} // namespace hac_internal
