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
// Tiling: a block of 4 wavefronts owns 32 RT batch rows x 128 columns of Y (RT = 1..4) and walks K = n
// in steps of 32; wavefront w owns the 32 columns [32 w, 32 w + 32) of the tile and all its rows, as RT
// MFMA tiles (two sums each, 32 RT accumulator registers).  LDS holds one K step of X and W, both with the 32 k of a
// row (a column) side by side, part by part, 208 bytes apart, so that an operand is one 128-bit read and 16
// lanes' reads fall on different banks.  The next step's global loads fly during the matrix
// instructions; two blocks share a CU, so that one splits and stores while the other multiplies.
// Measured (MI355X), fp32 instruction -> bf16 parts: 4608 x 512 layer pruned 60 %, 12544 rows, whole call
// 580 -> 351 us (59 GFLOP; a call includes decoding the stream, about 25 us); unpruned map of that size,
// 784 rows, 60.0 -> 37.4 us.  Matrix pipes 44 % busy at 12544 rows, four vector instructions beside each matrix one.
// Lane layout of v_mfma_f32_32x32x16_bf16: A operand lane l holds A[i = l % 32][k = 8 (l / 32) + 0..7], B
// operand lane l holds B[k = 8 (l / 32) + 0..7][j = l % 32], accumulator register v of lane l is
// D[(v % 4) + 8 (v / 4) + 4 (l / 32)][l % 32].
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "hac_internal.h"

namespace {

constexpr int BN = 128, BK = 32;
constexpr int PART = 2 * BK, PITCH = 3 * PART + 16;   // bytes: one part of a row's K step, one row in LDS
constexpr uint32_t kMinRT = 1, kMaxRT = 4;              // row tiles of 32 per block
constexpr uint32_t kLutLdsMax = 4096;              // representatives kept in LDS

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Four neighbouring pointers of one row of the map.
template <typename IdxT> struct Ptr4;
template <> struct Ptr4<uint8_t> {
    typedef uint32_t raw;
    static __device__ __forceinline__ uint32_t get(raw w, int c) { return (w >> (8 * c)) & 255u; }
    static __device__ __forceinline__ void ld(const uint8_t* p, uint32_t* out) {
        const uint32_t w = *reinterpret_cast<const uint32_t*>(p);
        out[0] = w & 255u; out[1] = (w >> 8) & 255u; out[2] = (w >> 16) & 255u; out[3] = w >> 24;
    }
};
template <> struct Ptr4<uint16_t> {
    typedef uint2 raw;
    static __device__ __forceinline__ uint32_t get(raw w, int c) { return ((c & 2 ? w.y : w.x) >> (16 * (c & 1))) & 65535u; }
    static __device__ __forceinline__ void ld(const uint16_t* p, uint32_t* out) {
        const uint2 w = *reinterpret_cast<const uint2*>(p);
        out[0] = w.x & 65535u; out[1] = w.x >> 16; out[2] = w.y & 65535u; out[3] = w.y >> 16;
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
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t two_bf16(f32x2 v) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2)); }   // to nearest even
__device__ __forceinline__ f32x2 two_f32(uint32_t p) { return f32x2{__uint_as_float(p << 16), __uint_as_float(p & 0xffff0000u)}; }

__device__ __forceinline__ uint32_t logical_tile(uint32_t tiles_padded)
{
    // consecutive logical tiles on one XCD: the column tiles of a row tile share X rows in that L2
    const uint32_t per = tiles_padded >> 3;
    return (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
}

// (blocks per CU: as many as the LDS of a K step lets in for 2 to 4 row tiles; left to itself the compiler spends
// registers on the fp32 pass and one block fewer fits)
template <typename IdxT, bool LUT_LDS, int RT, bool XVEC>
__global__ void __launch_bounds__(256, RT == 4 ? 2 : RT == 3 ? 3 : 4)
index_gemm_kernel(const float* __restrict__ X, uint64_t ldx, uint32_t B,
                  const IdxT* __restrict__ idx, uint64_t pitch,          // pitch in elements, a multiple of 16
                  const float* __restrict__ codebook, uint32_t k_sym, uint32_t zero_first,
                  uint32_t n, uint32_t m, float* __restrict__ Y, uint64_t ldy,
                  uint32_t tiles_n, uint32_t tiles, uint32_t x_vec,
                  uint32_t splits, uint32_t steps_per_split, float* __restrict__ part)
{
    constexpr int BM = 32 * RT;
    extern __shared__ __align__(16) float lds[];
    char* As = reinterpret_cast<char*>(lds);           // [BM] rows of PITCH bytes
    char* Bs = As + BM * PITCH;                        // [BN] columns of PITCH bytes
    uint2* lut = reinterpret_cast<uint2*>(Bs + BN * PITCH);   // [k_sym + zero_first] when LUT_LDS
    // work item = (tile, K split); with more than one split a block writes its partial tile to
    // part[split][B][m] and a second kernel adds the splits in order
    const uint32_t item = logical_tile(gridDim.x);
    if (item >= tiles * splits) return;
    const uint32_t tile = item / splits, split = item - tile * splits;
    const uint32_t tm = tile / tiles_n, tn = tile - tm * tiles_n;
    const uint32_t m0 = tm * BM, n0 = tn * BN;
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const uint32_t l32 = lane & 31, half = lane >> 5;

    // pointer -> value; entry 0 is 0.0 when the pointers were written with an offset of one
    const uint32_t k_tot = k_sym + zero_first;
    auto value_of = [&](uint32_t p) -> float { return (zero_first && p == 0) ? 0.0f : codebook[p - zero_first]; };
    uint32_t cut = 0;                                  // lower half not 0: some operand is more than its three parts
    auto parts_of = [&](uint32_t p) -> uint2 { return LUT_LDS ? lut[p] : split_weight(value_of(p), cut); };

    // Global -> registers.  X: rows a_row + 32 r, k = 4 q .. 4 q + 3; map: rows 4 q .. 4 q + 3, columns
    // b_col .. b_col + 3 (four k of a column in one thread, so that a part of them is one 64-bit store).
    // Rows past B and columns past the pitch are read from a clamped, valid address and never stored;
    // only the last, partial K step is guarded.
    struct Stage { float4 ra[RT]; typename Ptr4<IdxT>::raw rb[4]; };
    const uint32_t q = t & 7, a_row = t >> 3, b_col = 4 * (t >> 3);
    const float* xrow[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const uint32_t row = m0 + a_row + 32 * r;
        xrow[r] = X + (uint64_t)(row < B ? row : B - 1) * ldx + 4 * q;
    }
    const IdxT* icol = idx + (n0 + b_col < pitch ? n0 + b_col : 0);
    auto load_full = [&](uint32_t k0, Stage& st) {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const float* p = xrow[r] + k0;
            if (XVEC) st.ra[r] = *reinterpret_cast<const float4*>(p);
            else st.ra[r] = make_float4(p[0], p[1], p[2], p[3]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            st.rb[j] = *reinterpret_cast<const typename Ptr4<IdxT>::raw*>(icol + (uint64_t)(k0 + 4 * q + j) * pitch);
    };
    auto load_tail = [&](uint32_t k0, Stage& st) {
        const uint32_t k = k0 + 4 * q;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const float* p = xrow[r] + k0;
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (k < n) v.x = p[0];
            if (k + 1 < n) v.y = p[1];
            if (k + 2 < n) v.z = p[2];
            if (k + 3 < n) v.w = p[3];
            st.ra[r] = v;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {                  // (past the end: any row of the map, X is 0 there)
            const uint32_t kj = k + j < n ? k + j : n - 1;
            st.rb[j] = *reinterpret_cast<const typename Ptr4<IdxT>::raw*>(icol + (uint64_t)kj * pitch);
        }
    };
    // registers -> LDS.  __builtin_amdgcn_perm(hi, lo, ..) packs the upper (lower) halves of two words.
    auto upper = [](uint32_t hi, uint32_t lo) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); };
    auto lower = [](uint32_t hi, uint32_t lo) { return __builtin_amdgcn_perm(hi, lo, 0x05040100u); };
    auto store = [&](const Stage& st) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            uint2 w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = parts_of(Ptr4<IdxT>::get(st.rb[j], c));
            char* b = Bs + (b_col + c) * PITCH + 8 * q;
            *reinterpret_cast<uint2*>(b) = make_uint2(lower(w[1].x, w[0].x), lower(w[3].x, w[2].x));
            *reinterpret_cast<uint2*>(b + PART) = make_uint2(upper(w[1].x, w[0].x), upper(w[3].x, w[2].x));
            *reinterpret_cast<uint2*>(b + 2 * PART) = make_uint2(lower(w[1].y, w[0].y), lower(w[3].y, w[2].y));
        }
#pragma unroll
        for (int r = 0; r < RT; ++r) {
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
                // (a three-operand OR; from plain C the compiler reorders the whole step around it: 336 -> 359 us at
                // 4608 x 512, 12544 rows)
                asm("v_or3_b32 %0, %1, %2, %0" : "+v"(cut) : "v"(r2.x), "v"(r2.y));
            }
            char* a = As + (a_row + 32 * r) * PITCH + 8 * q;
            *reinterpret_cast<uint2*>(a) = make_uint2(p1[0], p1[1]);
            *reinterpret_cast<uint2*>(a + PART) = make_uint2(p2[0], p2[1]);
            *reinterpret_cast<uint2*>(a + 2 * PART) = make_uint2(p3[0], p3[1]);
        }
    };

    // x1 w1 has a sum of its own: the instruction rounds a sum once per 16 k, and the five others, 2^-8 of it
    // and less, would each round the large sum again (one sum for all six:
    // 5.8 times the error at 4608 x 512, 12544 rows, and 1.6 times that of the fp32 instruction)
    f32x16 acc[RT], low[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = low[i][v] = 0.0f;

    auto multiply = [&]() {
        const char* a = As + l32 * PITCH + 16 * half;
        const char* b = Bs + (wave * 32 + l32) * PITCH + 16 * half;
#pragma unroll
        for (int h = 0; h < 2; ++h) {                  // 16 k each
            bf16x8 w[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) w[p] = *reinterpret_cast<const bf16x8*>(b + p * PART + 32 * h);
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                bf16x8 x[3];
#pragma unroll
                for (int p = 0; p < 3; ++p) x[p] = *reinterpret_cast<const bf16x8*>(a + 32 * i * PITCH + p * PART + 32 * h);
                low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[2], w[0], low[i], 0, 0, 0);
                low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], w[2], low[i], 0, 0, 0);
                low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[1], w[1], low[i], 0, 0, 0);
                low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[1], w[0], low[i], 0, 0, 0);
                low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], w[1], low[i], 0, 0, 0);
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], w[0], acc[i], 0, 0, 0);
            }
        }
    };

    const uint32_t all_steps = (n + BK - 1) / BK;
    const uint32_t kt0 = split * steps_per_split;
    const uint32_t ksteps = kt0 + steps_per_split < all_steps ? kt0 + steps_per_split : all_steps;   // one past the last
    const uint32_t nfull = n / BK;
    Stage st;
    auto load = [&](uint32_t kt) { if (kt < nfull) load_full(kt * BK, st); else load_tail(kt * BK, st); };
    // true if f holds for any thread of the block: a word per wavefront and a barrier (0.3 us less per vote than
    // __syncthreads_or); every vote has words of its own
    __shared__ uint32_t votes[2][4];
    auto block_any = [&](bool f, int which) -> bool {
        const bool mine = __any(f);
        if (lane == 0) votes[which][wave] = mine ? 1u : 0u;
        __syncthreads();
        return (votes[which][0] | votes[which][1] | votes[which][2] | votes[which][3]) != 0;
    };
    // an operand was cut short, or a sum is not finite (an infinity or NaN among the operands, or an overflow)
    // (x * 0 is NaN exactly then: one instruction per sum; a comparison each took 0.2 us a block)
    auto unfit = [&]() -> bool {
        float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) t[v & 3] = fmaf(acc[i][v] + low[i][v], 0.0f, t[v & 3]);
        return (cut & 0xffffu) != 0 || !((t[0] + t[1]) + (t[2] + t[3]) == 0.0f);
    };
    // a look at some of the first step's X (non-finite, or small enough to be cut) and at the table: where all of X, or a
    // representative, is like this, parts are not tried first
    load(kt0);                                         // (in flight while the table is made)
    if (LUT_LDS)
        for (uint32_t i = t; i < k_tot; i += 256) lut[i] = split_weight(value_of(i), cut);
    bool again = (cut & 0xffffu) != 0 || n == 1;
    const float seen[4] = {st.ra[0].x, st.ra[0].y, st.ra[0].z, st.ra[0].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) again |= !(fabsf(seen[j]) <= 3.402823466e38f) || (seen[j] != 0.0f && fabsf(seen[j]) < 0x1p-110f);
    again = block_any(again, 0);                       // (a barrier: the table is complete)
    for (uint32_t kt = again ? ksteps : kt0; kt < ksteps; ++kt) {
        __syncthreads();                               // the last step's tiles are read
        store(st);
        __syncthreads();
        if (kt + 1 < ksteps) load(kt + 1);
        multiply();
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
        static_assert(4 * P32 <= PITCH, "the fp32 tiles take the place of the parts");
        float* Af = reinterpret_cast<float*>(As);
        float* Bf = reinterpret_cast<float*>(Bs);
        if (LUT_LDS)
            for (uint32_t i = t; i < k_tot; i += 256) lut[i].x = __float_as_uint(value_of(i));   // (the vote was a barrier)
        auto fp32_of = [&](uint32_t p) -> float { return LUT_LDS ? __uint_as_float(lut[p].x) : value_of(p); };
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
            for (int r = 0; r < RT; ++r) *reinterpret_cast<float4*>(Af + (a_row + 32 * r) * P32 + 4 * q) = st.ra[r];
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
            if (row < B && col < m) {
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

static size_t index_gemm_lds_bytes(uint32_t k_tot, int rt)
{
    return (size_t)(32 * rt + BN) * PITCH + (k_tot <= kLutLdsMax ? sizeof(uint2) * k_tot : 0);
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
    // shared pipes; 4 blocks of one or two row tiles, 3 of three and 2 of four fit.  The pass that adds the splits
    // takes 3 us and 0.4 us per MB of partial tiles, everything else 5 us.  The constants are fitted to 625 measured
    // pairs of 21 shapes (64 x 100 to 25088 x 1000, 33 to 12544 rows, 4 to 4000 work items): four in five estimates lie
    // within 8 % of the time, and the pairs they choose within 6 % of the best measured one (one shape: within 20 %).
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
    p.part_bytes = p.splits > 1 ? (size_t)p.splits * B * m * sizeof(float) : 0;
    p.steps = steps;
    return p;
}

namespace {

typedef void (*gemm_kern_t)(const float*, uint64_t, uint32_t, const void*, uint64_t, const float*, uint32_t, uint32_t,
                            uint32_t, uint32_t, float*, uint64_t, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t, float*);

template <typename IdxT, bool LUT_LDS, int RT>
void launch_one(dim3 grid, size_t lds, hipStream_t stream, hipError_t& err,
                const float* d_X, uint64_t ldx, uint32_t B, const void* d_idx, uint64_t pitch, const float* d_codebook,
                uint32_t k_sym, uint32_t zero_first, uint32_t n, uint32_t m, float* d_Y, uint64_t ldy, uint32_t tiles_n,
                uint32_t tiles, uint32_t x_vec, uint32_t splits, uint32_t steps_per_split, float* d_part)
{
    auto k = x_vec ? index_gemm_kernel<IdxT, LUT_LDS, RT, true> : index_gemm_kernel<IdxT, LUT_LDS, RT, false>;
    if (lds > 63 * 1024) {                             // (the votes take some of the 64 KB a kernel gets without asking)
        err = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (err != hipSuccess) return;
    }
    hipLaunchKernelGGL(k, grid, dim3(256), lds, stream, d_X, ldx, B, static_cast<const IdxT*>(d_idx), pitch, d_codebook,
                       k_sym, zero_first, n, m, d_Y, ldy, tiles_n, tiles, x_vec, splits, steps_per_split, d_part);
    note_kernel("index_gemm_kernel<unsigned %s, %s, %d, %s>", sizeof(IdxT) == 1 ? "char" : "short", LUT_LDS ? "true" : "false", RT,
                x_vec ? "true" : "false");
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
    const uint64_t items64 = plan.tiles * plan.splits;
    if (items64 > 0x7ffffff0ull) return hipErrorInvalidValue;
    if (plan.splits > 1 && !d_part) return hipErrorInvalidValue;
    if (idx_bits != 8 && idx_bits != 16) return hipErrorInvalidValue;
    const uint32_t tiles = (uint32_t)plan.tiles;
    const dim3 grid(((uint32_t)items64 + 7) / 8 * 8);
    const uint32_t k_tot = k_sym + zero_first;
    const bool lut_lds = k_tot <= kLutLdsMax;
    const size_t lds = index_gemm_lds_bytes(k_tot, (int)plan.rt);
    const uint32_t x_vec = (reinterpret_cast<uintptr_t>(d_X) % 16 == 0 && ldx % 4 == 0) ? 1u : 0u;
    hipError_t e = hipSuccess;
    if (idx_bits == 8) {
        if (lut_lds) launch_rt<uint8_t, true>(plan.rt, grid, lds, stream, e, d_X, ldx, B, d_idx, pitch, d_codebook, k_sym, zero_first,
                                              n, m, d_Y, ldy, tiles_n, tiles, x_vec, plan.splits, plan.steps_per_split, d_part);
        else launch_rt<uint8_t, false>(plan.rt, grid, lds, stream, e, d_X, ldx, B, d_idx, pitch, d_codebook, k_sym, zero_first,
                                       n, m, d_Y, ldy, tiles_n, tiles, x_vec, plan.splits, plan.steps_per_split, d_part);
    } else {
        if (lut_lds) launch_rt<uint16_t, true>(plan.rt, grid, lds, stream, e, d_X, ldx, B, d_idx, pitch, d_codebook, k_sym, zero_first,
                                               n, m, d_Y, ldy, tiles_n, tiles, x_vec, plan.splits, plan.steps_per_split, d_part);
        else launch_rt<uint16_t, false>(plan.rt, grid, lds, stream, e, d_X, ldx, B, d_idx, pitch, d_codebook, k_sym, zero_first,
                                        n, m, d_Y, ldy, tiles_n, tiles, x_vec, plan.splits, plan.steps_per_split, d_part);
    }
    if (e != hipSuccess || plan.splits == 1) return e;
    const uint64_t total = (uint64_t)B * m;
    const uint32_t rgrid = (uint32_t)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3(rgrid), dim3(256), 0, stream, d_part, plan.splits, B, m, d_Y, ldy);
    note_kernel("splitk_reduce_kernel");
    return hipGetLastError();
}

} // namespace hac_internal
