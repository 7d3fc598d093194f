// Batch kernel of libhac for matrices of few or long columns (gfx950): Y = X.W for 2 rows of X or more, with
// several wavefronts on one column of W.  Included by hac_kernels.hip only.
//
// dot_batch_kernel gives a column to one wavefront.  With 4096 columns that fills the 256 CUs with 16 wavefronts
// each; with 1000 columns, or 10, a wavefront walks its column's list alone, a row of X per lane group and turn, and
// what the product takes is the latency of those turns (4096 x 1000, 10 % non-zero, 64 rows: 10 of 14.6 us) while
// most of the chip idles.  Here a block of `waves` wavefronts owns `cols` columns, waves / cols of them on each:
//   staging : the words of the block's columns follow one another in the stream (and in ri), so all threads copy them;
//   decode  : the chunks of the block's columns are dealt to its wavefronts, at least 16 to one; the non-zeros go to one
//             list in LDS, in CSC order, and the ri fields are unpacked beside it by all threads;
//   multiply: the wavefronts of a column share its part of the list.  Two ways:
//     rows of the re-laid-out X (NBD = 0): a lane group fetches the row of a non-zero, 4 batch columns a lane, from the
//             feature-major copy XT; groups take entries in turn;
//     X as it is (NBD = 4, 8, 16, 24 or 32, the batch columns of a block): a lane takes a non-zero and fetches one value of each of
//             the block's rows of X.  Neighbouring lanes hold neighbouring rows of W, so that at the densities where
//             columns are long a wavefront's fetch touches few lines, and no copy of X is written first: a launch
//             less, which for small products is a third of the call (blocks behind those of the product leave the copy
//             all the same, for a later call with HAC_LAUNCH_REUSE_XT);
//   sums    : over the lanes of a wavefront, then over a column's wavefronts through LDS, always in the same order; in 64 bits,
//             but for the first of the lanes' where X is read as it is, and for the lanes' where columns are long (kTurns).
// Measured (MI355X, kernels back to back), one wavefront per column -> this kernel: 500 x 300, 30 % non-zero, 8 rows 8.3 -> 5.5 us;
// 4096 x 1000, 10 %, 64 rows 18.4 -> 13.2; 9973 x 1511, 7 %, 37 rows 26.6 -> 21.6; 21516 x 34, 34 %, 19 rows 161 -> 65;
// 4718 x 12, 6 %, 41 rows 16.7 -> 7.4.  What is left of the small ones is a launch, two trips to memory and the chain of one
// chunk's codewords.
// A block covers the batch columns of one tile; tiles are blocks of their own, each decodes its columns again (with few
// columns the CUs that do it have nothing else to do).
#ifndef HAC_SPLIT_H
#define HAC_SPLIT_H

namespace {

struct SplitParams {
    uint32_t waves, cols;                    // per block; cols divides waves
    uint32_t cols_log2, split_log2;          // of cols, of waves / cols
    uint32_t width;                          // batch columns of a tile (NBD, or those of a pass over XT)
    uint32_t nblocks;                        // blocks per tile
    uint32_t tiles;
    uint32_t copies;                         // blocks behind those of the product, which leave the copy of X
    uint32_t sbuf_words;                     // staged stream and ri words; the sums of the wavefronts take their place
    uint32_t list_cap;                       // non-zeros of a block's columns
};

// Copy 16-byte pieces [0, n4) with all threads of the block: the first two of a thread are requested by
// request_pieces, stored by finish_pieces, which copies the rest.  Addresses are clamped, so that the loads are on every path.
struct PieceRegs { uint4 v[2]; };

__device__ __forceinline__ void request_pieces(PieceRegs& p, const uint4* src, uint32_t n4)
{
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint32_t i = threadIdx.x + k * blockDim.x;
        p.v[k] = src[i < n4 ? i : n4 - 1u];
    }
}

__device__ __forceinline__ void finish_pieces(PieceRegs& p, uint4* dst, const uint4* src, uint32_t n4)
{
    asm volatile("" : HAC_PIN_U4(p.v[0]), HAC_PIN_U4(p.v[1]));
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint32_t i = threadIdx.x + k * blockDim.x;
        if (i < n4) dst[i] = p.v[k];
    }
    for (uint32_t i = threadIdx.x + 2 * blockDim.x; i < n4; i += blockDim.x) dst[i] = src[i];
}

// The feature-major copy of X (panels of w batch columns) by the blocks behind the first `before`: a thread reads one feature
// of a panel's rows of X (neighbouring lanes neighbouring features) and writes a row of the panel, up to a whole line; four
// columns a thread, so that eight threads share a line, took 0.2 us more.  They run beside the product's own blocks, which
// are few where X is read as it is.
__device__ __forceinline__ void leave_copy(uint32_t before, const float* __restrict__ X, uint64_t ldx, uint32_t B, uint32_t n,
                                           float* __restrict__ XT, uint32_t w)
{
    const uint32_t u = (blockIdx.x - before) * blockDim.x + threadIdx.x, p = u / n, r = u - p * n, b0 = p * w;
    if (b0 >= B) return;
    float* to = XT + (uint64_t)b0 * n + (uint64_t)r * w;
    if (w < 4) {                                                           // (two rows of X: w = 2)
        *reinterpret_cast<float2*>(to) = make_float2(X[r], X[ldx + r]);
        return;
    }
    for (uint32_t k0 = 0; k0 < w && b0 + k0 < B; k0 += 16) {
        float v[16];
#pragma unroll
        for (uint32_t k = 0; k < 16; ++k) v[k] = X[(uint64_t)(b0 + k0 + k < B ? b0 + k0 + k : B - 1) * ldx + r];
#pragma unroll
        for (uint32_t k = 0; k < 16; k += 4)
            if (k0 + k < w) *reinterpret_cast<float4*>(to + k0 + k) = make_float4(v[k], v[k + 1], v[k + 2], v[k + 3]);
    }
}

template <bool SHAC, int NBD, int SUMS = kHalves>             // SUMS: see fma_entries (NBD = 0)
__global__ void __launch_bounds__(1024)
dot_split_kernel(DevBlob d, SplitParams p, const float* __restrict__ X, uint32_t xrow, uint64_t xcol, uint32_t B,
                 float* __restrict__ Y, uint64_t ldy, float* __restrict__ copy, Epilogue epi)
{
    // X[r * xrow + b * xcol] with NBD; XT in panels of xrow batch columns without
    extern __shared__ uint32_t smem[];
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wib = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // (one branch for both, and the size of the grid read here: a branch more, or the arguments' last line read only where the
    // block size is needed, is another trip to memory before the work, 0.25 us of 5)
    const uint32_t grid = gridDim.x - p.copies, item = logical_block(grid);
    const bool behind = NBD != 0 && blockIdx.x >= grid;
    if (behind | (item >= p.nblocks * p.tiles)) {
        if (behind) leave_copy(grid, X, xcol, B, d.n, copy, epi.panel_w);
        return;
    }
    const uint32_t tile = item / p.nblocks;
    const uint32_t c0 = (item - tile * p.nblocks) << p.cols_log2;          // < m: there are ceil(m / cols) blocks
    const uint32_t ncols = d.m - c0 < p.cols ? d.m - c0 : p.cols;
    const uint32_t wave = item * p.waves + wib;                            // (HAC_MARK)
    HAC_MARK(0);
    uint32_t cchunk_l = 0, cpos_l = 0, cbit_l = 0;                         // lane l: column c0 + l
    if (lane <= ncols) {
        cchunk_l = d.colchunk[c0 + lane];
        cpos_l = d.colpos[c0 + lane];
        cbit_l = d.colbit[c0 + lane];
    }
    TableRegs tr = request_tables(d);
    const uint32_t gfirst = (uint32_t)__shfl((int)cchunk_l, 0, kWave);
    const uint32_t glast = (uint32_t)__shfl((int)cchunk_l, (int)ncols, kWave);
    const uint32_t posbase = (uint32_t)__shfl((int)cpos_l, 0, kWave);
    const uint32_t posend = (uint32_t)__shfl((int)cpos_l, (int)ncols, kWave);
    const uint32_t bit_lo = (uint32_t)__shfl((int)cbit_l, 0, kWave);
    const uint32_t bit_hi = (uint32_t)__shfl((int)cbit_l, (int)ncols, kWave);

    uint32_t* sbuf = smem + table_words_dev(d);
    uint2* list = reinterpret_cast<uint2*>(sbuf + p.sbuf_words);
    double* sums = reinterpret_cast<double*>(sbuf);                        // [wavefront][width], once the words are decoded

    const uint32_t swlo = (bit_lo >> 5) & ~3u;
    const uint32_t snw = (((bit_hi >> 5) + 4) - swlo + 4) & ~3u;           // the decoder reads three words past the current one
    const uint64_t rb_lo = (uint64_t)posbase * d.ri_bits, rb_hi = (uint64_t)posend * d.ri_bits;
    const uint32_t rwlo = (uint32_t)(rb_lo >> 5) & ~3u;
    const uint32_t rnw = SHAC ? ((((uint32_t)(rb_hi >> 5) + 2) - rwlo + 4) & ~3u) : 0u;
    // the host sized the buffers for any block of this blob; a header that does not belong to it must not lead past them
    const bool some = posend > posbase && posend - posbase <= p.list_cap && snw + rnw <= p.sbuf_words &&
                      glast > gfirst && glast - gfirst <= p.waves * kWave;

    // chunks of this wavefront: at least 16 where there are that many, 32 where most CUs have nothing to do (840 x 82,
    // 37 % non-zero, 10 rows: 6.6 -> 6.1 us; but 23016 x 246, 35 %, 19 rows: 42.1 -> 45.9)
    const uint32_t nchunks = some ? glast - gfirst : 0u, least = grid > 128u ? 16u : 32u;
    uint32_t per = (nchunks + p.waves - 1) / p.waves;
    per = per < least ? least : per;                                       // at most 64: nchunks <= 64 waves
    const uint32_t g = gfirst + wib * per + lane;
    const bool active = lane < per && g < gfirst + nchunks;
    uint2 ent_raw = make_uint2(0u, 0u);
    if (active) ent_raw = request_entry(d, g);
    request_table_values(d, tr);
    PieceRegs sq, rq;
    const uint4* s4 = reinterpret_cast<const uint4*>(some ? d.stream + swlo : d.canon);
    const uint4* r4 = reinterpret_cast<const uint4*>(some && SHAC ? d.ri + rwlo : d.canon);
    const uint32_t sn4 = some ? snw >> 2 : 1u, rn4 = some ? rnw >> 2 : 1u;
    request_pieces(sq, s4, sn4);
    if constexpr (SHAC) request_pieces(rq, r4, rn4);
    const Tables tb = store_tables(d, smem, tr);
    if (some) {
        finish_pieces(sq, reinterpret_cast<uint4*>(sbuf), s4, sn4);
        if constexpr (SHAC) finish_pieces(rq, reinterpret_cast<uint4*>(sbuf + snw), r4, rn4);
    }
    __syncthreads();
    HAC_MARK(1);

    // ---- decode: lanes = chunks ----
    {
        uint32_t rel = 0;                                                  // column of chunk g, counted from c0
        for (uint32_t k = 1; k < ncols; ++k) rel += (uint32_t)__shfl((int)cchunk_l, (int)k, kWave) <= g ? 1u : 0u;
        const uint32_t col_chunk0 = (uint32_t)__shfl((int)cchunk_l, (int)rel, kWave);
        const uint32_t col_pos0 = (uint32_t)__shfl((int)cpos_l, (int)rel, kWave);
        const uint32_t col_pos1 = (uint32_t)__shfl((int)cpos_l, (int)rel + 1, kWave);
        const uint32_t col_bit0 = (uint32_t)__shfl((int)cbit_l, (int)rel, kWave);
        if (active) {
            ChunkState st;
            uint32_t ent_rel, ent_row;
            entry_fields(d, ent_raw, ent_rel, ent_row);
            st.bp = col_bit0 + ent_rel;
            st.row = ent_row;
            const uint32_t chunk = hac_internal::chunk_of_column(d.chunk, col_pos1 - col_pos0);
            st.wpos = col_pos0 + (g - col_chunk0) * chunk;
            st.wend = st.wpos + chunk < col_pos1 ? st.wpos + chunk : col_pos1;
            auto emit = [&](uint32_t q, uint32_t row, uint32_t, float v) {
                if (SHAC) list[q - posbase].y = __float_as_uint(v);
                else list[q - posbase] = make_uint2(row, __float_as_uint(v));
            };
            const WordSrc<true> src = { sbuf, swlo };
            if (SHAC) shac_advance(d, tb, src, st, st.wend, emit);
            else if (d.rice) gap_advance(d, tb, src, st, st.wend, emit);
            else if (d.zero_len == 1) hac_advance_zrun(d, tb, src, st, st.wend, emit);
            else hac_advance(d, tb, src, st, st.wend, emit);
        }
    }
    HAC_MARK(2);
    if constexpr (SHAC) {
        if (some) {
            const WordSrc<true> rsrc = { sbuf + snw, rwlo };
            const uint32_t ri_rel0 = (uint32_t)(rb_lo - 32ull * rwlo);
            for (uint32_t q = threadIdx.x; q < posend - posbase; q += blockDim.x)
                list[q].x = rsrc.field_rel(__umul24(q, d.ri_bits) + ri_rel0, d.ri_bits);
        }
    }
    HAC_MARK(3);
    __syncthreads();
    HAC_MARK(4);

    // ---- multiply: the wavefronts of column j share list entries [lo, hi) ----
    const uint32_t j = wib >> p.split_log2, share = wib & ((1u << p.split_log2) - 1u), shares = 1u << p.split_log2;
    uint32_t lo = 0, hi = 0;
    if (some && j < ncols) {
        lo = (uint32_t)__builtin_amdgcn_readlane((int)cpos_l, (int)j) - posbase;
        hi = (uint32_t)__builtin_amdgcn_readlane((int)cpos_l, (int)j + 1) - posbase;
    }
    const uint32_t b0 = tile * p.width;
    const uint32_t nb = B - b0 < p.width ? B - b0 : p.width;               // batch columns of this tile
    if constexpr (NBD == 0) {
        const uint32_t gw = p.width >> 2, ng = kWave / gw;                 // lanes per row of X, rows side by side
        const uint32_t grp = lane / gw, lig = lane & (gw - 1);
        typename SumType<SUMS>::type a[4] = { 0, 0, 0, 0 };
        // (lanes whose four batch columns are all padding fetch nothing)
        if (4 * lig < nb)
            fma_entries<4, 10, SUMS>(list, 0u, lo, hi, ng * shares, share * ng + grp, X + panel_offset(xrow, d.n, b0 + 4 * lig), xrow, a);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            for (uint32_t off = 32; off >= gw; off >>= 1) a[i] += __shfl_xor(a[i], (int)off, kWave);
        HAC_MARK(5);
        if (grp == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) sums[wib * p.width + 4 * lig + i] = a[i];
        }
    } else {
        constexpr int N = NBD ? NBD : 4;
        float a[N];
#pragma unroll
        for (int i = 0; i < N; ++i) a[i] = 0.0f;
        const float* xb = X + (uint64_t)b0 * xcol;
        const uint32_t xrow4 = 4 * xrow;
        for (uint32_t i = lo + share * kWave + lane; i < hi; i += shares * kWave) {
            const uint2 e = list[i];
            const uint32_t off = e.x * xrow4;                              // (the host keeps X below 2^19 floats here)
            const float w = __uint_as_float(e.y);
            float x[N];
            // rows past the batch (fewer than four: the host picks N by the batch) are read at its last row; nobody stores their sums
#pragma unroll
            for (int k = 0; k < N; ++k)
                x[k] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(xb + (uint64_t)((uint32_t)k < nb ? (uint32_t)k : nb - 1u) * xcol) + off);
#pragma unroll
            for (int k = 0; k < N; ++k) a[k] = fmaf(x[k], w, a[k]);
        }
        // sums over the 64 lanes: a turn halves the sums a lane holds and doubles the lanes in each; what is left of an
        // odd number of sums is added over the remaining lanes.  The first turn adds in 32 bits, the others in 64: five turns in
        // 32 bits rounded short columns more often than a chain over their few non-zeros does (500 x 500, 5 %, 128 rows, relative error
        // 5.7e-8 one wavefront per column, 6.1e-8 with five, 4.1e-8 now; 542 x 135, 1 %, 8 rows 4.2e-8, 4.7e-8, 3.4e-8).  They cost 1 %
        // of a call (geometric mean over 172 products; worst 3.3 %: 300 x 120, 100 rows 7.0 -> 7.2 us), all turns in 64 bits 2 %.
        uint32_t first = 0;                                                // of the batch columns whose sums this lane ends up with
        constexpr int halves = N % 32 == 0 ? 5 : N % 16 == 0 ? 4 : N % 8 == 0 ? 3 : 2, left = N >> halves;
        double z[N / 4];
#pragma unroll
        for (int t = 0; t < halves; ++t) {
            const int h = N >> (t + 1);
            const bool up = (lane >> t & 1u) != 0;
#pragma unroll
            for (int k = 0; k < h; ++k) {
                if (t <= 1) {
                    float v0 = a[k], v1 = a[k + h];
                    asm("" : "+v"(v0), "+v"(v1));                          // (or the compiler indexes a[] by lane, with a chain of 32 selects)
                    const float mine = up ? v1 : v0, other = __shfl_xor(up ? v0 : v1, 1 << t, kWave);
                    if (t == 0) a[k] = mine + other;
                    else z[k] = (double)mine + (double)other;
                } else {
                    double v0 = z[k], v1 = z[k + h];
                    asm("" : "+v"(v0), "+v"(v1));
                    z[k] = (up ? v1 : v0) + __shfl_xor(up ? v0 : v1, 1 << t, kWave);
                }
            }
            first += up ? (uint32_t)h : 0u;
        }
#pragma unroll
        for (int t = halves; t < 6; ++t)
#pragma unroll
            for (int k = 0; k < left; ++k) z[k] += __shfl_xor(z[k], 1 << t, kWave);
        HAC_MARK(5);
        if (lane < (1u << halves)) {
#pragma unroll
            for (int k = 0; k < left; ++k) sums[wib * N + first + k] = z[k];
        }
    }
    __syncthreads();
    const uint32_t outs = nb << p.cols_log2;
    for (uint32_t o = threadIdx.x; o < outs; o += blockDim.x) {
        const uint32_t c = o & (p.cols - 1u), b = o >> p.cols_log2;        // neighbouring threads, neighbouring columns
        if (c >= ncols) continue;
        const double* s = sums + (c << p.split_log2) * p.width + b;
        double z = s[0];
        for (uint32_t k = 1; k < shares; ++k) z += s[k * p.width];
        const uint32_t col = c0 + c, row = b0 + b;
        const float v = epilogue_apply(epi, (float)z, col);
        if (epi.yt) epi.yt[panel_offset(epi.panel_w, d.m, row) + (uint64_t)col * epi.panel_w] = v;
        else Y[(uint64_t)row * ldy + col] = v;
    }
    HAC_MARK(6);
}

} // namespace

#endif
