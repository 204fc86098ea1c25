// The quantize+pack work of one 4096-element chunk (Eq. (5)-(6) and the message layout), shared by
// the kernels of dq_quantize_pack.hip and dq_bracketed.hip.
#pragma once
#include "dq_chunk_norm.h"
#include "dq_internal.h"

namespace {

constexpr int QP_THREADS = 256;
constexpr int QP_PER_LANE = 8;
constexpr int QP_TILE = QP_THREADS * QP_PER_LANE;      // 2048 elements: one tile of every wavefront
constexpr int QP_WAVE_TILE = 64 * QP_PER_LANE;         // 512 elements: a wavefront's tile
// Tiles per workgroup: its chunk is the 4096 elements of one entry of the plan's chunk table (one scale for
// all of it) and of the chunk norms.
constexpr int QP_TILES = DQ_CHUNK / QP_TILE;

// Writes the low B bytes of v at dst (LDS, byte offset a multiple of B) with naturally aligned
// stores only.
template <int B>
__device__ __forceinline__ void stage_bytes(uint8_t* dst, uint64_t v)
{
    if constexpr (B == 8) {
        *reinterpret_cast<uint64_t*>(dst) = v;
    } else if constexpr (B == 4) {
        *reinterpret_cast<uint32_t*>(dst) = static_cast<uint32_t>(v);
    } else if constexpr (B % 2 == 0) {
#pragma unroll
        for (int k = 0; k < B / 2; ++k) reinterpret_cast<uint16_t*>(dst)[k] = static_cast<uint16_t>(v >> (16 * k));
    } else {
#pragma unroll
        for (int k = 0; k < B; ++k) dst[k] = static_cast<uint8_t>(v >> (8 * k));
    }
}

// The same for a width that is a value.
__device__ __forceinline__ void stage_bytes_v(uint8_t* dst, uint64_t v, int b)
{
    switch (b) {
    case 1: stage_bytes<1>(dst, v); break;
    case 2: stage_bytes<2>(dst, v); break;
    case 3: stage_bytes<3>(dst, v); break;
    case 4: stage_bytes<4>(dst, v); break;
    case 5: stage_bytes<5>(dst, v); break;
    case 6: stage_bytes<6>(dst, v); break;
    case 7: stage_bytes<7>(dst, v); break;
    default: stage_bytes<8>(dst, v); break;
    }
}

// A lane's eight consecutive elements (two Philox blocks with counters quad, quad + 1): the sign
// byte (element 0 in bit 0) and the 8*B level bits (element 0 in the low B bits).  Per element, with
// a = min(|g| * scale, s) in binary32 and u = (word >> 8) * 2^-24: level = floor(a) + [u < a - floor(a)]
// (Eq. (5)-(6)).  Three routes, chosen per wavefront, all giving exactly those bits:
//   * every lane's eight products |g| * scale are zero (exact-zero stretches of a gradient, or a
//     tensor whose norm is unusable): every level is 0 whatever the random numbers, none are drawn;
//   * every product is below 1 (the usual case for a tensor of many elements: |g|/N ~ 1/sqrt(d)):
//     then a = min(a, s) = a, floor(a) = 0 and a - floor(a) = a, so the level is [u < a] -- no clamp,
//     no fract, no float-to-integer conversion;
//   * otherwise the general form: clamp, v_fract, convert, compare, add with carry.
// The wavefront-wide test costs a maximum over the eight products and two votes.
// S, b: the level count and bits of the tensor (template argument B > 0 fixes them at compile time).
// r[h][k] receives the random word of element 4h + k unless the all-zero route was taken (then no
// caller needs it: every level is zero).
// quantize_quads leaves the two groups of four apart (their Philox blocks are quad0 and quad1): sign
// nibbles and 4*B level bits each.
template <int B>
__device__ __forceinline__ void quantize_quads(const float4 x0, const float4 x1, const float scale, const float S_arg,
                                               const int b_arg, const uint32_t quad0, const uint32_t quad1,
                                               const uint32_t quad_hi, const uint32_t worker, const uint32_t step,
                                               const uint32_t key0, const uint32_t key1, uint32_t (&sign)[2],
                                               uint32_t (&lv)[2], uint32_t (&r)[2][4])
{
    const float S = B > 0 ? static_cast<float>((1 << (B > 0 ? B : 1)) - 1) : S_arg;
    const int b = B > 0 ? B : b_arg;
    const float v[8] = { x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w };
    float a[8];
    sign[0] = sign[1] = 0;
#pragma unroll
    for (int k = 7; k >= 0; --k) {
        sign[k >> 2] = __builtin_amdgcn_alignbit(sign[k >> 2], __float_as_uint(v[k]), 31); // element 4h ends in bit 0
        a[k] = fabsf(v[k]) * scale;                                                         // s|g|/N, one rounding
    }
    const float top = fmaxf(fmaxf(__builtin_fmaxf(__builtin_fmaxf(a[0], a[1]), a[2]), __builtin_fmaxf(__builtin_fmaxf(a[3], a[4]), a[5])),
                            __builtin_fmaxf(a[6], a[7]));
    lv[0] = lv[1] = 0u;
    if (__all(top == 0.0f)) return;
    dq_philox4x32_10(quad0, quad_hi, worker, step, key0, key1, r[0]);
    dq_philox4x32_10(quad1, quad_hi, worker, step, key0, key1, r[1]);
    if (__all(top < 1.0f)) {
#pragma unroll
        for (int h = 1; h >= 0; --h)
#pragma unroll
            for (int k = 3; k >= 0; --k) {
                const float u = static_cast<float>(r[h][k] >> 8) * 0x1p-24f; // exact, in [0,1)
                lv[h] = (lv[h] << b) + (u < a[4 * h + k] ? 1u : 0u);
            }
    } else {
#pragma unroll
        for (int h = 1; h >= 0; --h)
#pragma unroll
            for (int k = 3; k >= 0; --k) {
                const float c = fminf(a[4 * h + k], S);                      // clamped
                const float p = __builtin_amdgcn_fractf(c);                  // c - floor(c), exact
                const float u = static_cast<float>(r[h][k] >> 8) * 0x1p-24f;
                lv[h] = (lv[h] << b) + static_cast<uint32_t>(c) + (u < p ? 1u : 0u);
            }
    }
}

template <int B>
__device__ __forceinline__ void quantize8(const float4 x_lo, const float4 x_hi, const float scale, const float S_arg,
                                          const int b_arg, const uint32_t quad, const uint32_t quad_hi,
                                          const uint32_t worker, const uint32_t step, const uint32_t key0,
                                          const uint32_t key1, uint32_t& sign, uint64_t& level, uint32_t (&r)[2][4])
{
    uint32_t sg[2], lv[2];
    quantize_quads<B>(x_lo, x_hi, scale, S_arg, b_arg, quad, quad + 1u, quad_hi, worker, step, key0, key1, sg, lv, r);
    sign = sg[0] | (sg[1] << 4);
    level = static_cast<uint64_t>(lv[0]) | (static_cast<uint64_t>(lv[1]) << (4 * (B > 0 ? B : b_arg)));
}

// The same for a wavefront's tile as dq_load_wave_tile loaded it (not arranged) when one scale serves
// the whole tile: every lane quantizes the two quads it loaded, and the codes change places instead of
// the values -- two swaps in place of eight.  quad_tile: the tile's first quad.
template <int B>
__device__ __forceinline__ void quantize_wave_tile(const float4 lo, const float4 hi, const float scale, const float S_arg,
                                                   const int b_arg, const uint32_t quad_tile, const uint32_t lane,
                                                   const uint32_t quad_hi, const uint32_t worker, const uint32_t step,
                                                   const uint32_t key0, const uint32_t key1, uint32_t& sign, uint64_t& level)
{
    uint32_t sg[2], lv[2], r[2][4];
    const uint32_t quad = quad_tile + (lane & 31u) * 2u + (lane >> 5);
    quantize_quads<B>(lo, hi, scale, S_arg, b_arg, quad, quad + 64u, quad_hi, worker, step, key0, key1, sg, lv, r);
    const auto s = __builtin_amdgcn_permlane32_swap(sg[0], sg[1], false, false);
    const auto l = __builtin_amdgcn_permlane32_swap(lv[0], lv[1], false, false);
    sign = s[0] | (s[1] << 4);
    level = static_cast<uint64_t>(l[0]) | (static_cast<uint64_t>(l[1]) << (4 * (B > 0 ? B : b_arg)));
}

// First element (inside the chunk) of a lane's eight of tile `it`.  Each wavefront owns TILES
// consecutive tiles of 512 elements, i.e. one stretch of every plane: it stages and stores its own
// bytes, with no workgroup barrier between the two.
// BLOCK: the workgroup's lanes side by side in each of its tiles of 2048 elements instead (see qp_load_block).
template <int TILES, bool BLOCK = false>
__device__ __forceinline__ uint32_t qp_elem(uint32_t tid, int it)
{
    if constexpr (BLOCK) return it * QP_TILE + tid * QP_PER_LANE;
    return (tid >> 6) * (QP_WAVE_TILE * TILES) + it * QP_WAVE_TILE + (tid & 63u) * QP_PER_LANE;
}

// The lane's inputs of every tile, in flight together (dq_arrange_wave_tile completes them).  Lanes
// past the end of a ragged last chunk re-read its last elements (always in bounds); what they
// compute is never stored.
template <int TILES>
__device__ __forceinline__ void qp_load(const float* __restrict__ g, uint32_t tid, uint32_t n_elems, float4 (&x)[TILES][2])
{
#pragma unroll
    for (int it = 0; it < TILES; ++it)
        dq_load_wave_tile(g, (tid >> 6) * (QP_WAVE_TILE * TILES) + it * QP_WAVE_TILE, tid & 63u, n_elems, x[it][0], x[it][1]);
}

// The same for layouts whose chunks hold several tensors: each lane loads its own eight elements, so that
// nothing has to change places before they are used, and the workgroup stores its bytes together after a
// barrier.
template <int TILES>
__device__ __forceinline__ void qp_load_block(const float* __restrict__ g, uint32_t tid, uint32_t n_elems, float4 (&x)[TILES][2])
{
#pragma unroll
    for (int it = 0; it < TILES; ++it) {
        uint32_t e = qp_elem<TILES, true>(tid, it);
        e = e < n_elems ? e : n_elems - QP_PER_LANE;
        x[it][0] = *reinterpret_cast<const float4*>(g + e);
        x[it][1] = *reinterpret_cast<const float4*>(g + e + 4);
    }
}

// The granule (128 elements) of a lane's eight of tile `it`, clamped to the chunk's last one.
template <int TILES, bool BLOCK = false>
__device__ __forceinline__ uint32_t qp_granule(uint32_t tid, int it, uint32_t n_elems)
{
    const uint32_t e = qp_elem<TILES, BLOCK>(tid, it);
    return (e < n_elems ? e : n_elems - QP_PER_LANE) >> 7;
}

// A wavefront's staged bytes [0, bytes) (a multiple of 16) leave as 16-byte streaming stores.
__device__ __forceinline__ void qp_store_wave(uint8_t* __restrict__ dst, const uint8_t* src, uint32_t bytes, uint32_t lane)
{
    uint4* d = reinterpret_cast<uint4*>(dst);
    const uint4* f = reinterpret_cast<const uint4*>(src);
    for (uint32_t i = lane; i < bytes / 16; i += 64) dq_store_stream(d + i, f[i]);
}

// The workgroup's staged bytes [0, bytes) (a multiple of 16), after a barrier.
__device__ __forceinline__ void qp_store_block(uint8_t* __restrict__ dst, const uint8_t* src, uint32_t bytes, uint32_t tid)
{
    uint4* d = reinterpret_cast<uint4*>(dst);
    const uint4* f = reinterpret_cast<const uint4*>(src);
    for (uint32_t i = tid; i < bytes / 16; i += QP_THREADS) dq_store_stream(d + i, f[i]);
}

// What bounds it: the memory system's rate at 4 bytes read to (B+1)/8 written (about 6.1-6.2 TB/s, what a
// kernel with the same accesses and no arithmetic reaches), with the vector ALU at 80 % beside it.  A chunk
// that lies in one tensor (nearly all of a gradient of large tensors) takes the first route: two scalar
// loads and one division per wavefront in place of the granule table, LDS and a barrier, and the codes
// change places between the lanes instead of the values.  Measured at D = 2^28, M = 16 against the table
// route alone: b = 2 3.36 -> 3.06 ms (6.1 TB/s), b = 4 3.39 -> 3.28 ms; ResNet-18 shape, M = 8, b = 2
// 74.9 -> 66.9 us.  Chunks that hold a tensor's end or several tensors take the table.
// WHOLE = false (NORM = 0 only): no such route, and the lanes' elements as qp_load_block has them, for layouts with
// few chunks of one tensor (dq_plan::many_whole).  Measured there against the form with the route, in us: 5.4 M
// values in tensors of 128, M = 8 b = 4 38.0 -> 36.6, 16.8 M in tensors of 512, M = 8 b = 6 121.8 -> 114.8 and, with a
// widths table, b = 7 130.9 -> 122.4; 30.7 M in tensors of 1000, M = 4 b = 6 112.0 -> 104.5.
//
// NORM = 0: the norms are an input.  NORM = 1 (l2) or 2 (max): chunk-local plans only; the kernel
// computes the norms of its chunk's tensors itself, writes them to norms_out and quantizes from
// the registers it already holds -- one read of the gradient instead of two.
template <int B, int TILES, int NORM, bool WHOLE = true>
__device__ __forceinline__ void quantize_pack_chunk(
    const float* __restrict__ grads, int64_t worker_stride, const float* __restrict__ norms, int32_t n_seg,
    const dq_chunk_tensor* __restrict__ chunk_tensor, const int32_t* __restrict__ granule_cseg,
    const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems,
    uint32_t key0, uint32_t key1, uint32_t step, uint32_t worker_base, uint8_t* __restrict__ packed,
    int64_t packed_stride, float* __restrict__ norms_out, uint32_t chunk_index)
{
    constexpr int CHUNK = QP_TILE * TILES;
    constexpr int MAX_LOCAL_SEG = CHUNK / DQ_GRANULE;
    constexpr float S = static_cast<float>((1 << B) - 1);
    static_assert(CHUNK == DQ_CHUNK, "the chunk table and the fused norm work on 4096-element chunks");
    constexpr bool BLOCK = NORM == 0 && !WHOLE;

    __shared__ float lds_scale[MAX_LOCAL_SEG];
    __shared__ int32_t lds_valid_end[MAX_LOCAL_SEG]; // relative to the chunk, clamped to CHUNK
    __shared__ __align__(16) uint8_t lds_sign[TILES * QP_THREADS];
    __shared__ __align__(16) uint8_t lds_level[TILES * QP_THREADS * B];

    const uint32_t tid = threadIdx.x;
    const uint32_t w = blockIdx.y;
    const int64_t chunk0 = static_cast<int64_t>(chunk_index) * CHUNK;
    // elements of this chunk that exist (a multiple of 128, at least 128)
    const uint32_t n_elems = static_cast<uint32_t>(padded_elems - chunk0 < CHUNK ? padded_elems - chunk0 : CHUNK);
    const float* g = grads + static_cast<int64_t>(w) * worker_stride + chunk0; // uniform base
    const int32_t* gseg = granule_cseg + (chunk0 >> 7);

    // This lane's inputs first, so the loads are in flight while the segment table is built.
    float4 x[TILES][2];
    if constexpr (BLOCK)
        qp_load_block<TILES>(g, tid, n_elems, x);
    else
        qp_load<TILES>(g, tid, n_elems, x);

    // Philox counter words: quad index P>>2 (low word varies per lane, high word is uniform because
    // a chunk never straddles a multiple of 2^34 elements), worker, step
    const uint32_t quad_lo0 = static_cast<uint32_t>(static_cast<uint64_t>(chunk0) >> 2);
    const uint32_t quad_hi = static_cast<uint32_t>(static_cast<uint64_t>(chunk0) >> 34);
    const uint32_t worker = worker_base + w;
    uint8_t* msg = packed + static_cast<int64_t>(w) * packed_stride;
    const uint32_t wave0 = (tid >> 6) * (QP_WAVE_TILE * TILES);

    if constexpr (NORM == 0 && WHOLE) {
        const dq_chunk_tensor whole = dq_load_chunk_tensor(chunk_tensor, chunk0 / DQ_CHUNK);
        const float N = norms[static_cast<int64_t>(w) * n_seg + whole.seg]; // issued whatever cseg is: one wait less
        if (whole.cseg >= 0) { // 4096 elements of one tensor: one scale, nothing to mask, no table, no barrier
            const float scale = N >= DQ_MIN_NORM ? S / N : 0.0f;
#pragma unroll
            for (int it = 0; it < TILES; ++it) {
                uint32_t sign;
                uint64_t level;
                const uint32_t tile0 = wave0 + it * QP_WAVE_TILE, at = (tile0 >> 3) + (tid & 63u);
                quantize_wave_tile<B>(x[it][0], x[it][1], scale, 0.0f, 0, quad_lo0 + (tile0 >> 2), tid & 63u, quad_hi,
                                      worker, step, key0, key1, sign, level);
                lds_sign[at] = static_cast<uint8_t>(sign);
                stage_bytes<B>(&lds_level[at * B], level);
            }
            dq_wave_sync();
            qp_store_wave(msg + ((chunk0 + wave0) >> 3), &lds_sign[wave0 >> 3], QP_WAVE_TILE * TILES / 8, tid & 63u);
            qp_store_wave(msg + (padded_elems >> 3) + ((chunk0 + wave0) >> 3) * B, &lds_level[(wave0 >> 3) * B],
                          QP_WAVE_TILE * TILES / 8 * B, tid & 63u);
            return;
        }
    }

    int32_t seg[TILES];
#pragma unroll
    for (int it = 0; it < TILES; ++it) seg[it] = gseg[qp_granule<TILES, BLOCK>(tid, it, n_elems)];

    // compact segment indices grow by at most one per granule, so the chunk's segments fit the table
    const int32_t seg_first = gseg[0];
    const int32_t seg_last = gseg[(n_elems - 1) >> 7];
    if constexpr (NORM == 0) {
        if (static_cast<int32_t>(tid) <= seg_last - seg_first) {
            const float N = norms[static_cast<int64_t>(w) * n_seg + cseg_seg[seg_first + tid]];
            lds_scale[tid] = N >= DQ_MIN_NORM ? S / N : 0.0f; // zero, tiny or NaN norm: every level 0
            const int64_t rel = cseg_valid_end[seg_first + tid] - chunk0;
            lds_valid_end[tid] = rel < CHUNK ? static_cast<int32_t>(rel) : CHUNK;
        }
        __syncthreads();
        if constexpr (!BLOCK) {
#pragma unroll
            for (int it = 0; it < TILES; ++it) dq_arrange_wave_tile(x[it][0], x[it][1]);
        }
    } else {
        __shared__ double lds_gsum[DQ_CHUNK_GRANULES];
        __shared__ int32_t lds_glocal[DQ_CHUNK_GRANULES];
        if (static_cast<int32_t>(tid) <= seg_last - seg_first) {
            const int64_t rel = cseg_valid_end[seg_first + tid] - chunk0;
            lds_valid_end[tid] = rel < CHUNK ? static_cast<int32_t>(rel) : CHUNK;
        }
        __syncthreads();
        int valid[TILES], local[TILES], granule[TILES];
#pragma unroll
        for (int it = 0; it < TILES; ++it) {
            dq_arrange_wave_tile(x[it][0], x[it][1]);
            const uint32_t e = qp_elem<TILES, BLOCK>(tid, it);
            granule[it] = static_cast<int>(e >> 7);
            local[it] = seg[it] - seg_first;
            valid[it] = e < n_elems ? lds_valid_end[local[it]] - static_cast<int32_t>(e) : 0;
        }
        const int n_scan = dq_chunk_granule_sums<NORM == 2>(x, valid, local, granule, static_cast<int>(tid), lds_gsum,
                                                            lds_glocal, seg_first == seg_last,
                                                            static_cast<int>(n_elems >> 7));
        __syncthreads();
        if (tid < DQ_CHUNK_GRANULES)
            dq_chunk_tensor_norms<NORM == 2>(static_cast<int>(tid), n_scan, lds_gsum, lds_glocal,
                                             [&](int j, float N) {
                                                 norms_out[static_cast<int64_t>(w) * n_seg + cseg_seg[seg_first + j]] = N;
                                                 lds_scale[j] = N >= DQ_MIN_NORM ? S / N : 0.0f;
                                             });
        __syncthreads();
    }

#pragma unroll
    for (int it = 0; it < TILES; ++it) {
        const uint32_t e = qp_elem<TILES, BLOCK>(tid, it);
        if (e < n_elems) {
            const int local = seg[it] - seg_first;
            const float scale = lds_scale[local];
            const int32_t n_valid = lds_valid_end[local] - static_cast<int32_t>(e); // may be <= 0 or > 8

            const uint32_t quad = quad_lo0 + (e >> 2); // even; quad + 1 cannot carry
            uint32_t sign;
            uint64_t level;
            uint32_t r[2][4];
            quantize8<B>(x[it][0], x[it][1], scale, 0.0f, 0, quad, quad_hi, worker, step, key0, key1, sign, level, r);
            if (n_valid < QP_PER_LANE) { // the tensor ends inside (or before) this lane's eight elements
                const int nv = n_valid > 0 ? n_valid : 0;
                sign &= (1u << nv) - 1u;
                level &= (static_cast<uint64_t>(1) << (nv * B)) - 1u;
            }
            lds_sign[e >> 3] = static_cast<uint8_t>(sign);
            stage_bytes<B>(&lds_level[(e >> 3) * B], level);
        }
    }
    if constexpr (BLOCK) {
        __syncthreads();
        qp_store_block(msg + (chunk0 >> 3), lds_sign, n_elems >> 3, tid);
        qp_store_block(msg + (padded_elems >> 3) + (chunk0 >> 3) * B, lds_level, (n_elems >> 3) * B, tid);
        return;
    }
    dq_wave_sync();

    // 16-byte stores of this wavefront's stretch; every plane of it is a whole number of 16-byte
    // pieces because it holds a multiple of 128 elements
    if (wave0 < n_elems) {
        const uint32_t n_wave = n_elems - wave0 < QP_WAVE_TILE * TILES ? n_elems - wave0 : QP_WAVE_TILE * TILES;
        qp_store_wave(msg + ((chunk0 + wave0) >> 3), &lds_sign[wave0 >> 3], n_wave >> 3, tid & 63u);
        qp_store_wave(msg + (padded_elems >> 3) + ((chunk0 + wave0) >> 3) * B, &lds_level[(wave0 >> 3) * B],
                      (n_wave >> 3) * B, tid & 63u);
    }
}

// ---------------------------------------------------------------------------------------------
// Per-tensor widths.  Same work split; b, the level count and the place of the level bytes come
// from the widths table per segment instead of the template argument.  A wavefront's level bytes are
// still one contiguous stretch of the message (every segment's stretch is a whole number of
// 16-byte pieces per granule), so they are staged and stored the same way.
// ---------------------------------------------------------------------------------------------
template <int TILES, int NORM, bool WHOLE = true> // as in quantize_pack_chunk
__device__ __forceinline__ void quantize_pack_chunk_v(
    const float* __restrict__ grads, int64_t worker_stride, const float* __restrict__ norms, int32_t n_seg,
    const dq_chunk_tensor* __restrict__ chunk_tensor, const int32_t* __restrict__ granule_cseg,
    const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_valid_end,
    const dq_cseg_width* __restrict__ widths_table, int32_t widths_worker_stride, int64_t padded_elems,
    uint32_t key0, uint32_t key1, uint32_t step, uint32_t worker_base, uint8_t* __restrict__ packed,
    int64_t packed_stride, float* __restrict__ norms_out, uint32_t chunk_index)
{
    constexpr int CHUNK = QP_TILE * TILES;
    constexpr int MAX_LOCAL_SEG = CHUNK / DQ_GRANULE;
    static_assert(CHUNK == DQ_CHUNK, "the chunk table and the fused norm work on 4096-element chunks");
    constexpr bool BLOCK = NORM == 0 && !WHOLE;
    // this worker's row of the table (stride 0: the workers share one row)
    const dq_cseg_width* __restrict__ widths = widths_table + static_cast<int64_t>(blockIdx.y) * widths_worker_stride;

    __shared__ float lds_scale[MAX_LOCAL_SEG];
    __shared__ float lds_levels[MAX_LOCAL_SEG];      // s = 2^b - 1 of the segment
    __shared__ int32_t lds_b[MAX_LOCAL_SEG];
    __shared__ int32_t lds_level_base[MAX_LOCAL_SEG]; // byte offset, in the chunk's level bytes, the
                                                      // segment's fields would have at chunk element 0
    __shared__ int32_t lds_valid_end[MAX_LOCAL_SEG];
    __shared__ __align__(16) uint8_t lds_sign[TILES * QP_THREADS];
    __shared__ __align__(16) uint8_t lds_level[TILES * QP_THREADS * 8];

    const uint32_t tid = threadIdx.x;
    const uint32_t w = blockIdx.y;
    const int64_t chunk0 = static_cast<int64_t>(chunk_index) * CHUNK;
    const uint32_t n_elems = static_cast<uint32_t>(padded_elems - chunk0 < CHUNK ? padded_elems - chunk0 : CHUNK);
    const float* g = grads + static_cast<int64_t>(w) * worker_stride + chunk0;
    const int32_t* gseg = granule_cseg + (chunk0 >> 7);

    float4 x[TILES][2];
    if constexpr (BLOCK)
        qp_load_block<TILES>(g, tid, n_elems, x);
    else
        qp_load<TILES>(g, tid, n_elems, x);

    const uint32_t quad_lo0 = static_cast<uint32_t>(static_cast<uint64_t>(chunk0) >> 2);
    const uint32_t quad_hi = static_cast<uint32_t>(static_cast<uint64_t>(chunk0) >> 34);
    const uint32_t worker = worker_base + w;
    uint8_t* msg = packed + static_cast<int64_t>(w) * packed_stride;
    const uint32_t wave0 = (tid >> 6) * (QP_WAVE_TILE * TILES);

    if constexpr (NORM == 0 && WHOLE) { // one tensor: as in quantize_pack_chunk, its width from one (scalar) table entry
        const dq_chunk_tensor whole = dq_load_chunk_tensor(chunk_tensor, chunk0 / DQ_CHUNK);
        const float N = norms[static_cast<int64_t>(w) * n_seg + whole.seg];
        if (whole.cseg >= 0) {
            const dq_cseg_width e = widths[whole.cseg];
            const float S = static_cast<float>((1 << e.b) - 1);
            const float scale = N >= DQ_MIN_NORM ? S / N : 0.0f;
#pragma unroll
            for (int it = 0; it < TILES; ++it) {
                uint32_t sign;
                uint64_t level;
                const uint32_t tile0 = wave0 + it * QP_WAVE_TILE, at = (tile0 >> 3) + (tid & 63u);
                quantize_wave_tile<0>(x[it][0], x[it][1], scale, S, e.b, quad_lo0 + (tile0 >> 2), tid & 63u, quad_hi,
                                      worker, step, key0, key1, sign, level);
                lds_sign[at] = static_cast<uint8_t>(sign);
                stage_bytes_v(&lds_level[at * e.b], level, e.b);
            }
            dq_wave_sync();
            qp_store_wave(msg + ((chunk0 + wave0) >> 3), &lds_sign[wave0 >> 3], QP_WAVE_TILE * TILES / 8, tid & 63u);
            qp_store_wave(msg + (padded_elems >> 3) + e.level_start + ((chunk0 + wave0 - e.seg_start) >> 3) * e.b,
                          &lds_level[(wave0 >> 3) * e.b], QP_WAVE_TILE * TILES / 8 * e.b, tid & 63u);
            return;
        }
    }

    int32_t seg[TILES];
#pragma unroll
    for (int it = 0; it < TILES; ++it) seg[it] = gseg[qp_granule<TILES, BLOCK>(tid, it, n_elems)];

    const int32_t seg_first = gseg[0];
    const int32_t seg_last = gseg[(n_elems - 1) >> 7];
    // where the chunk's level bytes start in the level plane (uniform)
    const dq_cseg_width first = widths[seg_first];
    const int64_t chunk_level0 = first.level_start + ((chunk0 - first.seg_start) >> 3) * first.b;
    if (static_cast<int32_t>(tid) <= seg_last - seg_first) {
        const dq_cseg_width e = widths[seg_first + tid];
        const float S = static_cast<float>((1 << e.b) - 1);
        if constexpr (NORM == 0) {
            const float N = norms[static_cast<int64_t>(w) * n_seg + cseg_seg[seg_first + tid]];
            lds_scale[tid] = N >= DQ_MIN_NORM ? S / N : 0.0f;
        }
        lds_levels[tid] = S;
        lds_b[tid] = e.b;
        // chunk0 - seg_start is a multiple of 128 of either sign, so the shift is exact
        lds_level_base[tid] = static_cast<int32_t>(e.level_start + ((chunk0 - e.seg_start) >> 3) * e.b - chunk_level0);
        const int64_t rel = cseg_valid_end[seg_first + tid] - chunk0;
        lds_valid_end[tid] = rel < CHUNK ? static_cast<int32_t>(rel) : CHUNK;
    }
    __syncthreads();
    if constexpr (!BLOCK) {
#pragma unroll
        for (int it = 0; it < TILES; ++it) dq_arrange_wave_tile(x[it][0], x[it][1]);
    }
    if constexpr (NORM != 0) {
        __shared__ double lds_gsum[DQ_CHUNK_GRANULES];
        __shared__ int32_t lds_glocal[DQ_CHUNK_GRANULES];
        int valid[TILES], local[TILES], granule[TILES];
#pragma unroll
        for (int it = 0; it < TILES; ++it) {
            const uint32_t e = qp_elem<TILES, BLOCK>(tid, it);
            granule[it] = static_cast<int>(e >> 7);
            local[it] = seg[it] - seg_first;
            valid[it] = e < n_elems ? lds_valid_end[local[it]] - static_cast<int32_t>(e) : 0;
        }
        const int n_scan = dq_chunk_granule_sums<NORM == 2>(x, valid, local, granule, static_cast<int>(tid), lds_gsum,
                                                            lds_glocal, seg_first == seg_last,
                                                            static_cast<int>(n_elems >> 7));
        __syncthreads();
        if (tid < DQ_CHUNK_GRANULES)
            dq_chunk_tensor_norms<NORM == 2>(static_cast<int>(tid), n_scan, lds_gsum, lds_glocal,
                                             [&](int j, float N) {
                                                 norms_out[static_cast<int64_t>(w) * n_seg + cseg_seg[seg_first + j]] = N;
                                                 lds_scale[j] = N >= DQ_MIN_NORM ? lds_levels[j] / N : 0.0f;
                                             });
        __syncthreads();
    }

#pragma unroll
    for (int it = 0; it < TILES; ++it) {
        const uint32_t e = qp_elem<TILES, BLOCK>(tid, it);
        if (e < n_elems) {
            const int local = seg[it] - seg_first;
            const float scale = lds_scale[local];
            const float S = lds_levels[local];
            const int b = lds_b[local];
            const int32_t n_valid = lds_valid_end[local] - static_cast<int32_t>(e);

            const uint32_t quad = quad_lo0 + (e >> 2);
            uint32_t sign, r[2][4];
            uint64_t level;
            quantize8<0>(x[it][0], x[it][1], scale, S, b, quad, quad_hi, worker, step, key0, key1, sign, level, r);
            if (n_valid < QP_PER_LANE) {
                const int nv = n_valid > 0 ? n_valid : 0;
                sign &= (1u << nv) - 1u;
                level &= (static_cast<uint64_t>(1) << (nv * b)) - 1u;
            }
            lds_sign[e >> 3] = static_cast<uint8_t>(sign);
            // b bytes at an offset that is a multiple of b past a 16-byte boundary (every tensor's
            // stretch of a chunk starts on one), so the naturally aligned stores of stage_bytes apply
            stage_bytes_v(&lds_level[lds_level_base[local] + static_cast<int32_t>(e >> 3) * b], level, b);
        }
    }
    if constexpr (BLOCK) {
        __syncthreads();
        const int last = seg_last - seg_first;
        qp_store_block(msg + (chunk0 >> 3), lds_sign, n_elems >> 3, tid);
        qp_store_block(msg + (padded_elems >> 3) + chunk_level0, lds_level,
                       static_cast<uint32_t>(lds_level_base[last]) + (n_elems >> 3) * lds_b[last], tid);
        return;
    }
    dq_wave_sync();

    if (wave0 < n_elems) {
        const uint32_t n_wave = n_elems - wave0 < QP_WAVE_TILE * TILES ? n_elems - wave0 : QP_WAVE_TILE * TILES;
        qp_store_wave(msg + ((chunk0 + wave0) >> 3), &lds_sign[wave0 >> 3], n_wave >> 3, tid & 63u);
        // level bytes of the wavefront's first element up to those of its last granule
        // (their tensors from the wavefront's first and last lane: looked up in the table again, ahead of the stores,
        // they cost norms and messages in one read 3 to 4 %: 16.4 M values, M = 8, tensors of 4096 126.6 -> 122.4 us)
        const int a = __builtin_amdgcn_readfirstlane(seg[0]) - seg_first;
        const int z = __builtin_amdgcn_readlane(seg[TILES - 1], 63) - seg_first;
        const int32_t from = lds_level_base[a] + static_cast<int32_t>(wave0 >> 3) * lds_b[a];
        const int32_t to = lds_level_base[z] + static_cast<int32_t>((wave0 + n_wave) >> 3) * lds_b[z];
        qp_store_wave(msg + (padded_elems >> 3) + chunk_level0 + from, &lds_level[from], static_cast<uint32_t>(to - from),
                      tid & 63u);
    }
}

} // namespace
