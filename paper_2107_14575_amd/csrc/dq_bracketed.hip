// dq_norm_quantize_pack_bracketed: norms and messages in one pass over the gradient for ANY plan,
// given a bracket [lo, hi] for every norm (say, last iteration's norm give or take a margin) and a
// bit-width that is known beforehand (Algorithm 1: the worker received b_t with x_t).
//
// For a fixed element and random number the level of Eq. (5)-(6) never grows with the norm:
// s/N rounded to binary32 does not grow with N, |g| * scale rounded does not grow when the scale
// shrinks, and a -> floor(a) + [u < a - floor(a)] never decreases in a (inside one integer interval
// the indicator can only switch on; across intervals floor(a) + 1 <= floor(a')).  So an element
// whose level is the same at both ends of the bracket has that level for every norm inside it.
//
//   k_quantize_pack_bracketed  reads the gradient once: adds up each tensor's squares chunk by
//       chunk (binary64 partial sums, one slot per chunk and tensor).  A tensor that lies wholly
//       inside the chunk needs no bracket: its norm is finished on the spot and used.  For the
//       others the kernel quantizes with the low end
//       of the bracket (the largest levels), looks at the non-zero levels again with the high end,
//       writes the levels that agree, leaves the others' fields zero and records those elements
//       (index and value) in the chunk's block of the workspace.
//   k_bracket_norm_finish      for the tensors that cross a chunk boundary: adds the partial sums in
//       a fixed order: the norms, and whether each came out inside its bracket.
//   k_bracket_settle           one lane per chunk: quantizes the chunk's recorded elements with the
//       true norm and ORs their levels into the zero fields; a chunk with too many records, with
//       no usable bracket, or with a norm outside its bracket gets a bit in the redo map instead.
//   k_bracket_redo             quantizes the chunks of the redo map again in full from the
//       gradient (the only case that reads it twice); a few thousand workgroups walk the map, so
//       an empty map costs next to nothing.
//   k_bracket_settle_redo      both in one launch for up to 2^16 (worker, chunk) pairs: one wavefront per
//       chunk and a lane per record; a chunk to be quantized again is taken by its workgroup.  Up to 6144 pairs it
//       takes k_bracket_norm_finish's work too.
// The messages are exactly those of dq_quantize_pack for the norms this path computes.
#include "dq_quantize_core.h"

namespace {

// One element again with another scale: the level of Eq. (5)-(6) for element value v and random word r.
template <int B>
__device__ __forceinline__ uint32_t level_of(float v, float scale, uint32_t r)
{
    constexpr float S = static_cast<float>((1 << B) - 1);
    const float a = fminf(fabsf(v) * scale, S);
    const float p = __builtin_amdgcn_fractf(a);
    const float u = static_cast<float>(r >> 8) * 0x1p-24f;
    return static_cast<uint32_t>(a) + (u < p ? 1u : 0u);
}

// The same with the level count as a value (per-tensor widths).
__device__ __forceinline__ uint32_t level_of_s(float v, float scale, float S, uint32_t r)
{
    const float a = fminf(fabsf(v) * scale, S);
    const float p = __builtin_amdgcn_fractf(a);
    const float u = static_cast<float>(r >> 8) * 0x1p-24f;
    return static_cast<uint32_t>(a) + (u < p ? 1u : 0u);
}

// A quad's elements whose level the bracket leaves open: `open` holds their fields of b bits, and those fields of lv are
// cleared for the settle kernel.  e: the quad's first element in the chunk.  Few lanes have any, and seldom more than
// one: a lane takes one per turn and picks its value from the registers.  With code of its own for each of a lane's
// eight elements the kernels needed 85 to 88 registers for the random numbers kept across the second look (five wavefronts
// per SIMD); so they need 70 to 72 (seven): 2^24 values, M = 16, b = 2 254 -> 245 us, ResNet-18 shape, M = 8, b = 3
// 105 -> 97.
// B: the width, 0 where it is a value.
template <int B>
__device__ __forceinline__ void record_open(uint32_t open, const float4 x, const int b, const uint32_t e, uint32_t* count,
                                            dq_bracket_block* __restrict__ blk, uint32_t& lv)
{
    const uint32_t field = (1u << b) - 1u;
    open &= quad_fields<B>(b); // each turn clears one of four fields: at most four turns
    while (open != 0) {
        const int bit = __builtin_ctz(open);
        uint32_t k; // bit / b, for bits below 32
        if constexpr (B > 0)
            k = static_cast<uint32_t>(bit) * ((256 + (B > 0 ? B : 1) - 1) / (B > 0 ? B : 1)) >> 8;
        else
            k = (bit >= b ? 1u : 0u) + (bit >= 2 * b ? 1u : 0u) + (bit >= 3 * b ? 1u : 0u);
        const uint32_t keep = ~(field << (k * b));
        const float lo = (k & 1u) ? x.y : x.x, hi = (k & 1u) ? x.w : x.z;
        const uint32_t slot = atomicAdd(count, 1u);
        if (slot < DQ_BRACKET_CAP) { // a 32-bit offset from the uniform block: no 64-bit address in registers
            const uint32_t at = static_cast<uint32_t>(offsetof(dq_bracket_block, rec)) + slot * static_cast<uint32_t>(sizeof(uint2));
            *reinterpret_cast<uint2*>(reinterpret_cast<char*>(blk) + at) = make_uint2(e + k, __float_as_uint((k & 2u) ? hi : lo));
        }
        open &= keep;
        lv &= keep;
    }
}

// A chunk that lies in one tensor which goes on beyond it -- nearly every chunk of a gradient of large
// tensors: one bracket for all of it (two scalar loads and two divisions), nothing to mask.  The squares
// are added from the values as they were loaded, the lanes quantize the two quads they loaded and the
// codes change places.  Row totals and counts meet in LDS, and the wavefront that finishes last (a ticket in
// LDS) writes the chunk's partial sum and block header: no wavefront waits for another where the chunk's bytes of the
// message start on cache lines; elsewhere there is one barrier ahead of their stores (qp_store_chunk), so all of the
// workgroup has to come here.
// What bounds it: the vector ALU.  Measured against the general route below for every chunk: a lagged
// iteration of 2^26 values, 16 workers, b = 4 from the widths table 1172 -> 1081 us, of the ResNet-18 shape,
// 8 workers, b = 3 141 -> 132 us.
// `state` is the workgroup's: 16 row totals, then the count of open elements and the tickets, both
// cleared by the caller ahead of a barrier.
struct bracket_state {
    double row[16];
    uint32_t count, tickets;
};

template <int B, bool LINF>
__device__ __forceinline__ void bracketed_one_tensor(const float4 (&x)[2][2], float lo, float hi, uint32_t tid,
                                                     int64_t chunk0, uint32_t key0, uint32_t key1, uint32_t step,
                                                     uint32_t worker, bracket_state* state, uint8_t* lds_sign,
                                                     uint8_t* lds_level, uint8_t* __restrict__ sign_chunk,
                                                     uint8_t* __restrict__ level_chunk, dq_bracket_block* __restrict__ blk,
                                                     double* __restrict__ partial)
{
    constexpr float S = static_cast<float>((1 << B) - 1);
    const uint32_t lane = tid & 63u;

    double row;
    if constexpr (LINF) {
        float m = 0.0f;
#pragma unroll
        for (int it = 0; it < 2; ++it)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float v[4] = { fabsf(x[it][h].x), fabsf(x[it][h].y), fabsf(x[it][h].z), fabsf(x[it][h].w) };
#pragma unroll
                for (int k = 0; k < 4; ++k) m = v[k] > m ? v[k] : m; // a NaN never wins
            }
        float o;
        o = dq_row_ror<8>(m); m = o > m ? o : m;
        o = dq_row_ror<4>(m); m = o > m ? o : m;
        o = dq_row_ror<2>(m); m = o > m ? o : m;
        o = dq_row_ror<1>(m); m = o > m ? o : m;
        row = static_cast<double>(m);
    } else {
        row = 0.0;
#pragma unroll
        for (int it = 0; it < 2; ++it)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float v[4] = { x[it][h].x, x[it][h].y, x[it][h].z, x[it][h].w };
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double e = static_cast<double>(v[k]);
                    row = __builtin_fma(e, e, row);
                }
            }
        row += dq_row_ror<8>(row);
        row += dq_row_ror<4>(row);
        row += dq_row_ror<2>(row);
        row += dq_row_ror<1>(row);
    }
    if ((tid & 15u) == 0) state->row[tid >> 4] = row;

    // the zero path (norm below DQ_MIN_NORM) is not monotone against the rest: no bracket across it
    const bool usable = lo >= DQ_MIN_NORM && hi >= lo && hi <= 3.0e38f; // false for NaN; the same for all lanes
    if (usable) {
        // both in one division, a half of the wavefront each
        const float scales = S / (lane < 32u ? lo : hi);
        const float scale_hi = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(scales), 0));
        const float scale_lo = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(scales), 32));
        const uint32_t quad_lo0 = static_cast<uint32_t>(static_cast<uint64_t>(chunk0) >> 2);
        const uint32_t quad_hi = static_cast<uint32_t>(static_cast<uint64_t>(chunk0) >> 34);
        const uint32_t wave0 = (tid >> 6) * (QP_WAVE_TILE * 2);
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const uint32_t tile0 = wave0 + it * QP_WAVE_TILE;
            const uint32_t e0 = tile0 + (lane & 31u) * 8u + (lane >> 5) * 4u; // elements e0.. and e0 + 256..
            const uint32_t quad = quad_lo0 + (e0 >> 2);
            uint32_t lv[2], sign;
            uint64_t level;
            float t[8];
            // levels at the low end of the bracket: the largest any norm inside it can give
            const qp_range range = quantize_quads<B>(x[it][0], x[it][1], scale_hi, 0.0f, 0, quad, quad + 64u, quad_hi, worker,
                                                     step, key0, key1, lv, t);
            if (__any(((lv[0] | lv[1]) & quad_fields<B>(B)) != 0)) { // a zero at the low end is a zero everywhere in the bracket
                uint32_t lv_lo[2];
                quantize_again<B>(range, x[it][0], x[it][1], scale_lo, 0.0f, 0, t, lv_lo);
                record_open<B>(lv[0] ^ lv_lo[0], x[it][0], B, e0, &state->count, blk, lv[0]);
                record_open<B>(lv[1] ^ lv_lo[1], x[it][1], B, e0 + 256, &state->count, blk, lv[1]);
            }
            quantize_exchange<B>(x[it][0], x[it][1], lv, 0, sign, level);
            const uint32_t at = (tile0 >> 3) + lane;
            lds_sign[at] = static_cast<uint8_t>(sign);
            stage_bytes<B>(&lds_level[at * B], level);
        }
        qp_store_chunk(sign_chunk, level_chunk, lds_sign, lds_level, DQ_CHUNK, wave0, B, tid);
    }

    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    uint32_t ticket = 0;
    if (lane == 0) ticket = atomicAdd(&state->tickets, 1u);
    if (__builtin_amdgcn_readfirstlane(ticket) != QP_THREADS / 64 - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    double total = state->row[lane & 15u];
    total = dq_chunk_combine<LINF>(total, dq_row_ror<8>(total));
    total = dq_chunk_combine<LINF>(total, dq_row_ror<4>(total));
    total = dq_chunk_combine<LINF>(total, dq_row_ror<2>(total));
    total = dq_chunk_combine<LINF>(total, dq_row_ror<1>(total));
    if (lane == 0) {
        *partial = total;
        blk->count = usable ? state->count : 0u;
        blk->flags = usable ? 0u : 1u; // 1: nothing was quantized, the redo kernel takes the chunk from the gradient
    }
}

// Whether chunk k is one for bracketed_one_tensor: the tensor's compact index, or -1.
__device__ __forceinline__ int32_t bracketed_one_tensor_of(const dq_chunk_tensor whole, const int64_t* __restrict__ cseg_start,
                                                           const int64_t* __restrict__ cseg_valid_end)
{
    if (whole.cseg < 0) return -1;
    return cseg_valid_end[whole.cseg] - cseg_start[whole.cseg] > DQ_CHUNK ? whole.cseg : -1;
}

template <int B, bool LINF> // LINF: the max norm (p = infinity in Eq. (5)) instead of the l2 norm
__global__ __launch_bounds__(QP_THREADS) void k_quantize_pack_bracketed(
    const float* __restrict__ grads, int64_t worker_stride, const float* __restrict__ norm_lo,
    const float* __restrict__ norm_hi, int32_t n_seg, const dq_chunk_tensor* __restrict__ chunk_tensor,
    const int32_t* __restrict__ granule_cseg, const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_start,
    const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems, uint32_t key0, uint32_t key1, uint32_t step,
    uint32_t worker_base, uint8_t* __restrict__ packed, int64_t packed_stride, double* __restrict__ partials,
    int64_t n_slots, dq_bracket_block* __restrict__ blocks, int64_t n_chunks, float* __restrict__ norms_out,
    uint8_t* __restrict__ inside, int32_t n_cseg)
{
    constexpr int TILES = 2;
    constexpr int CHUNK = DQ_CHUNK;
    constexpr float S = static_cast<float>((1 << B) - 1);
    constexpr uint32_t FIELDS = quad_fields<B>(B);

    __shared__ float lds_scale_hi[DQ_CHUNK_GRANULES]; // s / lo: the larger scale
    __shared__ float lds_scale_lo[DQ_CHUNK_GRANULES]; // s / hi
    __shared__ int32_t lds_valid_end[DQ_CHUNK_GRANULES];
    __shared__ double lds_gsum[DQ_CHUNK_GRANULES];
    __shared__ int32_t lds_glocal[DQ_CHUNK_GRANULES];
    __shared__ uint32_t lds_count;
    __shared__ int32_t lds_whole[DQ_CHUNK_GRANULES]; // the tensor lies wholly inside this chunk
    __shared__ int32_t lds_any_whole;
    __shared__ __align__(16) uint8_t lds_sign[TILES * QP_THREADS];
    __shared__ __align__(16) uint8_t lds_level[TILES * QP_THREADS * B];

    const uint32_t tid = threadIdx.x;
    const uint32_t w = blockIdx.y;
    const int64_t chunk0 = static_cast<int64_t>(blockIdx.x) * CHUNK;
    const uint32_t n_elems = static_cast<uint32_t>(padded_elems - chunk0 < CHUNK ? padded_elems - chunk0 : CHUNK);
    const float* g = grads + static_cast<int64_t>(w) * worker_stride + chunk0;
    const int32_t* gseg = granule_cseg + (chunk0 >> 7);
    dq_bracket_block* blk = blocks + static_cast<int64_t>(w) * n_chunks + blockIdx.x;

    float4 x[TILES][2];
    qp_load<TILES>(g, tid, n_elems, x);
    __shared__ bracket_state state;
    const dq_chunk_tensor owner = dq_load_chunk_tensor(chunk_tensor, blockIdx.x);
    const float lo_one = norm_lo[static_cast<int64_t>(w) * n_seg + owner.seg], hi_one = norm_hi[static_cast<int64_t>(w) * n_seg + owner.seg];
    const int32_t one = bracketed_one_tensor_of(owner, cseg_start, cseg_valid_end);
    if (one >= 0) { // the same for the whole workgroup
        if (tid == 0) state.count = state.tickets = 0;
        __syncthreads();
        uint8_t* msg = packed + static_cast<int64_t>(w) * packed_stride;
        bracketed_one_tensor<B, LINF>(x, lo_one, hi_one, tid, chunk0, key0, key1, step, worker_base + w, &state, lds_sign,
                                      lds_level, msg + (chunk0 >> 3), msg + (padded_elems >> 3) + (chunk0 >> 3) * B, blk,
                                      &partials[static_cast<int64_t>(w) * n_slots + blockIdx.x + one]);
        return;
    }
    int32_t seg[TILES];
#pragma unroll
    for (int it = 0; it < TILES; ++it) seg[it] = gseg[qp_granule<TILES>(tid, it, n_elems)];

    const int32_t seg_first = gseg[0];
    const int32_t seg_last = gseg[(n_elems - 1) >> 7];
    int unusable = 0, whole_here = 0;
    if (static_cast<int32_t>(tid) <= seg_last - seg_first) { // at most 32 lanes, all in the first wavefront
        const int64_t at = static_cast<int64_t>(w) * n_seg + cseg_seg[seg_first + tid];
        const int64_t valid_end = cseg_valid_end[seg_first + tid];
        const bool whole = cseg_start[seg_first + tid] >= chunk0 && valid_end <= chunk0 + CHUNK;
        const float lo = norm_lo[at], hi = norm_hi[at];
        // the zero path (norm below DQ_MIN_NORM) is not monotone against the rest: no bracket across it
        const bool ok = lo >= DQ_MIN_NORM && hi >= lo && hi <= 3.0e38f; // false for NaN
        lds_scale_hi[tid] = ok ? S / lo : 0.0f; // replaced below for a tensor that is whole
        lds_scale_lo[tid] = ok ? S / hi : 0.0f;
        lds_whole[tid] = whole ? 1 : 0;
        whole_here = whole ? 1 : 0;
        unusable = (ok || whole) ? 0 : 1;
        const int64_t rel = valid_end - chunk0;
        lds_valid_end[tid] = rel < CHUNK ? static_cast<int32_t>(rel) : CHUNK;
    }
    // one lane writes both words: the first wavefront's vote says whether any tensor is whole
    const bool first_wave_any_whole = __ballot(whole_here) != 0;
    if (tid == 0) {
        lds_count = 0;
        lds_any_whole = first_wave_any_whole ? 1 : 0;
    }
    const int skip = __syncthreads_or(unusable); // also the barrier after the tables
    const bool any_whole = lds_any_whole != 0;

    // partial sums of squares (or maxima) of the chunk's tensors
    int valid[TILES], local[TILES], granule[TILES];
#pragma unroll
    for (int it = 0; it < TILES; ++it) {
        dq_arrange_wave_tile(x[it][0], x[it][1]);
        const uint32_t e = qp_elem<TILES>(tid, it);
        granule[it] = static_cast<int>(e >> 7);
        local[it] = seg[it] - seg_first;
        valid[it] = e < n_elems ? lds_valid_end[local[it]] - static_cast<int32_t>(e) : 0;
    }
    const int n_scan = dq_chunk_granule_sums<LINF>(x, valid, local, granule, static_cast<int>(tid), lds_gsum, lds_glocal,
                                                   seg_first == seg_last, static_cast<int>(n_elems >> 7));
    __syncthreads();
    if (tid < DQ_CHUNK_GRANULES)
        dq_chunk_tensor_totals<LINF>(static_cast<int>(tid), n_scan, lds_gsum, lds_glocal,
                                      [&](int j, double total) {
                                          partials[static_cast<int64_t>(w) * n_slots + blockIdx.x + seg_first + j] = total;
                                          if (lds_whole[j]) { // all of the tensor is here: this is its norm, no bracket involved
                                              const float N = LINF ? static_cast<float>(total) : static_cast<float>(sqrt(total));
                                              norms_out[static_cast<int64_t>(w) * n_seg + cseg_seg[seg_first + j]] = N;
                                              inside[static_cast<int64_t>(w) * n_cseg + seg_first + j] = 1;
                                              const float scale = N >= DQ_MIN_NORM ? S / N : 0.0f;
                                              lds_scale_hi[j] = scale;
                                              lds_scale_lo[j] = scale;
                                          }
                                      });
    if (any_whole) __syncthreads(); // uniform: scales written just above
    if (skip) { // uniform: the redo kernel quantizes this chunk from the gradient
        if (tid == 0) {
            blk->count = 0;
            blk->flags = 1;
        }
        return;
    }

    const uint32_t quad_lo0 = static_cast<uint32_t>(static_cast<uint64_t>(chunk0) >> 2);
    const uint32_t quad_hi = static_cast<uint32_t>(static_cast<uint64_t>(chunk0) >> 34);
    const uint32_t worker = worker_base + w;

#pragma unroll
    for (int it = 0; it < TILES; ++it) {
        const uint32_t e = qp_elem<TILES>(tid, it);
        if (e < n_elems) {
            const uint32_t quad = quad_lo0 + (e >> 2);
            // levels at the low end of the bracket: the largest any norm inside it can give
            uint32_t lv[2];
            float t[8];
            const qp_range range = quantize_quads<B>(x[it][0], x[it][1], lds_scale_hi[local[it]], 0.0f, 0, quad, quad + 1u,
                                                     quad_hi, worker, step, key0, key1, lv, t);
            lv[0] &= FIELDS;
            lv[1] &= FIELDS;
            const int nv = valid[it] >= QP_PER_LANE ? QP_PER_LANE : (valid[it] > 0 ? valid[it] : 0);
            uint32_t sign = quantize_sign_byte(x[it][0], x[it][1]);
            if (nv < QP_PER_LANE) { // the tensor ends inside (or before) this lane's eight elements
                sign &= (1u << nv) - 1u;
                const uint64_t fields = (static_cast<uint64_t>(1) << (nv * B)) - 1u;
                lv[0] &= static_cast<uint32_t>(fields);
                lv[1] &= static_cast<uint32_t>(fields >> (4 * B));
            }
            if ((lv[0] | lv[1]) != 0) { // a zero at the low end is a zero everywhere in the bracket
                uint32_t lv_lo[2];
                quantize_again<B>(range, x[it][0], x[it][1], lds_scale_lo[local[it]], 0.0f, 0, t, lv_lo);
                // (lv is zero past the tensor's end, so is what lv_lo has there once masked)
                const uint64_t fields = nv < QP_PER_LANE ? (static_cast<uint64_t>(1) << (nv * B)) - 1u : ~static_cast<uint64_t>(0);
                record_open<B>(lv[0] ^ (lv_lo[0] & static_cast<uint32_t>(fields) & FIELDS), x[it][0], B, e, &lds_count, blk, lv[0]);
                record_open<B>(lv[1] ^ (lv_lo[1] & static_cast<uint32_t>(fields >> (4 * B)) & FIELDS), x[it][1], B, e + 4u, &lds_count, blk, lv[1]);
            }
            const uint64_t level = static_cast<uint64_t>(lv[0]) | (static_cast<uint64_t>(lv[1]) << (4 * B));
            lds_sign[e >> 3] = static_cast<uint8_t>(sign);
            stage_bytes<B>(&lds_level[(e >> 3) * B], level);
        }
    }
    __syncthreads();

    uint8_t* msg = packed + static_cast<int64_t>(w) * packed_stride;
    qp_store_block(msg + (chunk0 >> 3), lds_sign, n_elems >> 3, tid);
    qp_store_block(msg + (padded_elems >> 3) + (chunk0 >> 3) * B, lds_level, (n_elems >> 3) * B, tid);
    if (tid == 0) {
        blk->count = lds_count;
        blk->flags = 0;
    }
}

// The first kernel with per-tensor widths (dq_widths_t: one row shared by the workers or one row per
// worker): b, the level count and the place of the level bytes of every tensor the chunk touches
// come from the widths table, as in quantize_pack_chunk_v; everything else as above.
// Seven wavefronts per SIMD as there, which the compiler takes 74 registers to miss unless told: 2^26 values, M = 16, b = 4
// 962 -> 938 us; eight spill (1393).
template <bool LINF>
__global__ __launch_bounds__(QP_THREADS, 7) void k_quantize_pack_bracketed_v(
    const float* __restrict__ grads, int64_t worker_stride, const float* __restrict__ norm_lo,
    const float* __restrict__ norm_hi, int32_t n_seg, const dq_chunk_tensor* __restrict__ chunk_tensor,
    const int32_t* __restrict__ granule_cseg, const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_start,
    const int64_t* __restrict__ cseg_valid_end, const dq_cseg_width* __restrict__ widths_table,
    int32_t widths_worker_stride, int64_t padded_elems, uint32_t key0, uint32_t key1, uint32_t step,
    uint32_t worker_base, uint8_t* __restrict__ packed, int64_t packed_stride, double* __restrict__ partials,
    int64_t n_slots, dq_bracket_block* __restrict__ blocks, int64_t n_chunks, float* __restrict__ norms_out,
    uint8_t* __restrict__ inside, int32_t n_cseg)
{
    constexpr int TILES = 2;
    constexpr int CHUNK = DQ_CHUNK;
    const dq_cseg_width* __restrict__ widths = widths_table + static_cast<int64_t>(blockIdx.y) * widths_worker_stride;

    __shared__ float lds_scale_hi[DQ_CHUNK_GRANULES];
    __shared__ float lds_scale_lo[DQ_CHUNK_GRANULES];
    __shared__ float lds_levels[DQ_CHUNK_GRANULES]; // s = 2^b - 1 of the tensor
    __shared__ int32_t lds_b[DQ_CHUNK_GRANULES];
    __shared__ int32_t lds_level_base[DQ_CHUNK_GRANULES];
    __shared__ int32_t lds_valid_end[DQ_CHUNK_GRANULES];
    __shared__ double lds_gsum[DQ_CHUNK_GRANULES];
    __shared__ int32_t lds_glocal[DQ_CHUNK_GRANULES];
    __shared__ uint32_t lds_count;
    __shared__ int32_t lds_whole[DQ_CHUNK_GRANULES];
    __shared__ int32_t lds_any_whole;
    __shared__ __align__(16) uint8_t lds_sign[TILES * QP_THREADS];
    __shared__ __align__(16) uint8_t lds_level[TILES * QP_THREADS * 8];

    const uint32_t tid = threadIdx.x;
    const uint32_t w = blockIdx.y;
    const int64_t chunk0 = static_cast<int64_t>(blockIdx.x) * CHUNK;
    const uint32_t n_elems = static_cast<uint32_t>(padded_elems - chunk0 < CHUNK ? padded_elems - chunk0 : CHUNK);
    const float* g = grads + static_cast<int64_t>(w) * worker_stride + chunk0;
    const int32_t* gseg = granule_cseg + (chunk0 >> 7);
    dq_bracket_block* blk = blocks + static_cast<int64_t>(w) * n_chunks + blockIdx.x;

    float4 x[TILES][2];
    qp_load<TILES>(g, tid, n_elems, x);
    __shared__ bracket_state state;
    const dq_chunk_tensor owner = dq_load_chunk_tensor(chunk_tensor, blockIdx.x);
    const float lo_one = norm_lo[static_cast<int64_t>(w) * n_seg + owner.seg], hi_one = norm_hi[static_cast<int64_t>(w) * n_seg + owner.seg];
    const int32_t one = bracketed_one_tensor_of(owner, cseg_start, cseg_valid_end);
    if (one >= 0) { // the same for the whole workgroup
        if (tid == 0) state.count = state.tickets = 0;
        __syncthreads();
        uint8_t* msg = packed + static_cast<int64_t>(w) * packed_stride;
        const dq_cseg_width e = widths[one];
        const int b = __builtin_amdgcn_readfirstlane(e.b);
        dq_with_width(b, [&](auto width) {
            bracketed_one_tensor<decltype(width)::value, LINF>(
                x, lo_one, hi_one, tid, chunk0, key0, key1, step, worker_base + w, &state, lds_sign, lds_level,
                msg + (chunk0 >> 3), msg + (padded_elems >> 3) + e.level_start + ((chunk0 - e.seg_start) >> 3) * b, blk,
                &partials[static_cast<int64_t>(w) * n_slots + blockIdx.x + one]);
        });
        return;
    }
    int32_t seg[TILES];
#pragma unroll
    for (int it = 0; it < TILES; ++it) seg[it] = gseg[qp_granule<TILES>(tid, it, n_elems)];

    const int32_t seg_first = gseg[0];
    const int32_t seg_last = gseg[(n_elems - 1) >> 7];
    const dq_cseg_width first = widths[seg_first];
    const int64_t chunk_level0 = first.level_start + ((chunk0 - first.seg_start) >> 3) * first.b;
    int unusable = 0, whole_here = 0;
    if (static_cast<int32_t>(tid) <= seg_last - seg_first) { // at most 32 lanes, all in the first wavefront
        const dq_cseg_width e = widths[seg_first + tid];
        const float S = static_cast<float>((1 << e.b) - 1);
        const int64_t at = static_cast<int64_t>(w) * n_seg + cseg_seg[seg_first + tid];
        const int64_t valid_end = cseg_valid_end[seg_first + tid];
        const bool whole = cseg_start[seg_first + tid] >= chunk0 && valid_end <= chunk0 + CHUNK;
        const float lo = norm_lo[at], hi = norm_hi[at];
        const bool ok = lo >= DQ_MIN_NORM && hi >= lo && hi <= 3.0e38f;
        lds_scale_hi[tid] = ok ? S / lo : 0.0f;
        lds_scale_lo[tid] = ok ? S / hi : 0.0f;
        lds_levels[tid] = S;
        lds_b[tid] = e.b;
        lds_level_base[tid] = static_cast<int32_t>(e.level_start + ((chunk0 - e.seg_start) >> 3) * e.b - chunk_level0);
        lds_whole[tid] = whole ? 1 : 0;
        whole_here = whole ? 1 : 0;
        unusable = (ok || whole) ? 0 : 1;
        const int64_t rel = valid_end - chunk0;
        lds_valid_end[tid] = rel < CHUNK ? static_cast<int32_t>(rel) : CHUNK;
    }
    const bool first_wave_any_whole = __ballot(whole_here) != 0;
    if (tid == 0) {
        lds_count = 0;
        lds_any_whole = first_wave_any_whole ? 1 : 0;
    }
    const int skip = __syncthreads_or(unusable);
    const bool any_whole = lds_any_whole != 0;

    int valid[TILES], local[TILES], granule[TILES];
#pragma unroll
    for (int it = 0; it < TILES; ++it) {
        dq_arrange_wave_tile(x[it][0], x[it][1]);
        const uint32_t e = qp_elem<TILES>(tid, it);
        granule[it] = static_cast<int>(e >> 7);
        local[it] = seg[it] - seg_first;
        valid[it] = e < n_elems ? lds_valid_end[local[it]] - static_cast<int32_t>(e) : 0;
    }
    const int n_scan = dq_chunk_granule_sums<LINF>(x, valid, local, granule, static_cast<int>(tid), lds_gsum, lds_glocal,
                                                   seg_first == seg_last, static_cast<int>(n_elems >> 7));
    __syncthreads();
    if (tid < DQ_CHUNK_GRANULES)
        dq_chunk_tensor_totals<LINF>(static_cast<int>(tid), n_scan, lds_gsum, lds_glocal,
                                     [&](int j, double total) {
                                         partials[static_cast<int64_t>(w) * n_slots + blockIdx.x + seg_first + j] = total;
                                         if (lds_whole[j]) {
                                             const float N = LINF ? static_cast<float>(total) : static_cast<float>(sqrt(total));
                                             norms_out[static_cast<int64_t>(w) * n_seg + cseg_seg[seg_first + j]] = N;
                                             inside[static_cast<int64_t>(w) * n_cseg + seg_first + j] = 1;
                                             const float scale = N >= DQ_MIN_NORM ? lds_levels[j] / N : 0.0f;
                                             lds_scale_hi[j] = scale;
                                             lds_scale_lo[j] = scale;
                                         }
                                     });
    if (any_whole) __syncthreads();
    if (skip) {
        if (tid == 0) {
            blk->count = 0;
            blk->flags = 1;
        }
        return;
    }

    const uint32_t quad_lo0 = static_cast<uint32_t>(static_cast<uint64_t>(chunk0) >> 2);
    const uint32_t quad_hi = static_cast<uint32_t>(static_cast<uint64_t>(chunk0) >> 34);
    const uint32_t worker = worker_base + w;

#pragma unroll
    for (int it = 0; it < TILES; ++it) {
        const uint32_t e = qp_elem<TILES>(tid, it);
        if (e < n_elems) {
            const float S = lds_levels[local[it]];
            const int b = lds_b[local[it]];
            const uint32_t FIELDS = quad_fields<0>(b);
            const uint32_t quad = quad_lo0 + (e >> 2);
            uint32_t lv[2];
            float t[8];
            const qp_range range = quantize_quads<0>(x[it][0], x[it][1], lds_scale_hi[local[it]], S, b, quad, quad + 1u,
                                                     quad_hi, worker, step, key0, key1, lv, t);
            const int left = lds_valid_end[local[it]] - static_cast<int32_t>(e); // read again: seven wavefronts leave no register for it
            const int nv = left >= QP_PER_LANE ? QP_PER_LANE : (left > 0 ? left : 0);
            uint32_t sign = quantize_sign_byte(x[it][0], x[it][1]);
            if (nv < QP_PER_LANE) { // the tensor ends inside (or before) this lane's eight elements
                sign &= (1u << nv) - 1u;
                const uint64_t fields = (static_cast<uint64_t>(1) << (nv * b)) - 1u;
                lv[0] &= static_cast<uint32_t>(fields) & FIELDS;
                lv[1] &= static_cast<uint32_t>(fields >> (4 * b));
            }
            if ((lv[0] | lv[1]) != 0) { // a zero at the low end is a zero everywhere in the bracket
                uint32_t lv_lo[2];
                quantize_again<0>(range, x[it][0], x[it][1], lds_scale_lo[local[it]], S, b, t, lv_lo);
                // (lv is zero past the tensor's end, so is what lv_lo has there once masked)
                const uint64_t fields = nv < QP_PER_LANE ? (static_cast<uint64_t>(1) << (nv * b)) - 1u : ~static_cast<uint64_t>(0);
                record_open<0>(lv[0] ^ (lv_lo[0] & static_cast<uint32_t>(fields) & FIELDS), x[it][0], b, e, &lds_count, blk, lv[0]);
                record_open<0>(lv[1] ^ (lv_lo[1] & static_cast<uint32_t>(fields >> (4 * b))), x[it][1], b, e + 4u, &lds_count, blk, lv[1]);
            }
            const uint64_t level = static_cast<uint64_t>(lv[0]) | (static_cast<uint64_t>(lv[1]) << (4 * b));
            lds_sign[e >> 3] = static_cast<uint8_t>(sign);
            stage_bytes_v(&lds_level[lds_level_base[local[it]] + static_cast<int32_t>(e >> 3) * b], level, b);
        }
    }
    __syncthreads();

    uint8_t* msg = packed + static_cast<int64_t>(w) * packed_stride;
    const int last = seg_last - seg_first;
    qp_store_block(msg + (chunk0 >> 3), lds_sign, n_elems >> 3, tid);
    qp_store_block(msg + (padded_elems >> 3) + chunk_level0, lds_level,
                   static_cast<uint32_t>(lds_level_base[last]) + (n_elems >> 3) * lds_b[last], tid);
    if (tid == 0) {
        blk->count = lds_count;
        blk->flags = 0;
    }
}

// grid (n_span, M), the tensors that cross a chunk boundary (the others are finished by the first
// kernel): the norm of tensor c of worker w from its partial sums (or maxima), slots
// [first chunk + c, last chunk + c]: eight lane-strided running sums per lane, combined in a fixed
// order, then a fixed tree over the lanes.  Also notes whether the norm lies inside its bracket.
template <bool LINF>
__global__ __launch_bounds__(256) void k_bracket_norm_finish(
    const double* __restrict__ partials, int64_t n_slots, const int64_t* __restrict__ cseg_start,
    const int64_t* __restrict__ cseg_valid_end, const int32_t* __restrict__ cseg_seg, const int32_t* __restrict__ span_cseg,
    int32_t n_seg, int32_t n_cseg, const float* __restrict__ norm_lo, const float* __restrict__ norm_hi,
    float* __restrict__ norms, uint8_t* __restrict__ inside)
{
    __shared__ double part[256];
    const int tid = threadIdx.x;
    const int32_t c = span_cseg[blockIdx.x];
    const int w = blockIdx.y;
    const int64_t first = cseg_start[c] / DQ_CHUNK;
    const int64_t last = (cseg_valid_end[c] - 1) / DQ_CHUNK;
    const double* p = partials + static_cast<int64_t>(w) * n_slots + first + c;
    const int64_t n = last - first + 1;
    double acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.0;
    int64_t i = tid;
    for (; i + 7 * 256 < n; i += 8 * 256) {
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] = dq_chunk_combine<LINF>(acc[k], p[i + k * 256]);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) // fewer than eight are left
        if (i + k * 256 < n) acc[k] = dq_chunk_combine<LINF>(acc[k], p[i + k * 256]);
    part[tid] = dq_chunk_combine<LINF>(
        dq_chunk_combine<LINF>(dq_chunk_combine<LINF>(acc[0], acc[1]), dq_chunk_combine<LINF>(acc[2], acc[3])),
        dq_chunk_combine<LINF>(dq_chunk_combine<LINF>(acc[4], acc[5]), dq_chunk_combine<LINF>(acc[6], acc[7])));
    __syncthreads();
    for (int off = 128; off >= 1; off >>= 1) {
        if (tid < off) part[tid] = dq_chunk_combine<LINF>(part[tid], part[tid + off]);
        __syncthreads();
    }
    if (tid == 0) {
        const int64_t at = static_cast<int64_t>(w) * n_seg + cseg_seg[c];
        const float N = LINF ? static_cast<float>(part[0]) : static_cast<float>(sqrt(part[0]));
        norms[at] = N;
        inside[static_cast<int64_t>(w) * n_cseg + c] = (N >= norm_lo[at] && N <= norm_hi[at]) ? 1 : 0;
    }
}

// One recorded element of tensor c with norm N: its level, ORed into the zero field the first kernel left.
// B = 0: per-tensor widths, b and the place of the tensor's level fields come from `widths` (this
// worker's row of the table).
template <int B>
__device__ __forceinline__ void settle_element(uint2 rec, int64_t chunk0, int32_t c, float N, uint32_t key0, uint32_t key1,
                                               uint32_t step, uint32_t worker, uint32_t* __restrict__ plane,
                                               const dq_cseg_width* __restrict__ widths)
{
    const uint64_t P = static_cast<uint64_t>(chunk0) + rec.x;
    uint32_t r[4];
    dq_philox4x32_10(static_cast<uint32_t>(P >> 2), static_cast<uint32_t>(P >> 34), worker, step, key0, key1, r);
    const uint32_t word = (P & 2u) ? ((P & 1u) ? r[3] : r[2]) : ((P & 1u) ? r[1] : r[0]);
    uint32_t level;
    uint64_t bit;
    int b;
    if constexpr (B == 0) {
        const dq_cseg_width wd = widths[c];
        b = wd.b;
        const float S = static_cast<float>((1 << b) - 1);
        level = level_of_s(__uint_as_float(rec.y), N >= DQ_MIN_NORM ? S / N : 0.0f, S, word);
        bit = static_cast<uint64_t>(wd.level_start) * 8u + (P - static_cast<uint64_t>(wd.seg_start)) * static_cast<uint64_t>(b);
    } else {
        constexpr float S = static_cast<float>((1 << B) - 1);
        b = B;
        level = level_of<B>(__uint_as_float(rec.y), N >= DQ_MIN_NORM ? S / N : 0.0f, word);
        bit = P * B;
    }
    if (level != 0) {
        // fields of other elements in the same words are not touched
        const uint32_t sh = static_cast<uint32_t>(bit & 31u);
        atomicOr(plane + (bit >> 5), level << sh);
        if (sh + b > 32) atomicOr(plane + (bit >> 5) + 1, level >> (32 - sh));
    }
}

// The same, with the element's tensor looked up first.
template <int B>
__device__ __forceinline__ void settle_record(uint2 rec, int64_t chunk0, uint32_t w, const float* __restrict__ norms,
                                              int32_t n_seg, const int32_t* __restrict__ granule_cseg,
                                              const int32_t* __restrict__ cseg_seg, uint32_t key0, uint32_t key1,
                                              uint32_t step, uint32_t worker, uint32_t* __restrict__ plane,
                                              const dq_cseg_width* __restrict__ widths)
{
    const uint32_t e = rec.x; // < 4096 and inside the layout: written by the first kernel for this chunk
    const int32_t c = granule_cseg[(chunk0 >> 7) + (e >> 7)];
    settle_element<B>(rec, chunk0, c, norms[static_cast<int64_t>(w) * n_seg + cseg_seg[c]], key0, key1, step, worker, plane, widths);
}

// What the settle kernels decide per chunk: true if the chunk has to be quantized again.
__device__ __forceinline__ bool chunk_needs_redo(uint32_t count, uint32_t flags, int64_t chunk0, int64_t padded_elems,
                                                 uint32_t w, int32_t n_cseg, const int32_t* __restrict__ granule_cseg,
                                                 const uint8_t* __restrict__ inside)
{
    const int64_t last_granule = ((chunk0 + DQ_CHUNK < padded_elems ? chunk0 + DQ_CHUNK : padded_elems) - 1) >> 7;
    const int32_t c_first = granule_cseg[chunk0 >> 7], c_last = granule_cseg[last_granule];
    bool again = flags != 0 || count > DQ_BRACKET_CAP;
    for (int32_t c = c_first; c <= c_last; ++c) again = again || inside[static_cast<int64_t>(w) * n_cseg + c] == 0;
    return again;
}

// grid (ceil(n_chunks / 4), M), one wavefront per chunk and one lane per record, and the workgroup itself
// quantizes those of its four chunks again that need it: for plans of moderate size, where a launch of
// that many workgroups is cheap and a chunk may hold dozens of records.  One launch where clearing the redo
// map, settling and walking the map were three: the lagged iteration of the ResNet-18 shape, M = 8, b = 3
// takes 131.5 us instead of 135.5.
// A workgroup quantizes its flagged chunks one after the other.  Against three launches, with a workgroup of its own for
// every flagged chunk, whole calls in us (among them what the first kernel gained): ResNet-18 shape, M = 8, b = 3 norms
// inside their brackets 119 -> 109, all outside 188 -> 172, one worker's outside 130 -> 116; b = 6 at +-12.5 % (a fifth of
// the chunks again) 156 -> 146; transformer shape, M = 16, b = 8 (two fifths) 319 -> 293; 2^20 elements of one worker inside
// 17.8 -> 12.6, all outside 18.7 -> 17.1.
// What bounds it: memory latency.  A chunk of one tensor (nearly all) gets norm and bracket test from the chunk table beside
// its block instead of by granule, record and tensor in turn, and the quantizer's lane arithmetic stays inside the loop
// (66 to 72 registers, were 82 to 98): ResNet-18 shape, M = 8, b = 2 18.9 -> 14.7 us, b = 3 20.4 -> 15.4, b = 5 30.3 -> 25.1.
// Two chunks to a wavefront: 12.1, 14.7, but 32.6 where a fifth are taken again (a workgroup takes its chunks in turn).
// FOLD: k_bracket_norm_finish is not launched; a wavefront adds the partial sums of its chunk's tensors itself (up to two of them
// go on beyond the chunk), and the one with a tensor's first chunk writes the norm.  That reads a tensor's sums once per chunk and
// worker, a few KB from the L2, in place of a launch.  Lagged iterations, us, up to the line (one round of the
// kernel's wavefronts): 4197 elements, M = 2 b = 2 25.2 -> 21.0, 2^20, M = 4 25.1 -> 21.2, 0.5 M ragged, M = 8 24.7 -> 21.4, 2^22, M = 4 31.4 -> 30.1;
// beyond it every further round pays for the sums: 2^22, M = 8 45.6 -> 46.0, M = 16 77.0 -> 79.0, ResNet-18 shape, M = 8 b = 3 114.4 -> 118.4.
constexpr int SETTLE_FOLD_CHUNKS = 1024; // 16 sums a lane
constexpr int64_t SETTLE_FOLD_PAIRS = 6144; // (worker, chunk) pairs
struct bracket_finish { // what k_bracket_norm_finish takes
    const double* partials;
    int64_t n_slots;
    const int64_t* cseg_start;
    const float* norm_lo;
    const float* norm_hi;
    float* norms;
    int linf;
};

// The sum (or maximum) of a tensor's n <= SETTLE_FOLD_CHUNKS slots, in every lane: the additions of k_bracket_norm_finish in its
// order (four lanes of its 256 to one here), so the same bits.
template <bool LINF>
__device__ __forceinline__ double bracket_slots_total(const double* __restrict__ p, int n, int lane)
{
    double part[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        double v[4] = { 0.0, 0.0, 0.0, 0.0 };
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = lane + 64 * q + 256 * k;
            if (i < n) v[k] = p[i];
        }
        part[q] = dq_chunk_combine<LINF>(dq_chunk_combine<LINF>(v[0], v[1]), dq_chunk_combine<LINF>(v[2], v[3]));
    }
    double total = dq_chunk_combine<LINF>(dq_chunk_combine<LINF>(part[0], part[2]), dq_chunk_combine<LINF>(part[1], part[3]));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) total = dq_chunk_combine<LINF>(total, __shfl_down(total, off, 64));
    return __longlong_as_double(static_cast<long long>(
        (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint64_t>(__double_as_longlong(total)) >> 32)))) << 32) |
        static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint64_t>(__double_as_longlong(total)))))));
}

// Norms that a wavefront has worked out: of segment seg[k], N[k] (seg -1: none).
struct bracket_norms {
    int32_t seg[2];
    float N[2];
    __device__ __forceinline__ float operator()(const float* row, int32_t s) const
    {
        return s == seg[0] ? N[0] : s == seg[1] ? N[1] : row[s];
    }
};

// Tensor c (the same for the whole wavefront) of worker w, if it goes on beyond the chunk at chunk0: its norm as entry k of `out`,
// written to the caller's norms if this is its first chunk.  Returns whether the norm lies inside its bracket (true for a tensor
// that lies wholly inside the chunk: the first kernel has finished and used its norm).
__device__ __forceinline__ bool bracket_finish_tensor(const bracket_finish& f, int32_t c, uint32_t w, int64_t chunk0, int32_t n_seg,
                                                      const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_valid_end,
                                                      int lane, int k, bracket_norms& out)
{
    const int64_t start = f.cseg_start[c], end = cseg_valid_end[c];
    const int32_t seg = cseg_seg[c];
    const int64_t first = start / DQ_CHUNK, n = (end - 1) / DQ_CHUNK - first + 1;
    out.seg[k] = -1;
    if (n == 1) return true;
    const double* p = f.partials + static_cast<int64_t>(w) * f.n_slots + first + c;
    const int64_t at = static_cast<int64_t>(w) * n_seg + seg;
    const float lo = f.norm_lo[at], hi = f.norm_hi[at];
    const float N = f.linf ? static_cast<float>(bracket_slots_total<true>(p, static_cast<int>(n), lane))
                           : static_cast<float>(sqrt(bracket_slots_total<false>(p, static_cast<int>(n), lane)));
    out.seg[k] = seg;
    out.N[k] = N;
    if (first * DQ_CHUNK + DQ_CHUNK > chunk0 && lane == 0) f.norms[at] = N;
    return N >= lo && N <= hi;
}

template <int B, bool FOLD>
__global__ __launch_bounds__(QP_THREADS) void k_bracket_settle_redo(
    const float* __restrict__ grads, int64_t worker_stride, const float* __restrict__ norms, int32_t n_seg,
    int32_t n_cseg, const dq_chunk_tensor* __restrict__ chunk_tensor, const int32_t* __restrict__ granule_cseg,
    const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems, uint32_t key0,
    uint32_t key1, uint32_t step, uint32_t worker_base, uint8_t* __restrict__ packed, int64_t packed_stride,
    dq_bracket_block* __restrict__ blocks, int64_t n_chunks, const uint8_t* __restrict__ inside,
    const dq_cseg_width* __restrict__ widths_table, int32_t widths_worker_stride, const bracket_finish finish)
{
    constexpr int WAVES = QP_THREADS / 64;
    __shared__ int lds_again[WAVES];
    __shared__ bracket_norms lds_norms[FOLD ? WAVES : 1];
    const dq_cseg_width* __restrict__ widths = widths_table + static_cast<int64_t>(blockIdx.y) * widths_worker_stride;
    const uint32_t w = blockIdx.y;
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t chunk_first = static_cast<int64_t>(blockIdx.x) * WAVES, chunk = chunk_first + wave;
    // all that the wavefront needs, in flight together; past the last chunk it is the last one's, and not used
    const int64_t own = chunk < n_chunks ? chunk : n_chunks - 1;
    dq_bracket_block* blk = blocks + static_cast<int64_t>(w) * n_chunks + own;
    const dq_chunk_tensor owner = dq_load_chunk_tensor(chunk_tensor, own);
    const uint2 rec = blk->rec[lane < DQ_BRACKET_CAP ? lane : 0];
    const uint32_t count = blk->count, flags = blk->flags;
    const float* row = norms + static_cast<int64_t>(w) * n_seg;
    const int64_t chunk0 = chunk * DQ_CHUNK;
    bool again = false;
    bracket_norms own_norms = { { -1, -1 }, { 0.0f, 0.0f } };
    float N = 0.0f;     // of the chunk's only tensor, if it has one,
    uint32_t in = 0;    // and whether it lies inside its bracket
    if constexpr (!FOLD) {
        N = row[owner.seg];
        in = inside[static_cast<int64_t>(w) * n_cseg + (owner.cseg >= 0 ? owner.cseg : 0)];
    }
    if (chunk < n_chunks) { // the same for the whole wavefront
        again = flags != 0 || count > DQ_BRACKET_CAP;
        if constexpr (FOLD) {
            if (owner.cseg >= 0) {
                again = !bracket_finish_tensor(finish, owner.cseg, w, chunk0, n_seg, cseg_seg, cseg_valid_end, lane, 0, own_norms) || again;
                N = own_norms.N[0]; // a tensor of this one chunk has no records
            } else {
                const int64_t last_granule = ((chunk0 + DQ_CHUNK < padded_elems ? chunk0 + DQ_CHUNK : padded_elems) - 1) >> 7;
                const int32_t c_first = granule_cseg[chunk0 >> 7], c_last = granule_cseg[last_granule];
                again = !bracket_finish_tensor(finish, c_first, w, chunk0, n_seg, cseg_seg, cseg_valid_end, lane, 0, own_norms) || again;
                if (c_last != c_first)
                    again = !bracket_finish_tensor(finish, c_last, w, chunk0, n_seg, cseg_seg, cseg_valid_end, lane, 1, own_norms) || again;
            }
        } else if (owner.cseg >= 0) {
            again = again || in == 0;
        } else {
            again = chunk_needs_redo(count, flags, chunk0, padded_elems, w, n_cseg, granule_cseg, inside);
        }
        if (again) {
            if (lane == 0) blk->flags = flags | 2u;
        } else if (lane < count) {
            uint32_t* plane = reinterpret_cast<uint32_t*>(packed + static_cast<int64_t>(w) * packed_stride + (padded_elems >> 3));
            if (owner.cseg >= 0) {
                settle_element<B>(rec, chunk0, owner.cseg, N, key0, key1, step, worker_base + w, plane, widths);
            } else if constexpr (FOLD) { // the record's tensor first (rec.x < 4096 and inside the layout: the first kernel wrote it)
                const int32_t c = granule_cseg[(chunk0 >> 7) + (rec.x >> 7)];
                settle_element<B>(rec, chunk0, c, own_norms(row, cseg_seg[c]), key0, key1, step, worker_base + w, plane, widths);
            } else {
                settle_record<B>(rec, chunk0, w, norms, n_seg, granule_cseg, cseg_seg, key0, key1, step, worker_base + w, plane,
                                 widths);
            }
        }
    }
    if (lane == 0) {
        lds_again[wave] = again ? 1 : 0;
        if constexpr (FOLD) lds_norms[wave] = own_norms;
    }
    __syncthreads();
    for (int k = 0; k < WAVES; ++k) {
        if (__builtin_amdgcn_readfirstlane(lds_again[k]) == 0) continue; // the same for the whole workgroup
        const uint32_t c = static_cast<uint32_t>(chunk_first) + k;
        auto redo = [&](auto norm_of) {
            if constexpr (B == 0)
                quantize_pack_chunk_v<2, 0>(grads, worker_stride, norms, n_seg, chunk_tensor, granule_cseg, cseg_seg, cseg_valid_end,
                                            widths_table, widths_worker_stride, padded_elems, key0, key1, step, worker_base,
                                            packed, packed_stride, nullptr, c, qp_tid_in_loop(), norm_of);
            else
                quantize_pack_chunk<B, 2, 0>(grads, worker_stride, norms, n_seg, chunk_tensor, granule_cseg, cseg_seg,
                                             cseg_valid_end, padded_elems, key0, key1, step, worker_base, packed, packed_stride,
                                             nullptr, c, qp_tid_in_loop(), norm_of);
        };
        if constexpr (FOLD)
            redo(lds_norms[k]);
        else
            redo(qp_norm_given{});
        __syncthreads(); // the chunk's staging in LDS is reused by the next one
    }
}

// grid (ceil(n_chunks / 256), M), one lane per chunk: for large plans with few records per chunk.
template <int B>
__global__ __launch_bounds__(256) void k_bracket_settle(
    const float* __restrict__ norms, int32_t n_seg, int32_t n_cseg, const int32_t* __restrict__ granule_cseg,
    const int32_t* __restrict__ cseg_seg, int64_t padded_elems, uint32_t key0, uint32_t key1, uint32_t step,
    uint32_t worker_base, uint8_t* __restrict__ packed, int64_t packed_stride, dq_bracket_block* __restrict__ blocks,
    int64_t n_chunks, const uint8_t* __restrict__ inside, unsigned long long* __restrict__ redo_map, int64_t n_words,
    const dq_cseg_width* __restrict__ widths_table, int32_t widths_worker_stride)
{
    const dq_cseg_width* __restrict__ widths = widths_table + static_cast<int64_t>(blockIdx.y) * widths_worker_stride;
    const uint32_t w = blockIdx.y;
    const int64_t chunk = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const bool active = chunk < n_chunks;
    bool again = false;
    if (active) {
        dq_bracket_block* blk = blocks + static_cast<int64_t>(w) * n_chunks + chunk;
        const uint32_t count = blk->count, flags = blk->flags;
        const int64_t chunk0 = chunk * DQ_CHUNK;
        again = chunk_needs_redo(count, flags, chunk0, padded_elems, w, n_cseg, granule_cseg, inside);
        if (again) {
            blk->flags = flags | 2u;
        } else {
            uint32_t* plane = reinterpret_cast<uint32_t*>(packed + static_cast<int64_t>(w) * packed_stride +
                                                          (padded_elems >> 3));
            for (uint32_t k = 0; k < count; ++k)
                settle_record<B>(blk->rec[k], chunk0, w, norms, n_seg, granule_cseg, cseg_seg, key0, key1, step,
                                 worker_base + w, plane, widths);
        }
    }
    // 64 consecutive chunks per wavefront: one word of the redo map (blockDim is a multiple of 64)
    const unsigned long long bits = __ballot(active && again);
    if ((threadIdx.x & 63) == 0 && (chunk >> 6) < n_words) redo_map[static_cast<int64_t>(w) * n_words + (chunk >> 6)] = bits;
}

// grid (ceil(n_words / REDO_WORDS), M): each workgroup walks REDO_WORDS words of the redo map and
// quantizes the chunks whose bit is set.
constexpr int REDO_WORDS = 8;
// Up to this many (worker, chunk) pairs one kernel settles and quantizes again, a wavefront per chunk.  At 2^16 pairs
// (2^26 elements, M = 4, b = 4) it takes 261 us where the separate kernels take 249 if nothing is quantized again, 443
// against 1062 if everything is, and 303 against 1059 for one worker's quarter; at 2^15 134 against 131, and 230 against
// 954.  Beyond, settling a chunk per wavefront costs more (at 2^20 pairs 0.32 ms against 0.055).
constexpr int64_t SETTLE_WIDE_MAX = 1 << 16;

template <int B>
__global__ __launch_bounds__(QP_THREADS) void k_bracket_redo(
    const float* __restrict__ grads, int64_t worker_stride, const float* __restrict__ norms, int32_t n_seg,
    const dq_chunk_tensor* __restrict__ chunk_tensor, const int32_t* __restrict__ granule_cseg,
    const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems, uint32_t key0, uint32_t key1, uint32_t step,
    uint32_t worker_base, uint8_t* __restrict__ packed, int64_t packed_stride,
    const unsigned long long* __restrict__ redo_map, int64_t n_words, const dq_cseg_width* __restrict__ widths_table,
    int32_t widths_worker_stride)
{
    const int64_t word0 = static_cast<int64_t>(blockIdx.x) * REDO_WORDS;
    const unsigned long long* map = redo_map + static_cast<int64_t>(blockIdx.y) * n_words;
    for (int k = 0; k < REDO_WORDS && word0 + k < n_words; ++k) {
        // the same value in every lane (one address), made scalar so that the loop below is uniform
        const unsigned long long loaded = map[word0 + k];
        unsigned long long bits =
            (static_cast<unsigned long long>(__builtin_amdgcn_readfirstlane(static_cast<int>(loaded >> 32))) << 32) |
            static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(loaded)));
        while (bits != 0) {
            const int bit = __builtin_ctzll(bits);
            bits &= bits - 1;
            const uint32_t chunk = static_cast<uint32_t>((word0 + k) * 64 + bit);
            if constexpr (B == 0)
                quantize_pack_chunk_v<2, 0>(grads, worker_stride, norms, n_seg, chunk_tensor, granule_cseg, cseg_seg, cseg_valid_end,
                                            widths_table, widths_worker_stride, padded_elems, key0, key1, step,
                                            worker_base, packed, packed_stride, nullptr, chunk, qp_tid_in_loop());
            else
                quantize_pack_chunk<B, 2, 0>(grads, worker_stride, norms, n_seg, chunk_tensor, granule_cseg, cseg_seg, cseg_valid_end,
                                             padded_elems, key0, key1, step, worker_base, packed, packed_stride, nullptr,
                                             chunk, qp_tid_in_loop());
            __syncthreads(); // the chunk's staging in LDS is reused by the next one
        }
    }
}

// Statistics of one call, from the blocks: elements settled afterwards and chunks quantized again.
// 256 workgroups at most add their totals to the two counters.
constexpr int BS_PER_LANE = 16;

__global__ __launch_bounds__(256) void k_bracket_stats(const dq_bracket_block* __restrict__ blocks, int64_t n_blocks,
                                                       unsigned long long* __restrict__ stats)
{
    __shared__ unsigned long long part[2][256];
    const int tid = threadIdx.x;
    unsigned long long settled = 0, again = 0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + tid; i < n_blocks;
         i += static_cast<int64_t>(gridDim.x) * 256) {
        const uint32_t count = blocks[i].count, flags = blocks[i].flags;
        if (flags & 2u)
            ++again;
        else
            settled += count;
    }
    part[0][tid] = settled;
    part[1][tid] = again;
    __syncthreads();
    for (int off = 128; off >= 1; off >>= 1) {
        if (tid < off) {
            part[0][tid] += part[0][tid + off];
            part[1][tid] += part[1][tid + off];
        }
        __syncthreads();
    }
    if (tid == 0) {
        if (part[0][0]) atomicAdd(&stats[0], part[0][0]);
        if (part[1][0]) atomicAdd(&stats[1], part[1][0]);
    }
}

__global__ void k_zero_two(unsigned long long* __restrict__ stats)
{
    stats[threadIdx.x] = 0;
}

// B = 0: per-tensor widths from `widths_table` (row stride `widths_row`: 0 when the workers share a row)
template <int B, bool LINF>
int launch_bracketed(const dq_plan* plan, const float* grads, int64_t worker_stride, int M, const float* norm_lo,
                     const float* norm_hi, uint64_t seed, uint32_t step, uint32_t worker_base, float* norms,
                     uint8_t* packed, int64_t packed_stride, void* workspace, unsigned long long* stats,
                     hipStream_t stream, const dq_cseg_width* widths_table = nullptr, int32_t widths_row = 0)
{
    const dq_bracket_layout L = dq_bracket_layout_of(plan, M);
    if (L.n_chunks > INT32_MAX) return DQ_ERR_INVALID_ARG;
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    double* partials = reinterpret_cast<double*>(ws);
    dq_bracket_block* blocks = reinterpret_cast<dq_bracket_block*>(ws + L.blocks_at);
    uint8_t* inside = ws + L.inside_at;
    unsigned long long* redo_map = reinterpret_cast<unsigned long long*>(ws + L.redo_at);
    const dim3 grid(static_cast<unsigned>(L.n_chunks), M), block(QP_THREADS);
    const uint32_t key0 = static_cast<uint32_t>(seed), key1 = static_cast<uint32_t>(seed >> 32);
    if constexpr (B == 0)
        hipLaunchKernelGGL(k_quantize_pack_bracketed_v<LINF>, grid, block, 0, stream, grads, worker_stride, norm_lo, norm_hi,
                           plan->n_seg, plan->d_chunk_tensor, plan->d_granule_cseg, plan->d_cseg_seg, plan->d_cseg_start, plan->d_cseg_valid_end,
                           widths_table, widths_row, plan->padded_elems, key0, key1, step, worker_base, packed,
                           packed_stride, partials, L.n_slots, blocks, L.n_chunks, norms, inside, plan->n_cseg);
    else
        hipLaunchKernelGGL((k_quantize_pack_bracketed<(B == 0 ? 1 : B), LINF>), grid, block, 0, stream, grads, worker_stride,
                           norm_lo, norm_hi, plan->n_seg, plan->d_chunk_tensor, plan->d_granule_cseg, plan->d_cseg_seg, plan->d_cseg_start,
                           plan->d_cseg_valid_end, plan->padded_elems, key0, key1, step, worker_base, packed,
                           packed_stride, partials, L.n_slots, blocks, L.n_chunks, norms, inside, plan->n_cseg);
    const bool wide = static_cast<int64_t>(M) * L.n_chunks <= SETTLE_WIDE_MAX;
    const bool fold = static_cast<int64_t>(M) * L.n_chunks <= SETTLE_FOLD_PAIRS && plan->n_span > 0 && plan->span_chunks <= SETTLE_FOLD_CHUNKS;
    if (plan->n_span > 0 && !fold)
        hipLaunchKernelGGL(k_bracket_norm_finish<LINF>, dim3(plan->n_span, M), dim3(256), 0, stream, partials, L.n_slots,
                           plan->d_cseg_start, plan->d_cseg_valid_end, plan->d_cseg_seg, plan->d_span_cseg, plan->n_seg,
                           plan->n_cseg, norm_lo, norm_hi, norms, inside);
    if (wide) {
        const bracket_finish finish = { partials, L.n_slots, plan->d_cseg_start, norm_lo, norm_hi, norms, LINF ? 1 : 0 };
        auto settle = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((L.n_chunks + 3) / 4), M), block, 0, stream, grads, worker_stride,
                               norms, plan->n_seg, plan->n_cseg, plan->d_chunk_tensor, plan->d_granule_cseg, plan->d_cseg_seg,
                               plan->d_cseg_valid_end, plan->padded_elems, key0, key1, step, worker_base, packed, packed_stride, blocks,
                               L.n_chunks, inside, widths_table, widths_row, finish);
        };
        if (fold)
            settle(k_bracket_settle_redo<B, true>);
        else
            settle(k_bracket_settle_redo<B, false>);
    } else {
        hipLaunchKernelGGL(k_bracket_settle<B>, dim3(static_cast<unsigned>((L.n_chunks + 255) / 256), M), dim3(256), 0,
                           stream, norms, plan->n_seg, plan->n_cseg, plan->d_granule_cseg, plan->d_cseg_seg,
                           plan->padded_elems, key0, key1, step, worker_base, packed, packed_stride, blocks, L.n_chunks,
                           inside, redo_map, L.n_words, widths_table, widths_row);
        hipLaunchKernelGGL(k_bracket_redo<B>, dim3(static_cast<unsigned>((L.n_words + REDO_WORDS - 1) / REDO_WORDS), M),
                           block, 0, stream, grads, worker_stride, norms, plan->n_seg, plan->d_chunk_tensor, plan->d_granule_cseg,
                           plan->d_cseg_seg, plan->d_cseg_valid_end, plan->padded_elems, key0, key1, step, worker_base,
                           packed, packed_stride, redo_map, L.n_words, widths_table, widths_row);
    }
    if (stats) {
        const int64_t n_blocks = static_cast<int64_t>(M) * L.n_chunks;
        const int64_t wgs = (n_blocks + 256 * BS_PER_LANE - 1) / (256 * BS_PER_LANE);
        hipLaunchKernelGGL(k_zero_two, dim3(1), dim3(2), 0, stream, stats);
        hipLaunchKernelGGL(k_bracket_stats, dim3(static_cast<unsigned>(wgs < 256 ? wgs : 256)), dim3(256), 0, stream,
                           blocks, n_blocks, stats);
    }
    return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
}

} // namespace

namespace {

__global__ __launch_bounds__(256) void k_norm_bracket(const float* __restrict__ norms, int64_t n, float below, float above,
                                                      float* __restrict__ lo, float* __restrict__ hi)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) {
        const float N = norms[i];
        lo[i] = N * below;
        hi[i] = N * above;
    }
}

} // namespace

extern "C" int dq_norm_bracket(const float* norms_dev, int64_t n, float margin, float* norm_lo_dev, float* norm_hi_dev,
                               void* hip_stream)
{
    if (!norms_dev || !norm_lo_dev || !norm_hi_dev || n < 0 || n > (INT64_C(1) << 38)) return DQ_ERR_INVALID_ARG;
    if (!(margin >= 0.0f) || !(margin < 1.0f)) return DQ_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(norms_dev) & 3u) || (reinterpret_cast<uintptr_t>(norm_lo_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(norm_hi_dev) & 3u))
        return DQ_ERR_INVALID_ARG;
    if (n == 0) return DQ_OK;
    dq_forget_earlier_errors();
    hipLaunchKernelGGL(k_norm_bracket, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0,
                       static_cast<hipStream_t>(hip_stream), norms_dev, n, 1.0f - margin, 1.0f + margin, norm_lo_dev,
                       norm_hi_dev);
    return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
}

extern "C" int64_t dq_bracketed_workspace_bytes(const dq_plan_t* plan, int M)
{
    if (!plan || M < 1 || M > DQ_MAX_WORKERS) return -1;
    return dq_bracket_layout_of(plan, M).total;
}

extern "C" int dq_norm_quantize_pack_bracketed(const dq_plan_t* plan, const float* grads_dev,
                                               int64_t worker_stride_elems, int M, int linf, const float* norm_lo_dev,
                                               const float* norm_hi_dev, int b, uint64_t seed, uint32_t step,
                                               uint32_t worker_base, float* norms_dev, uint8_t* packed_dev,
                                               int64_t packed_worker_stride_bytes, void* workspace_dev,
                                               int64_t* stats_dev, void* hip_stream)
{
    if (!plan || !grads_dev || !norm_lo_dev || !norm_hi_dev || !norms_dev || !packed_dev || !workspace_dev)
        return DQ_ERR_INVALID_ARG;
    if (M < 1 || M > DQ_MAX_WORKERS || b < 1 || b > 8) return DQ_ERR_INVALID_ARG;
    if (worker_stride_elems < plan->padded_elems || (worker_stride_elems & 3)) return DQ_ERR_INVALID_ARG;
    if (packed_worker_stride_bytes < dq_packed_bytes(plan, b) || (packed_worker_stride_bytes & 15))
        return DQ_ERR_INVALID_ARG;
    if (!dq_aligned16(grads_dev) || !dq_aligned16(packed_dev) || !dq_aligned16(workspace_dev)) return DQ_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(norm_lo_dev) & 3u) || (reinterpret_cast<uintptr_t>(norm_hi_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(norms_dev) & 3u) || (reinterpret_cast<uintptr_t>(stats_dev) & 7u))
        return DQ_ERR_INVALID_ARG;
    const int rc = dq_plan_check_device(plan);
    if (rc != DQ_OK) return rc;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (plan->n_cseg < plan->n_seg) { // tensors without elements: norm zero
        const int zrc = dq_zero_floats(norms_dev, static_cast<int64_t>(M) * plan->n_seg, stream);
        if (zrc != DQ_OK) return zrc;
    }
    if (plan->padded_elems == 0) return DQ_OK;
    unsigned long long* stats = reinterpret_cast<unsigned long long*>(stats_dev);
#define DQ_BRACKETED(B)                                                                                              \
    case B:                                                                                                          \
        return linf ? launch_bracketed<B, true>(plan, grads_dev, worker_stride_elems, M, norm_lo_dev, norm_hi_dev,  \
                                                seed, step, worker_base, norms_dev, packed_dev,                      \
                                                packed_worker_stride_bytes, workspace_dev, stats, stream)            \
                    : launch_bracketed<B, false>(plan, grads_dev, worker_stride_elems, M, norm_lo_dev, norm_hi_dev, \
                                                 seed, step, worker_base, norms_dev, packed_dev,                     \
                                                 packed_worker_stride_bytes, workspace_dev, stats, stream)
    switch (b) {
        DQ_BRACKETED(1);
        DQ_BRACKETED(2);
        DQ_BRACKETED(3);
        DQ_BRACKETED(4);
        DQ_BRACKETED(5);
        DQ_BRACKETED(6);
        DQ_BRACKETED(7);
    default:
        DQ_BRACKETED(8);
    }
#undef DQ_BRACKETED
}

extern "C" int dq_norm_quantize_pack_bracketed_v(const dq_plan_t* plan, const dq_widths_t* widths, const float* grads_dev,
                                                 int64_t worker_stride_elems, int M, int linf, const float* norm_lo_dev,
                                                 const float* norm_hi_dev, uint64_t seed, uint32_t step,
                                                 uint32_t worker_base, float* norms_dev, uint8_t* packed_dev,
                                                 int64_t packed_worker_stride_bytes, void* workspace_dev,
                                                 int64_t* stats_dev, void* hip_stream)
{
    if (!plan || !widths || !grads_dev || !norm_lo_dev || !norm_hi_dev || !norms_dev || !packed_dev || !workspace_dev)
        return DQ_ERR_INVALID_ARG;
    if (widths->plan != plan || widths->packed_bytes < 0) return DQ_ERR_INVALID_ARG;
    if (M < 1 || M > DQ_MAX_WORKERS) return DQ_ERR_INVALID_ARG;
    if (widths->n_workers != 1 && widths->n_workers != M) return DQ_ERR_INVALID_ARG;
    const int32_t row_stride = widths->n_workers == 1 ? 0 : plan->n_cseg;
    if (worker_stride_elems < plan->padded_elems || (worker_stride_elems & 3)) return DQ_ERR_INVALID_ARG;
    if (packed_worker_stride_bytes < widths->packed_bytes || (packed_worker_stride_bytes & 15))
        return DQ_ERR_INVALID_ARG;
    if (!dq_aligned16(grads_dev) || !dq_aligned16(packed_dev) || !dq_aligned16(workspace_dev)) return DQ_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(norm_lo_dev) & 3u) || (reinterpret_cast<uintptr_t>(norm_hi_dev) & 3u) ||
        (reinterpret_cast<uintptr_t>(norms_dev) & 3u) || (reinterpret_cast<uintptr_t>(stats_dev) & 7u))
        return DQ_ERR_INVALID_ARG;
    const int rc = dq_plan_check_device(plan);
    if (rc != DQ_OK) return rc;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (plan->n_cseg < plan->n_seg) {
        const int zrc = dq_zero_floats(norms_dev, static_cast<int64_t>(M) * plan->n_seg, stream);
        if (zrc != DQ_OK) return zrc;
    }
    if (plan->padded_elems == 0) return DQ_OK;
    unsigned long long* stats = reinterpret_cast<unsigned long long*>(stats_dev);
    return linf ? launch_bracketed<0, true>(plan, grads_dev, worker_stride_elems, M, norm_lo_dev, norm_hi_dev, seed, step,
                                            worker_base, norms_dev, packed_dev, packed_worker_stride_bytes, workspace_dev,
                                            stats, stream, widths->d_table, row_stride)
                : launch_bracketed<0, false>(plan, grads_dev, worker_stride_elems, M, norm_lo_dev, norm_hi_dev, seed, step,
                                             worker_base, norms_dev, packed_dev, packed_worker_stride_bytes, workspace_dev,
                                             stats, stream, widths->d_table, row_stride);
}
