// dq_quantize_pack: the EWU quantizer of Eq. (5)-(6) fused with the packing of the message whose
// size Eq. (7) counts.
//
// Work split.  One workgroup (256 lanes) owns a chunk of 4096 consecutive padded elements of one worker, each of its
// four wavefronts two tiles of 512; a lane's eight elements of a tile (two Philox blocks) give exactly one sign byte
// and B level bytes.  A tile is loaded by two instructions of 1 KiB each, which hand a lane two quads of elements
// from different places (dq_load_wave_tile).  The bytes are staged in LDS and leave the wavefront as 16-byte stores
// that cover each plane's bytes contiguously.
//
// A chunk inside one tensor (nearly every one of a gradient of large tensors): the plan's chunk table names the
// tensor, so one scalar load of 8 bytes, one of the norm and one binary32 division per wavefront give the scale;
// the lanes quantize the quads as loaded and the codes change places.  Other chunks: the granule table (4 bytes per
// 128 elements) names their tensors, whose scales s/N and ends are put in LDS once per workgroup, and the values
// change places.  Layouts with few chunks of the first kind have a form of their own (qp_load_block).
//
// HBM traffic per element: 4 bytes read, (B+1)/8 bytes written, plus the tables.
#include "dq_quantize_core.h"

namespace {

template <int B, int TILES, int NORM, bool WHOLE, bool KEEP>
__global__ __launch_bounds__(QP_THREADS) void k_quantize_pack(
    const float* __restrict__ grads, int64_t worker_stride, const float* __restrict__ norms, int32_t n_seg,
    const dq_chunk_tensor* __restrict__ chunk_tensor, const int32_t* __restrict__ granule_cseg,
    const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_valid_end,
    int64_t padded_elems,
    uint32_t key0, uint32_t key1, uint32_t step, uint32_t worker_base, uint8_t* __restrict__ packed,
    int64_t packed_stride, float* __restrict__ norms_out, dq_buckets buckets)
{
    quantize_pack_chunk<B, TILES, NORM, WHOLE, KEEP>(grads, worker_stride, norms, n_seg, chunk_tensor, granule_cseg, cseg_seg,
                                                     cseg_valid_end, padded_elems, key0, key1, step, worker_base, packed,
                                                     packed_stride, norms_out, blockIdx.x, threadIdx.x, {}, buckets);
}

template <int TILES, int NORM, bool WHOLE, bool KEEP> // as in k_quantize_pack
__global__ __launch_bounds__(QP_THREADS) void k_quantize_pack_v(
    const float* __restrict__ grads, int64_t worker_stride, const float* __restrict__ norms, int32_t n_seg,
    const dq_chunk_tensor* __restrict__ chunk_tensor, const int32_t* __restrict__ granule_cseg,
    const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_valid_end,
    const dq_cseg_width* __restrict__ widths_table,
    int32_t widths_worker_stride, int64_t padded_elems,
    uint32_t key0, uint32_t key1, uint32_t step, uint32_t worker_base, uint8_t* __restrict__ packed,
    int64_t packed_stride, float* __restrict__ norms_out)
{
    quantize_pack_chunk_v<TILES, NORM, WHOLE, KEEP>(grads, worker_stride, norms, n_seg, chunk_tensor, granule_cseg, cseg_seg,
                                                    cseg_valid_end, widths_table, widths_worker_stride, padded_elems, key0,
                                                    key1, step, worker_base, packed, packed_stride, norms_out, blockIdx.x);
}

// ---------------------------------------------------------------------------------------------
// Sign-only messages (the one-bit baseline of the paper's Table 2): the sign plane alone.  Same
// work split; no random numbers, no norms.
// HBM traffic per element: 4 bytes read, 1/8 byte written.
//
// What bounds it: the memory system's rate for a read stream with a thirtieth of writes in it (a kernel with these accesses and no
// arithmetic reaches 6.3 to 6.4 TB/s at 4 GiB, without its stores 7.1).  Wavefronts that are done sooner leave more requests in
// flight than that takes and lose some of it: a chunk of one tensor needs no table (two serial lookups behind the loads), and that alone made large
// calls 1 % slower, until fewer workgroups were resident.  WHOLE (layouts of large tensors): two tiles a wavefront and six workgroups per CU (by the size of the LDS request;
// eight fit) against four tiles, all chunks by the table and eight, us, with the reduce: ResNet-18 shape, M = 8 72.9 -> 72.0, M = 40 306 -> 302;
// transformer shape, M = 60 532 -> 524; 4 M values, M = 8 29.2 -> 27.3; 2^24, M = 64 725 -> 699.  Eight per CU: M = 40 306, 532, 28.1, 706; five
// 303, 534, 28.9, 718; four tiles and eight per CU 309, 536, 28.1, -.
// Otherwise (most chunks hold several tensors) the lookups are on every wavefront's way, and four tiles, all by the table, with eight per CU hide them:
// 16.8 M values in tensors of 128, 300, 1000, M = 4, pack alone 12.9, 16.6, 13.7 us against 14.6, 18.9, 14.8 in the first form (13.5, 17.7, 14.4 with eight per CU).
// The line is half of the chunks: tensors of 5000, 6000 and 8000 (18, 32 and 51 % of them) 0.97 to 1.05, 0.99 to 1.04 and 0.93 to 1.0 in the first form.
// ---------------------------------------------------------------------------------------------
template <bool WHOLE> constexpr int SP_TILES = WHOLE ? 2 : 4;
constexpr size_t SP_LDS_SIX_PER_CU = dq_lds_for(6) - SP_TILES<true> * QP_THREADS; // beside what the kernel declares

template <bool WHOLE, bool KEEP> // KEEP: as in k_quantize_pack (sign_keep_messages)
__global__ __launch_bounds__(QP_THREADS) void k_sign_pack(const float* __restrict__ grads, int64_t worker_stride,
                                                          const dq_chunk_tensor* __restrict__ chunk_tensor,
                                                          const int32_t* __restrict__ granule_cseg,
                                                          const int64_t* __restrict__ cseg_valid_end,
                                                          int64_t padded_elems, uint8_t* __restrict__ packed,
                                                          int64_t packed_stride)
{
    constexpr int TILES = SP_TILES<WHOLE>, CHUNK = QP_TILE * TILES;
    static_assert(!WHOLE || CHUNK == DQ_CHUNK, "a workgroup's elements are one entry of the chunk table");
    __shared__ __align__(16) uint8_t lds_sign[TILES * QP_THREADS];

    const uint32_t tid = threadIdx.x;
    const uint32_t w = blockIdx.y;
    const int64_t chunk0 = static_cast<int64_t>(blockIdx.x) * CHUNK;
    const uint32_t n_elems = static_cast<uint32_t>(padded_elems - chunk0 < CHUNK ? padded_elems - chunk0 : CHUNK);
    const float* g = grads + static_cast<int64_t>(w) * worker_stride + chunk0;
    const int32_t* gseg = granule_cseg + (chunk0 >> 7);

    float4 x[TILES][2];
    int64_t valid_end[TILES];
    // Global loads with clamped offsets here: as buffer loads (qp_load) the eight of a lane stream 1 to 1.5 % slower (2^26
    // values, M = 16 687 -> 693 us, ResNet-18 shape, M = 35 261 -> 264), and there is no arithmetic to gain on.
#pragma unroll
    for (int it = 0; it < TILES; ++it) {
        const uint32_t base = (tid >> 6) * (QP_WAVE_TILE * TILES) + it * QP_WAVE_TILE;
        uint32_t e0 = base + (tid & 31u) * 8u + ((tid >> 5) & 1u) * 4u, e1 = e0 + 256u;
        e0 = e0 < n_elems ? e0 : n_elems - 4u; // in bounds, and only lanes past the end receive it
        e1 = e1 < n_elems ? e1 : n_elems - 4u;
        const char* at = reinterpret_cast<const char*>(g); // 32-bit byte offsets from the uniform base
        x[it][0] = dq_load_stream(reinterpret_cast<const float4*>(at + e0 * 4u));
        x[it][1] = dq_load_stream(reinterpret_cast<const float4*>(at + e1 * 4u));
    }
    const uint32_t wave0 = (tid >> 6) * (QP_WAVE_TILE * TILES);
    bool whole = false;
    if constexpr (WHOLE) whole = dq_load_chunk_tensor(chunk_tensor, blockIdx.x).cseg >= 0;
    if (whole) { // 4096 elements of one tensor, the same for the whole workgroup: nothing to mask, and the codes change places
#pragma unroll
        for (int it = 0; it < TILES; ++it) {
            const auto w = __builtin_amdgcn_permlane32_swap(quantize_signs_below(0u, x[it][0]), quantize_signs_below(0u, x[it][1]), false, false);
            lds_sign[((wave0 + it * QP_WAVE_TILE) >> 3) + (tid & 63u)] = static_cast<uint8_t>(w[0] | (w[1] << 4));
        }
    } else {
#pragma unroll
        for (int it = 0; it < TILES; ++it) valid_end[it] = cseg_valid_end[gseg[qp_granule<TILES>(tid, it, n_elems)]];
#pragma unroll
        for (int it = 0; it < TILES; ++it) {
            dq_arrange_wave_tile(x[it][0], x[it][1]);
            const uint32_t e = qp_elem<TILES>(tid, it);
            if (e < n_elems) {
                uint32_t sign = quantize_sign_byte(x[it][0], x[it][1]);
                const int64_t n_valid = valid_end[it] - (chunk0 + e);
                if (n_valid < QP_PER_LANE) sign &= (1u << (n_valid > 0 ? static_cast<int>(n_valid) : 0)) - 1u;
                lds_sign[e >> 3] = static_cast<uint8_t>(sign);
            }
        }
    }
    uint8_t* dst = packed + static_cast<int64_t>(w) * packed_stride + (chunk0 >> 3);
    if (qp_on_lines(dst, dst)) { // as in qp_store_chunk
        dq_wave_sync();
        if (wave0 < n_elems) {
            const uint32_t n_wave = n_elems - wave0 < QP_WAVE_TILE * TILES ? n_elems - wave0 : QP_WAVE_TILE * TILES;
            qp_store_wave<KEEP>(dst + (wave0 >> 3), &lds_sign[wave0 >> 3], n_wave >> 3, tid & 63u);
        }
    } else {
        __syncthreads();
        qp_store_block<KEEP>(dst, lds_sign, n_elems >> 3, tid);
    }
}

// Whether the messages go through to the last-level cache (dq_store_buffer) and not past it with the streaming hint: they are
// read next, by the same GPU's reduce or by whatever sends them.  Whole iterations decide (norm, quantize, reduce on gradients
// not seen before), 390 of them drawn over 2^17 to 2^28 values, M = 1..64, one tensor and ragged ones, all widths; time against the
// hint: 0.92 to 1.0 up to 190 to 400 MB of messages whatever their number (2^24 values, M = 8 b = 2, 5, 8 0.955, 0.950, 0.971; 2^25, M = 2 b = 5
// 0.925; transformer shape, M = 24 with update b = 7 0.966), still 0.97 to 0.98 at 400 to 670 MB for b <= 4; beyond that most of them
// are gone from the 256 MB before they are read and the stores cost 1 to 5 % (2^28, M = 16 b = 4 6400 -> 6490 us).  Plain stores, which
// leave the lines dirty in the XCDs' caches, were 1 to 2 % slower than this at the sizes where they gain, and lose at others.
// With b = 5 to 7, whose level loads carry no hint without update, the line lies at 320 MB: iterations of one tensor or many large ones, M = 1 to 32, time against the
// hint without and with update at 195 to 260 MB 0.88 to 0.98 and 0.92 to 0.99, at 290 to 310 0.95 to 0.99 and 0.94 to 0.99, at 350 to 400 0.99 to 1.04 and 0.95 to
// 0.97 (transformer shape, M = 16 b = 7, 192 MB: 333 -> 307 and 331 -> 327 us; 34 M, M = 13 b = 6, 369 MB: 708 -> 726 and 727 -> 700).  Layouts of small tensors, whose
// workgroups store together, lose 0 to 3 % beyond 190 MB, and so more than 32 workers' messages at b >= 5 did when the lines were drawn.
// Narrow calls of 4 to 13 MB gain or lose up to 2 %.
inline bool qp_keep_messages(const dq_plan* plan, int M, int b)
{
    const int64_t megabytes = b <= 4 ? 640 : M > 32 ? 190 : b == 8 ? 400 : plan->many_whole ? 320 : 190;
    return M * dq_packed_bytes(plan, b) <= megabytes << 20;
}
// Widths that may be known to the GPU only: six bits stand for the usual.
inline bool qp_keep_messages_v(const dq_plan* plan, int M) { return M * dq_packed_bytes(plan, 6) <= 190 << 20; }

// The same for sign messages, which are small: whatever their number, from 12 M elements or 14 MB on.  Pack and majority, us, with the hint / through: 2^25
// values, M = 8 201 / 193, 2^26 401 / 385, M = 16 758 / 723, 2^28 - 333, M = 4 923 / 891; transformer and ResNet-18 shapes, M = 16 to 60 the same.
// Fewer bytes of smaller models gain 1 % (4 M values, M = 8) or lose up to 3 % (ResNet-18 shape, M = 2 26.9 / 27.7).
constexpr int64_t SP_KEEP_FROM_ELEMS = 12 << 20, SP_KEEP_FROM_BYTES = 14 << 20;
inline bool sign_keep_messages(const dq_plan* plan, int M)
{
    return plan->padded_elems >= SP_KEEP_FROM_ELEMS || M * (plan->padded_elems / 8) >= SP_KEEP_FROM_BYTES;
}

// Seven workgroups per CU in calls of many rounds (eight of the kernels of one width fit): norm, rule, quantize and reduce, ResNet-18 shape, M = 8
// 174.1 -> 172.7 us, 2^28 values, M = 16 6337 -> 6266; six 174.2 and 6259, and 3 M values, M = 5, whose rounds are few, 33.3 -> 33.5.
constexpr size_t QP_TABLE_LDS = 2 * sizeof(float) * DQ_CHUNK_GRANULES; // scales and ends, beside the staged bytes

template <int B, int NORM>
int launch(const dq_plan* plan, const float* grads, int64_t worker_stride, int M, const float* norms,
           uint64_t seed, uint32_t step, uint32_t worker_base, uint8_t* packed, int64_t packed_stride,
           float* norms_out, hipStream_t stream)
{
    const int64_t n_chunks = (plan->padded_elems + DQ_CHUNK - 1) / DQ_CHUNK;
    if (n_chunks > INT32_MAX) return DQ_ERR_INVALID_ARG;
    const dim3 grid(static_cast<unsigned>(n_chunks), M), block(QP_THREADS);
    const size_t lds = NORM == 0 && n_chunks * M >= DQ_MANY_WORKGROUPS ? dq_lds_for(7) - QP_TABLE_LDS - (1 + B) * QP_TILES * QP_THREADS : 0;
#define DQ_LAUNCH_Q(WHOLE, KEEP)                                                                                        \
    hipLaunchKernelGGL((k_quantize_pack<B, QP_TILES, NORM, WHOLE, KEEP>), grid, block, lds, stream, grads, worker_stride, \
                       norms, plan->n_seg, plan->d_chunk_tensor, plan->d_granule_cseg, plan->d_cseg_seg,                \
                       plan->d_cseg_valid_end, plan->padded_elems, static_cast<uint32_t>(seed),                         \
                       static_cast<uint32_t>(seed >> 32), step, worker_base, packed, packed_stride, norms_out, plan->buckets)
    if constexpr (NORM != 0) { // WHOLE: with the buckets' route
        if (plan->buckets.chunks > 0)
            DQ_LAUNCH_Q(true, false);
        else
            DQ_LAUNCH_Q(false, false);
    } else {
        const bool keep = qp_keep_messages(plan, M, B);
        if (plan->many_whole && keep)
            DQ_LAUNCH_Q(true, true);
        else if (plan->many_whole)
            DQ_LAUNCH_Q(true, false);
        else if (keep)
            DQ_LAUNCH_Q(false, true);
        else
            DQ_LAUNCH_Q(false, false);
    }
#undef DQ_LAUNCH_Q
    return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
}

template <int NORM>
int launch_width(int b, const dq_plan* plan, const float* grads, int64_t worker_stride, int M, const float* norms,
                 uint64_t seed, uint32_t step, uint32_t worker_base, uint8_t* packed, int64_t packed_stride,
                 float* norms_out, hipStream_t stream)
{
    switch (b) {
    case 1: return launch<1, NORM>(plan, grads, worker_stride, M, norms, seed, step, worker_base, packed, packed_stride, norms_out, stream);
    case 2: return launch<2, NORM>(plan, grads, worker_stride, M, norms, seed, step, worker_base, packed, packed_stride, norms_out, stream);
    case 3: return launch<3, NORM>(plan, grads, worker_stride, M, norms, seed, step, worker_base, packed, packed_stride, norms_out, stream);
    case 4: return launch<4, NORM>(plan, grads, worker_stride, M, norms, seed, step, worker_base, packed, packed_stride, norms_out, stream);
    case 5: return launch<5, NORM>(plan, grads, worker_stride, M, norms, seed, step, worker_base, packed, packed_stride, norms_out, stream);
    case 6: return launch<6, NORM>(plan, grads, worker_stride, M, norms, seed, step, worker_base, packed, packed_stride, norms_out, stream);
    case 7: return launch<7, NORM>(plan, grads, worker_stride, M, norms, seed, step, worker_base, packed, packed_stride, norms_out, stream);
    default: return launch<8, NORM>(plan, grads, worker_stride, M, norms, seed, step, worker_base, packed, packed_stride, norms_out, stream);
    }
}

} // namespace

extern "C" int dq_quantize_pack(const dq_plan_t* plan, const float* grads_dev, int64_t worker_stride_elems,
                                int M, const float* norms_dev, int b, uint64_t seed, uint32_t step,
                                uint32_t worker_base, uint8_t* packed_dev,
                                int64_t packed_worker_stride_bytes, void* hip_stream)
{
    if (!plan || !grads_dev || !norms_dev || !packed_dev) return DQ_ERR_INVALID_ARG;
    if (M < 1 || M > DQ_MAX_WORKERS || b < 1 || b > 8) return DQ_ERR_INVALID_ARG;
    if (worker_stride_elems < plan->padded_elems || (worker_stride_elems & 3)) return DQ_ERR_INVALID_ARG;
    if (packed_worker_stride_bytes < dq_packed_bytes(plan, b) || (packed_worker_stride_bytes & 15))
        return DQ_ERR_INVALID_ARG;
    if (!dq_aligned16(grads_dev) || !dq_aligned16(packed_dev) || (reinterpret_cast<uintptr_t>(norms_dev) & 3u))
        return DQ_ERR_INVALID_ARG;
    const int rc = dq_plan_check_device(plan);
    if (rc != DQ_OK) return rc;
    if (plan->padded_elems == 0) return DQ_OK;
    return launch_width<0>(b, plan, grads_dev, worker_stride_elems, M, norms_dev, seed, step, worker_base, packed_dev,
                           packed_worker_stride_bytes, nullptr, static_cast<hipStream_t>(hip_stream));
}

namespace {

int quantize_v_entry(int norm_mode, const dq_plan_t* plan, const dq_widths_t* widths, const float* grads_dev,
                     int64_t worker_stride_elems, int M, const float* norms_in, float* norms_out, uint64_t seed,
                     uint32_t step, uint32_t worker_base, uint8_t* packed_dev, int64_t packed_worker_stride_bytes,
                     void* hip_stream)
{
    const float* norms_any = norm_mode == 0 ? norms_in : norms_out;
    if (!plan || !widths || !grads_dev || !norms_any || !packed_dev) return DQ_ERR_INVALID_ARG;
    if (widths->plan != plan || widths->packed_bytes < 0) return DQ_ERR_INVALID_ARG;
    if (norm_mode != 0 && !plan->chunk_local) return DQ_ERR_INVALID_ARG;
    if (M < 1 || M > DQ_MAX_WORKERS) return DQ_ERR_INVALID_ARG;
    if (widths->n_workers != 1 && widths->n_workers != M) return DQ_ERR_INVALID_ARG;
    const int32_t row_stride = widths->n_workers == 1 ? 0 : plan->n_cseg;
    if (worker_stride_elems < plan->padded_elems || (worker_stride_elems & 3)) return DQ_ERR_INVALID_ARG;
    if (packed_worker_stride_bytes < widths->packed_bytes || (packed_worker_stride_bytes & 15))
        return DQ_ERR_INVALID_ARG;
    if (!dq_aligned16(grads_dev) || !dq_aligned16(packed_dev) || (reinterpret_cast<uintptr_t>(norms_any) & 3u))
        return DQ_ERR_INVALID_ARG;
    const int rc = dq_plan_check_device(plan);
    if (rc != DQ_OK) return rc;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (norm_mode != 0 && plan->n_cseg < plan->n_seg) { // tensors without elements: norm zero
        const int zrc = dq_zero_floats(norms_out, static_cast<int64_t>(M) * plan->n_seg, stream);
        if (zrc != DQ_OK) return zrc;
    }
    if (plan->padded_elems == 0) return DQ_OK;
    const int64_t n_chunks = (plan->padded_elems + DQ_CHUNK - 1) / DQ_CHUNK;
    if (n_chunks > INT32_MAX) return DQ_ERR_INVALID_ARG;
    const dim3 grid(static_cast<unsigned>(n_chunks), M), block(QP_THREADS);
    const bool keep = qp_keep_messages_v(plan, M);
#define DQ_LAUNCH_QV(NORM, WHOLE, KEEP)                                                                           \
    hipLaunchKernelGGL((k_quantize_pack_v<QP_TILES, NORM, WHOLE, KEEP>), grid, block, 0, stream, grads_dev,       \
                       worker_stride_elems, norms_in, plan->n_seg, plan->d_chunk_tensor, plan->d_granule_cseg,    \
                       plan->d_cseg_seg, plan->d_cseg_valid_end, widths->d_table, row_stride, plan->padded_elems, \
                       static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32), step, worker_base,         \
                       packed_dev, packed_worker_stride_bytes, norms_out)
    if (norm_mode == 1)
        DQ_LAUNCH_QV(1, true, false);
    else if (norm_mode == 2)
        DQ_LAUNCH_QV(2, true, false);
    else if (plan->many_whole && keep)
        DQ_LAUNCH_QV(0, true, true);
    else if (plan->many_whole)
        DQ_LAUNCH_QV(0, true, false);
    else if (keep)
        DQ_LAUNCH_QV(0, false, true);
    else
        DQ_LAUNCH_QV(0, false, false);
#undef DQ_LAUNCH_QV
    return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
}

} // namespace

extern "C" int dq_quantize_pack_v(const dq_plan_t* plan, const dq_widths_t* widths, const float* grads_dev,
                                  int64_t worker_stride_elems, int M, const float* norms_dev, uint64_t seed,
                                  uint32_t step, uint32_t worker_base, uint8_t* packed_dev,
                                  int64_t packed_worker_stride_bytes, void* hip_stream)
{
    return quantize_v_entry(0, plan, widths, grads_dev, worker_stride_elems, M, norms_dev, nullptr, seed, step,
                            worker_base, packed_dev, packed_worker_stride_bytes, hip_stream);
}

extern "C" int dq_norm_quantize_pack_v(const dq_plan_t* plan, const dq_widths_t* widths, const float* grads_dev,
                                       int64_t worker_stride_elems, int M, int linf, uint64_t seed, uint32_t step,
                                       uint32_t worker_base, float* norms_dev, uint8_t* packed_dev,
                                       int64_t packed_worker_stride_bytes, void* hip_stream)
{
    return quantize_v_entry(linf ? 2 : 1, plan, widths, grads_dev, worker_stride_elems, M, nullptr, norms_dev, seed,
                            step, worker_base, packed_dev, packed_worker_stride_bytes, hip_stream);
}

extern "C" int dq_sign_pack(const dq_plan_t* plan, const float* grads_dev, int64_t worker_stride_elems, int M,
                            uint8_t* packed_dev, int64_t packed_worker_stride_bytes, void* hip_stream)
{
    if (!plan || !grads_dev || !packed_dev) return DQ_ERR_INVALID_ARG;
    if (M < 1 || M > DQ_MAX_WORKERS) return DQ_ERR_INVALID_ARG;
    if (worker_stride_elems < plan->padded_elems || (worker_stride_elems & 3)) return DQ_ERR_INVALID_ARG;
    if (packed_worker_stride_bytes < plan->padded_elems / 8 || (packed_worker_stride_bytes & 15))
        return DQ_ERR_INVALID_ARG;
    if (!dq_aligned16(grads_dev) || !dq_aligned16(packed_dev)) return DQ_ERR_INVALID_ARG;
    const int rc = dq_plan_check_device(plan);
    if (rc != DQ_OK) return rc;
    if (plan->padded_elems == 0) return DQ_OK;
    auto go = [&](auto kernel, int64_t chunk, size_t lds) {
        const int64_t n_chunks = (plan->padded_elems + chunk - 1) / chunk;
        if (n_chunks > INT32_MAX) return false;
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(n_chunks), M), dim3(QP_THREADS), lds, static_cast<hipStream_t>(hip_stream), grads_dev,
                           worker_stride_elems, plan->d_chunk_tensor, plan->d_granule_cseg, plan->d_cseg_valid_end, plan->padded_elems, packed_dev,
                           packed_worker_stride_bytes);
        return true;
    };
    const bool keep = sign_keep_messages(plan, M);
    constexpr int64_t CHUNK = QP_TILE * SP_TILES<true>, LARGE = QP_TILE * SP_TILES<false>;
    const bool fits = plan->mostly_whole ? (keep ? go(k_sign_pack<true, true>, CHUNK, SP_LDS_SIX_PER_CU) : go(k_sign_pack<true, false>, CHUNK, SP_LDS_SIX_PER_CU))
                                         : (keep ? go(k_sign_pack<false, true>, LARGE, 0) : go(k_sign_pack<false, false>, LARGE, 0));
    if (!fits) return DQ_ERR_INVALID_ARG;
    return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
}

extern "C" int dq_norm_quantize_pack(const dq_plan_t* plan, const float* grads_dev, int64_t worker_stride_elems,
                                     int M, int linf, int b, uint64_t seed, uint32_t step, uint32_t worker_base,
                                     float* norms_dev, uint8_t* packed_dev, int64_t packed_worker_stride_bytes,
                                     void* hip_stream)
{
    if (!plan || !grads_dev || !norms_dev || !packed_dev) return DQ_ERR_INVALID_ARG;
    if (!plan->chunk_local) return DQ_ERR_INVALID_ARG;
    if (M < 1 || M > DQ_MAX_WORKERS || b < 1 || b > 8) return DQ_ERR_INVALID_ARG;
    if (worker_stride_elems < plan->padded_elems || (worker_stride_elems & 3)) return DQ_ERR_INVALID_ARG;
    if (packed_worker_stride_bytes < dq_packed_bytes(plan, b) || (packed_worker_stride_bytes & 15))
        return DQ_ERR_INVALID_ARG;
    if (!dq_aligned16(grads_dev) || !dq_aligned16(packed_dev) || (reinterpret_cast<uintptr_t>(norms_dev) & 3u))
        return DQ_ERR_INVALID_ARG;
    const int rc = dq_plan_check_device(plan);
    if (rc != DQ_OK) return rc;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    // tensors without elements belong to no chunk: their norm is zero
    if (plan->n_cseg < plan->n_seg) {
        const int zrc = dq_zero_floats(norms_dev, static_cast<int64_t>(M) * plan->n_seg, stream);
        if (zrc != DQ_OK) return zrc;
    }
    if (plan->padded_elems == 0) return DQ_OK;
    return linf ? launch_width<2>(b, plan, grads_dev, worker_stride_elems, M, nullptr, seed, step, worker_base,
                                  packed_dev, packed_worker_stride_bytes, norms_dev, stream)
                : launch_width<1>(b, plan, grads_dev, worker_stride_elems, M, nullptr, seed, step, worker_base,
                                  packed_dev, packed_worker_stride_bytes, norms_dev, stream);
}
