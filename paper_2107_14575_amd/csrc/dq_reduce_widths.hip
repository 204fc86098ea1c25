// The server's reduce for messages with a widths table (per tensor, and per tensor and worker) and for sign messages.
#include "dq_reduce_core.h"

namespace {

// Per-tensor widths: a wavefront inside one tensor takes its b and the place of its level dwords from the
// widths table (scalar) and runs the accumulation specialised for that b.  Elsewhere each lane does: its
// 32 elements lie in one 128-element granule, hence in one segment.
template <bool UPDATE, bool STREAM, bool ONCE, int W> // as in k_unpack_dequant_reduce
__global__ __launch_bounds__(UR_THREADS, ur_min_waves<W>(0)) void k_unpack_dequant_reduce_v(
    const uint8_t* __restrict__ packed, int64_t packed_stride, int M, const float* __restrict__ norms,
    int32_t n_seg, const int32_t* __restrict__ granule_cseg, const int32_t* __restrict__ cseg_seg,
    const int64_t* __restrict__ cseg_valid_end, const dq_cseg_width* __restrict__ widths, int64_t padded_elems,
    float inv_M, float* __restrict__ out, float* __restrict__ x, float eta)
{
    extern __shared__ __align__(16) uint8_t lds_raw[];
    float4* lds_out = reinterpret_cast<float4*>(lds_raw);

    const int tid = threadIdx.x, lane = tid & 63;
    const wave_span span = wave_span_of<W>(tid, padded_elems, granule_cseg);
    if (span.n_lanes <= 0) return;
    const int64_t P0 = span.start + lane * ur_per_lane<W>;
    const bool active = lane < span.n_lanes;
    const uint8_t* level_plane = packed + (padded_elems >> 3);

    float acc[ur_per_lane<W>];
#pragma unroll
    for (int k = 0; k < ur_per_lane<W>; ++k) acc[k] = 0.0f;
    int64_t n_valid = 0;
    int b = 0;

    if (span.first == span.last) {
        const dq_cseg_width e = widths[span.first];
        const int32_t seg = cseg_seg[span.first];
        n_valid = cseg_valid_end[span.first] - P0;
        b = __builtin_amdgcn_readfirstlane(e.b);
        const float unit = lane < M ? ur_unit(norms[static_cast<int64_t>(lane) * n_seg + seg], b) : 0.0f;
        const uint8_t* level_wave = level_plane + e.level_start + ((span.start - e.seg_start) >> 3) * b;
        dq_with_width(b, [&](auto width) {
            accumulate_wave<decltype(width)::value, W, ur_group_of<W>(decltype(width)::value), STREAM>(
                packed + (span.start >> 3), [&](int w) { return level_wave + static_cast<int64_t>(w) * packed_stride; },
                packed_stride, M, [] {}, [&](int w) { return lane_value(unit, w); }, span.n_lanes, acc, slots_of<W>(lds_out, tid));
        });
    } else {
        // the lane's own tensor, fetched beside the table (lanes past the end: the first one's)
        const int32_t c = granule_cseg[(active ? P0 : span.start) >> 7];
        n_valid = cseg_valid_end[c] - P0;
        const dq_cseg_width e = widths[c];
        float* lds_unit = reinterpret_cast<float*>(lds_raw + ur_tile<W> * sizeof(float)) + (tid >> 6) * ur_wave_segs<W> * M;
        const int n_local = span.last - span.first + 1;
        for (int i = lane; i < n_local * M; i += 64) {
            const int local = i / M, w = i - local * M;
            lds_unit[i] = ur_unit(norms[static_cast<int64_t>(w) * n_seg + cseg_seg[span.first + local]],
                                  widths[span.first + local].b);
        }
        dq_wave_sync();
        if (active) {
            b = e.b;
            const uint8_t* level_ptr = level_plane + e.level_start + ((P0 - e.seg_start) >> 3) * e.b; // dword aligned
            const float* unit_ptr = lds_unit + (c - span.first) * M;
            dq_with_width(b, [&](auto width) {
                accumulate_lane<decltype(width)::value, W>(packed + (P0 >> 3), level_ptr, packed_stride, M, unit_ptr, acc,
                                                        slots_of<W>(lds_out, tid));
            });
        }
    }
    finish_tile<W, UPDATE, ONCE>(acc, active, n_valid, inv_M * ur_sum_scale(b), lds_out, tid, span.start, padded_elems, out, x, eta);
}

// Per-worker widths: every worker's message has its own layout.  Workers' gradients of one tensor are alike,
// so most tensors have one width with all workers: a wavefront inside such a tensor runs the accumulation
// specialised for it, only the place of the level bytes differs from worker to worker.  Elsewhere a lane
// looks up b and the place of its level dwords once per worker and decodes that worker's dwords with the
// code specialised for its b.
struct worker_entry { // what a lane needs to decode one worker's tensor: 16 bytes, one LDS read
    float unit;         // N / s for that worker and tensor
    int32_t b;          // level bits
    int64_t level_base; // level-plane byte offset of padded index P is level_base + (P >> 3) * b
};

template <bool UPDATE, bool STREAM, bool ONCE> // as in k_unpack_dequant_reduce
__global__ __launch_bounds__(UR_THREADS, UR_MIN_WAVES) void k_unpack_dequant_reduce_w(
    const uint8_t* __restrict__ packed, int64_t packed_stride, int M, const float* __restrict__ norms,
    int32_t n_seg, int32_t n_cseg, const int32_t* __restrict__ granule_cseg, const int32_t* __restrict__ cseg_seg,
    const int64_t* __restrict__ cseg_valid_end, const dq_cseg_width* __restrict__ widths, int64_t padded_elems,
    float inv_M, float* __restrict__ out, float* __restrict__ x, float eta)
{
    extern __shared__ __align__(16) uint8_t lds_raw[];
    float4* lds_out = reinterpret_cast<float4*>(lds_raw);

    const int tid = threadIdx.x, lane = tid & 63;
    const wave_span span = wave_span_of<1>(tid, padded_elems, granule_cseg);
    if (span.n_lanes <= 0) return;
    const int64_t P0 = span.start + lane * ur_per_lane<1>;
    const bool active = lane < span.n_lanes;
    const uint8_t* level_plane = packed + (padded_elems >> 3);

    float acc[ur_per_lane<1>];
#pragma unroll
    for (int k = 0; k < ur_per_lane<1>; ++k) acc[k] = 0.0f;
    int64_t n_valid = 0;

    if (span.first == span.last) {
        const int32_t seg = cseg_seg[span.first];
        n_valid = cseg_valid_end[span.first] - P0;
        const int mine = lane < M ? lane : 0; // this lane's worker
        const dq_cseg_width e = widths[static_cast<int64_t>(mine) * n_cseg + span.first];
        const float N = norms[static_cast<int64_t>(mine) * n_seg + seg];
        const int b = __builtin_amdgcn_readfirstlane(e.b);
        if (__all(e.b == b)) {
            const int64_t at = e.level_start + ((span.start - e.seg_start) >> 3) * b;
            const uint32_t at_lo = static_cast<uint32_t>(at), at_hi = static_cast<uint32_t>(static_cast<uint64_t>(at) >> 32);
            const float unit = ur_unit(N, b);
            dq_with_width(b, [&](auto width) {
                accumulate_wave<decltype(width)::value, 1, ur_group_of<1>(decltype(width)::value), STREAM>(
                    packed + (span.start >> 3),
                    [&](int w) {
                        const uint64_t off = (static_cast<uint64_t>(__builtin_amdgcn_readlane(at_hi, w)) << 32) |
                                             static_cast<uint32_t>(__builtin_amdgcn_readlane(at_lo, w));
                        return level_plane + (static_cast<int64_t>(w) * packed_stride + static_cast<int64_t>(off));
                    },
                    packed_stride, M, [] {}, [&](int w) { return lane_value(unit, w); }, span.n_lanes, acc, slots_of<1>(lds_out, tid));
            });
            // This route ends here.  Joined with the general one ahead of finish_tile, the kernel spilled 18 registers,
            // and the general one paid: widths mixed, 4.2 M ragged elements, M = 64 152 us before there were two routes,
            // 206 joined, 137 now; one width in buckets of 512, M = 8, b = 2 33, 42, 31; this route, ResNet-18 shape, M = 8, b = 4
            // 24.0 joined, 21.2 now.
            finish_tile<1, UPDATE, ONCE>(acc, active, n_valid, inv_M * ur_sum_scale(b), lds_out, tid, span.start, padded_elems, out, x, eta);
            return;
        }
    }

    // the lane's own tensor, fetched beside the table (lanes past the end: the first one's)
    const int32_t c = granule_cseg[(active ? P0 : span.start) >> 7];
    n_valid = cseg_valid_end[c] - P0;
    worker_entry* lds_entry = reinterpret_cast<worker_entry*>(lds_raw + ur_tile<1> * sizeof(float)) +
                              (tid >> 6) * ur_wave_segs<1> * M; // [local seg][M]
    const int n_local = span.last - span.first + 1;
    for (int i = lane; i < n_local * M; i += 64) {
        const int local = i / M, w = i - local * M;
        const dq_cseg_width e = widths[static_cast<int64_t>(w) * n_cseg + span.first + local];
        worker_entry we;
        // every worker's sum is kept with the factor 2^-17 of widths 5 to 8: the narrower ones, whose
        // own factor is 2^-9, get the rest of it on their unit (exact: a usable norm is at least 2^-100)
        we.unit = ur_unit(norms[static_cast<int64_t>(w) * n_seg + cseg_seg[span.first + local]], e.b) *
                  (ur_fp8_width(e.b) ? UR_FP8_SCALE / UR_FP16_SCALE : 1.0f);
        we.b = e.b;
        we.level_base = e.level_start - (e.seg_start >> 3) * e.b; // seg_start is a multiple of 128
        lds_entry[i] = we;
    }
    dq_wave_sync();
    if (active) {
        const worker_entry* entry = lds_entry + (c - span.first) * M;
        const uint8_t* sign_ptr = packed + (P0 >> 3);
        // workers four at a time: sign dwords and up to eight level dwords each are fetched first
        // (loads past a worker's width are skipped), then decoded width by width
        constexpr int GROUP = 4;
        block_total<1> total{ slots_of<1>(lds_out, tid) }; // the block sums of accumulate_workers: same order of additions
        for (int w0 = 0; w0 < M; w0 += GROUP) {
            uint32_t sg[GROUP], wd[GROUP][8];
            worker_entry we[GROUP];
#pragma unroll
            for (int i = 0; i < GROUP; ++i) {
                we[i].b = 0;
                if (w0 + i < M) {
                    we[i] = entry[w0 + i];
                    const int64_t msg = static_cast<int64_t>(w0 + i) * packed_stride;
                    const uint32_t* lp =
                        reinterpret_cast<const uint32_t*>(level_plane + msg + we[i].level_base + (P0 >> 3) * we[i].b);
                    sg[i] = dq_load_stream(reinterpret_cast<const uint32_t*>(sign_ptr + msg));
#pragma unroll
                    for (int q = 0; q < 8; ++q) wd[i][q] = q < we[i].b ? lp[q] : 0u;
                }
            }
#pragma unroll
            for (int i = 0; i < GROUP; ++i) // b = 0: past the last worker
                dq_with_width(we[i].b, [&](auto width) {
                    accumulate_first_words<decltype(width)::value>(sg[i], wd[i], we[i].unit, acc);
                });
            if (((w0 + GROUP) & (UR_SUM_BLOCK - 1)) == 0 && w0 + GROUP < M) total.flush(acc);
        }
        total.finish(acc);
    }
    finish_tile<1, UPDATE, ONCE>(acc, active, n_valid, inv_M * UR_FP16_SCALE, lds_out, tid, span.start, padded_elems, out, x, eta);
}

// acc[k] += sgn_k * scale for a lane's elements: the scale with its sign flipped where the bit is set.
// (Conversion routes were measured here too and the integer form stays: (sign << 7) | 0x38 as an 8-bit
// float 0.40 ms against 0.35 ms at D = 2^28, M = 16; (sign << 15) | 0x3C00 as the 16-bit operand of a
// mixed-precision FMA, which issues at half rate, 33.8 against 30.8 us on 4.2 M elements at M = 64.)
template <int W>
__device__ __forceinline__ void add_signed_scale(uint32_t sg, float scale, float (&acc)[ur_per_lane<W>])
{
    const uint32_t unit = __float_as_uint(scale);
#pragma unroll
    for (int k = 0; k < ur_per_lane<W>; ++k) acc[k] += __uint_as_float(unit ^ ((sg << (31 - k)) & 0x80000000u));
}

// The workers in ascending order, eight loads in flight.
template <int W, typename Load, typename Scale>
__device__ __forceinline__ void accumulate_signs(int M, Load&& load, Scale&& scale, float (&acc)[ur_per_lane<W>])
{
    auto group = [&](auto g, int w) {
        constexpr int G = decltype(g)::value;
        uint32_t sg[G];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            sg[i] = load(w + i);
            __builtin_amdgcn_sched_barrier(0); // in the order of their use, as in accumulate_workers
        }
#pragma unroll
        for (int i = 0; i < G; ++i) add_signed_scale<W>(sg[i], scale(w + i), acc);
    };
    int w = 0;
    for (; w + 8 <= M; w += 8) group(std::integral_constant<int, 8>{}, w);
    if (w + 4 <= M) { group(std::integral_constant<int, 4>{}, w); w += 4; }
    if (w + 2 <= M) { group(std::integral_constant<int, 2>{}, w); w += 2; }
    if (w < M) group(std::integral_constant<int, 1>{}, w);
}

// Sign-only messages (the one-bit baseline of the paper's Table 2): the mean of scale * sgn,
// summed over workers ascending like the quantized average.
// HBM traffic per output element: M/8 bytes read, 4 bytes written.
template <int W>
__global__ __launch_bounds__(UR_THREADS) void k_sign_reduce_scaled(
    const uint8_t* __restrict__ packed, int64_t packed_stride, int M, const float* __restrict__ scales,
    int32_t n_seg, const int32_t* __restrict__ granule_cseg, const int32_t* __restrict__ cseg_seg,
    const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems, float inv_M, float* __restrict__ out)
{
    extern __shared__ __align__(16) uint8_t lds_raw[];
    float4* lds_out = reinterpret_cast<float4*>(lds_raw);

    const int tid = threadIdx.x, lane = tid & 63;
    const wave_span span = wave_span_of<W>(tid, padded_elems, granule_cseg);
    const int64_t P0 = span.start + lane * ur_per_lane<W>;
    const bool active = lane < span.n_lanes;

    // The scales first, then the messages, as at the narrow widths of the quantized average (ur_table_first).
    // Against the first loads ahead of the scales, in us: 2^24 values, M = 4, 8, 16 18.0, 21.1, 27.4 -> 16.8, 18.4,
    // 25.8; 2^28 x 16 340 -> 334; 2^24 values in tensors of 512, M = 8 21.8 -> 19.1; 2^24 x 64 68.5 -> 70.6.
    int64_t n_valid = 0;
    float* table = reinterpret_cast<float*>(lds_raw + ur_tile<W> * sizeof(float)) + (tid >> 6) * ur_wave_segs<W> * M;
    const float* scale_ptr = nullptr;
    if (span.n_lanes > 0)
        scale_ptr = wave_table(span, lane, M, P0, granule_cseg, cseg_valid_end, table, n_valid, [&](int w, int32_t c) {
            return scales[static_cast<int64_t>(w) * n_seg + cseg_seg[c]];
        });
    __syncthreads();
    if (span.n_lanes <= 0) return; // the whole wavefront; there is no workgroup barrier below

    float acc[ur_per_lane<W>];
#pragma unroll
    for (int k = 0; k < ur_per_lane<W>; ++k) acc[k] = 0.0f;
    const uint8_t* sign_wave = packed + (span.start >> 3);
    const uint32_t at = (active ? lane : span.n_lanes - 1) * (4u / W);
    accumulate_signs<W>(
        M,
        [&](int w) {
            return load_sign<W>(scalar_address(sign_wave + static_cast<int64_t>(w) * packed_stride) + at);
        },
        [&](int w) { return scale_ptr[w]; }, acc);
    finish_tile<W, false>(acc, active, n_valid, inv_M, lds_out, tid, span.start, padded_elems, out, nullptr, 0.0f);
}

// Sign-only messages without scales: per element only the number of workers whose bit is set
// matters.  A lane keeps that count for its 32 elements bit-sliced in PLANES dwords (bit k of
// plane j = bit j of element k's count, PLANES >= bit length of M) and adds each worker's sign
// dword with a ripple of half adders -- two bit operations per plane for 32 elements at once.
// MAJORITY: out = sgn(M - 2*count) in {-1, 0, +1}; otherwise out = (M - 2*count) / M.
template <int PLANES, bool MAJORITY>
__global__ __launch_bounds__(UR_THREADS) void k_sign_reduce_count(
    const uint8_t* __restrict__ packed, int64_t packed_stride, int M, const int32_t* __restrict__ granule_cseg,
    const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems, float inv_M, float* __restrict__ out)
{
    extern __shared__ __align__(16) uint8_t lds_raw[];
    float4* lds_out = reinterpret_cast<float4*>(lds_raw);

    const int tid = threadIdx.x;
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * ur_tile<1>;
    const int64_t tile_end = tile0 + ur_tile<1> < padded_elems ? tile0 + ur_tile<1> : padded_elems;
    const int64_t P0 = tile0 + tid * ur_per_lane<1>;
    const bool active = P0 < tile_end;

    float acc[ur_per_lane<1>];
#pragma unroll
    for (int k = 0; k < ur_per_lane<1>; ++k) acc[k] = 0.0f;
    int64_t n_valid = 0;
    if (active) {
        n_valid = cseg_valid_end[granule_cseg[P0 >> 7]] - P0;
        const uint8_t* sign_ptr = packed + (P0 >> 3);
        uint32_t plane[PLANES];
#pragma unroll
        for (int j = 0; j < PLANES; ++j) plane[j] = 0u;
        auto add = [&](uint32_t carry) {
#pragma unroll
            for (int j = 0; j < PLANES; ++j) {
                const uint32_t t = plane[j] & carry;
                plane[j] ^= carry;
                carry = t;
            }
        };
        constexpr int GROUP = 8;
        int w = 0;
        for (; w + GROUP <= M; w += GROUP) {
            uint32_t sg[GROUP];
#pragma unroll
            for (int i = 0; i < GROUP; ++i)
                sg[i] = dq_load_stream(reinterpret_cast<const uint32_t*>(sign_ptr + static_cast<int64_t>(w + i) * packed_stride));
#pragma unroll
            for (int i = 0; i < GROUP; ++i) add(sg[i]);
        }
        for (; w < M; ++w)
            add(dq_load_stream(reinterpret_cast<const uint32_t*>(sign_ptr + static_cast<int64_t>(w) * packed_stride)));
#pragma unroll
        for (int k = 0; k < ur_per_lane<1>; ++k) {
            uint32_t count = 0;
#pragma unroll
            for (int j = 0; j < PLANES; ++j) count |= __builtin_amdgcn_ubfe(plane[j], k, 1) << j;
            const int votes = M - 2 * static_cast<int>(count);
            if constexpr (MAJORITY)
                acc[k] = votes > 0 ? 1.0f : (votes < 0 ? -1.0f : 0.0f);
            else
                acc[k] = static_cast<float>(votes);
        }
    }
    finish_tile<1, false>(acc, active, n_valid, MAJORITY ? 1.0f : inv_M, lds_out, tid, tile0 + (tid >> 6) * ur_wave_elems<1>,
                       padded_elems, out, nullptr, 0.0f);
}

int reduce_entry_v(const dq_plan_t* plan, const dq_widths_t* widths, const uint8_t* packed_dev,
                   int64_t packed_worker_stride_bytes, int M, const float* norms_dev, float* out_dev, float* x_dev,
                   float eta, void* hip_stream)
{
    if (!plan || !widths || !packed_dev || !norms_dev || (!out_dev && !x_dev)) return DQ_ERR_INVALID_ARG;
    if (widths->plan != plan || widths->packed_bytes < 0) return DQ_ERR_INVALID_ARG;
    if (M < 1 || M > DQ_MAX_WORKERS) return DQ_ERR_INVALID_ARG;
    if (widths->n_workers != 1 && widths->n_workers != M) return DQ_ERR_INVALID_ARG;
    if (packed_worker_stride_bytes < widths->packed_bytes || (packed_worker_stride_bytes & 15))
        return DQ_ERR_INVALID_ARG;
    if (!dq_aligned16(packed_dev) || !dq_aligned16(out_dev) || !dq_aligned16(x_dev) ||
        (reinterpret_cast<uintptr_t>(norms_dev) & 3u))
        return DQ_ERR_INVALID_ARG;
    if (x_dev && !(eta == eta)) return DQ_ERR_INVALID_ARG;
    const int rc = dq_plan_check_device(plan);
    if (rc != DQ_OK) return rc;
    if (plan->padded_elems == 0) return DQ_OK;
    const int64_t n_tiles = (plan->padded_elems + ur_tile<1> - 1) / ur_tile<1>;
    if (n_tiles > INT32_MAX) return DQ_ERR_INVALID_ARG;
    // No fewer workgroups per CU here (as launch() has them for wide messages): the widths may be known to the GPU
    // only, and where it is b >= 5 that gains (1 to 4 % from 8192 tiles on), b = 2 loses (2 to 4 %) and so do small tensors
    // (16.8 M in buckets of 512, M = 16, b = 1 8 %).
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const float inv_M = 1.0f / static_cast<float>(M);
    const bool per_worker = widths->n_workers != 1;
    const ur_form form = ur_form_of(plan, 0, M, x_dev != nullptr, per_worker);
    // (with a row of widths per worker iterations lost by two workers to a word, ResNet-18 shape, M = 8 170.2 -> 174.0 us, transformer shape, M = 16
    // 375.4 -> 376.8, 1.3 M ragged values, M = 43 148.6 -> 151.3, although the reduce alone gained)
    const bool two = form.two;
    const dim3 grid(static_cast<unsigned>(two ? (plan->padded_elems + ur_tile<2> - 1) / ur_tile<2> : n_tiles)), block(UR_THREADS);
    const size_t tile_bytes = (two ? ur_tile<2> : ur_tile<1>) * sizeof(float);
    const size_t rows = static_cast<size_t>(two ? ur_max_local_seg<2> : ur_max_local_seg<1>) * M;
    if (per_worker) {
        const size_t lds_w = tile_bytes + rows * sizeof(worker_entry);
        int max_lds = 64 * 1024;
        if (lds_w > 64 * 1024) {
            if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, plan->device) != hipSuccess)
                return DQ_ERR_HIP;
            if (lds_w > static_cast<size_t>(max_lds)) return DQ_ERR_INVALID_ARG;
        }
        bool refused = false;
        auto go = [&](auto kernel) {
            // beyond 64 KiB of LDS per workgroup (M > 32) the kernel has to be told
            if (lds_w > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                         static_cast<int>(lds_w)) != hipSuccess) {
                refused = true;
                return;
            }
            hipLaunchKernelGGL(kernel, grid, block, lds_w, stream, packed_dev, packed_worker_stride_bytes, M, norms_dev, plan->n_seg,
                               plan->n_cseg, plan->d_granule_cseg, plan->d_cseg_seg, plan->d_cseg_valid_end, widths->d_table,
                               plan->padded_elems, inv_M, out_dev, x_dev, eta);
        };
        if (x_dev)
            ur_with_policy<true>(form.stream, form.once, [&](auto s, auto o) {
                go(k_unpack_dequant_reduce_w<true, decltype(s)::value, decltype(o)::value>);
            });
        else
            go(k_unpack_dequant_reduce_w<false, false, false>);
        if (refused) {
            (void)hipGetLastError();
            return DQ_ERR_HIP;
        }
        return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
    }
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, tile_bytes + rows * sizeof(float), stream, packed_dev, packed_worker_stride_bytes, M, norms_dev,
                           plan->n_seg, plan->d_granule_cseg, plan->d_cseg_seg, plan->d_cseg_valid_end, widths->d_table, plan->padded_elems, inv_M,
                           out_dev, x_dev, eta);
    };
    if (!x_dev) {
        if (two && form.stream)
            go(k_unpack_dequant_reduce_v<false, true, false, 2>);
        else if (two)
            go(k_unpack_dequant_reduce_v<false, false, false, 2>);
        else
            go(k_unpack_dequant_reduce_v<false, false, false, 1>);
    } else if (two) {
        if (form.once) // (a model of that size is most of what form.stream asks for: it is set)
            go(k_unpack_dequant_reduce_v<true, true, true, 2>);
        else if (form.stream)
            go(k_unpack_dequant_reduce_v<true, true, false, 2>);
        else
            go(k_unpack_dequant_reduce_v<true, false, false, 2>);
    } else if (form.stream) { // (and not form.once: such calls take W = 2)
        go(k_unpack_dequant_reduce_v<true, true, false, 1>);
    } else if (form.once) {
        go(k_unpack_dequant_reduce_v<true, false, true, 1>);
    } else {
        go(k_unpack_dequant_reduce_v<true, false, false, 1>);
    }
    return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
}

int sign_reduce_entry(bool majority, const dq_plan_t* plan, const uint8_t* packed_dev,
                      int64_t packed_worker_stride_bytes, int M, const float* scales_dev, float* out_dev,
                      void* hip_stream)
{
    if (!plan || !packed_dev || !out_dev) return DQ_ERR_INVALID_ARG;
    if (M < 1 || M > DQ_MAX_WORKERS) return DQ_ERR_INVALID_ARG;
    if (packed_worker_stride_bytes < plan->padded_elems / 8 || (packed_worker_stride_bytes & 15))
        return DQ_ERR_INVALID_ARG;
    if (!dq_aligned16(packed_dev) || !dq_aligned16(out_dev) || (reinterpret_cast<uintptr_t>(scales_dev) & 3u))
        return DQ_ERR_INVALID_ARG;
    const int rc = dq_plan_check_device(plan);
    if (rc != DQ_OK) return rc;
    if (plan->padded_elems == 0) return DQ_OK;
    const int64_t n_tiles = (plan->padded_elems + ur_tile<1> - 1) / ur_tile<1>;
    if (n_tiles > INT32_MAX) return DQ_ERR_INVALID_ARG;
    const dim3 grid(static_cast<unsigned>(n_tiles)), block(UR_THREADS);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const float inv_M = 1.0f / static_cast<float>(M);
    const size_t tile_bytes = ur_tile<1> * sizeof(float);
    if (!majority && scales_dev) {
        // Two halves of the elements' words a lane up to 200 tiles (3.0 to 17.7 us x 0.69 to 0.95); beyond them more wavefronts do not help and the
        // decoding, the same for half as many elements, costs (1366 tiles, M = 8 1.02, M = 64 1.24).
        auto go = [&](auto kernel, int tile) {
            hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((plan->padded_elems + tile - 1) / tile)), block,
                               tile * sizeof(float) + static_cast<size_t>(tile / DQ_GRANULE) * M * sizeof(float), stream, packed_dev,
                               packed_worker_stride_bytes, M, scales_dev, plan->n_seg, plan->d_granule_cseg, plan->d_cseg_seg,
                               plan->d_cseg_valid_end, plan->padded_elems, inv_M, out_dev);
        };
        if (n_tiles <= 200)
            go(k_sign_reduce_scaled<2>, ur_tile<2>);
        else
            go(k_sign_reduce_scaled<1>, ur_tile<1>);
        return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
    }
    // planes for the bit-sliced count: the bit length of M, rounded up to 3, 5 or 7 (M <= 64)
#define DQ_LAUNCH_COUNT(PLANES, MAJ)                                                                              \
    hipLaunchKernelGGL((k_sign_reduce_count<PLANES, MAJ>), grid, block, tile_bytes, stream, packed_dev,          \
                       packed_worker_stride_bytes, M, plan->d_granule_cseg, plan->d_cseg_valid_end,              \
                       plan->padded_elems, inv_M, out_dev)
    if (M < 8) {
        if (majority) DQ_LAUNCH_COUNT(3, true); else DQ_LAUNCH_COUNT(3, false);
    } else if (M < 32) {
        if (majority) DQ_LAUNCH_COUNT(5, true); else DQ_LAUNCH_COUNT(5, false);
    } else {
        if (majority) DQ_LAUNCH_COUNT(7, true); else DQ_LAUNCH_COUNT(7, false);
    }
#undef DQ_LAUNCH_COUNT
    return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
}

} // namespace

extern "C" int dq_sign_reduce(const dq_plan_t* plan, const uint8_t* packed_dev, int64_t packed_worker_stride_bytes,
                              int M, const float* scales_dev, float* out_dev, void* hip_stream)
{
    return sign_reduce_entry(false, plan, packed_dev, packed_worker_stride_bytes, M, scales_dev, out_dev, hip_stream);
}

extern "C" int dq_sign_majority(const dq_plan_t* plan, const uint8_t* packed_dev, int64_t packed_worker_stride_bytes,
                                int M, float* out_dev, void* hip_stream)
{
    return sign_reduce_entry(true, plan, packed_dev, packed_worker_stride_bytes, M, nullptr, out_dev, hip_stream);
}

extern "C" int dq_unpack_dequant_reduce_v(const dq_plan_t* plan, const dq_widths_t* widths,
                                          const uint8_t* packed_dev, int64_t packed_worker_stride_bytes, int M,
                                          const float* norms_dev, float* out_dev, void* hip_stream)
{
    if (!out_dev) return DQ_ERR_INVALID_ARG;
    return reduce_entry_v(plan, widths, packed_dev, packed_worker_stride_bytes, M, norms_dev, out_dev, nullptr,
                          0.0f, hip_stream);
}

extern "C" int dq_unpack_dequant_reduce_update_v(const dq_plan_t* plan, const dq_widths_t* widths,
                                                 const uint8_t* packed_dev, int64_t packed_worker_stride_bytes,
                                                 int M, const float* norms_dev, float eta, float* x_dev,
                                                 float* ghat_dev, void* hip_stream)
{
    if (!x_dev) return DQ_ERR_INVALID_ARG;
    return reduce_entry_v(plan, widths, packed_dev, packed_worker_stride_bytes, M, norms_dev, ghat_dev, x_dev, eta,
                          hip_stream);
}
