// dq_unpack_dequant_reduce: the server average of Algorithm 1 / Eq. (2),
//     out_P = (1/M) sum_i sgn_{i,P} * level_{i,P} * (N_{i,l} / s),
// with every worker's message read exactly once.
//
// Work split.  One workgroup (256 lanes) owns 8192 consecutive padded elements; a lane owns 32 of them, so that per worker it reads one sign dword
// and B level dwords -- every load is dword aligned for every B -- and keeps 32 binary32 accumulators (W = 1).  Or it owns 4096, a lane 16 of
// them, and the words that it decodes hold one worker's fields in one half and the next one's in the other (W = 2).  ur_two_workers says which calls take it.
//
// Arithmetic per (worker, element).  B <= 4: the level fields are spread one per byte word-wise
// (byte permutes and a shift/mask per four elements), the four sign bits of the word's elements go
// onto bit 7 of its bytes with one shift and one and-or, and each byte -- (sign << 7) | level --
// is converted as an 8-bit float, which is exactly +-level * 2^-9: half a conversion instruction
// and one FMA per element, no sign handling per element (about 2.6-3.4 vector instructions per
// worker and element against 4.5 with a conversion, a sign shift, a sign merge and an FMA each).
// B >= 5: the same with pairs of half-words that a mixed-precision FMA takes as 16-bit floats.
//
// What bounds it: reading the messages (5.7-6.1 TB/s at D = 2^28, M = 16); at M = 64 and B >= 5 the vector
// ALU beside it.  Measured with the half-word route, full-line loads and per-wavefront tables, before and
// after: 2^26 x 16 b = 5 199 -> 183 us, b = 6 214 -> 203, b = 8 255 -> 249; 4.2 M ragged elements with
// update, M = 64, b = 5 66.9 -> 52 us, b = 8 76.6 -> 66; ResNet-18 shape with update, M = 8, b = 6
// 35.4 -> 28.4 us.  Narrow widths are where they were before those changes or below: 2^28 x 16 b = 1 402 -> 380,
// b = 2 466 -> 447, b = 3 538 -> 532, b = 4 594 -> 588 and with update 875 -> 768; ResNet-18 shape, M = 8, b = 1, 2, 3
// 15.0, 15.4, 16.9 -> 14.6, 15.3, 16.7 (see ur_table_first).  With two workers to a word: 4.2 M ragged elements with update, M = 64,
// b = 5 55.5 -> 46.9 us (5.0 TB/s), ResNet-18 shape with update, M = 8, b = 6, messages in no cache 34.3 -> 29.5, 3 M, M = 20 with update b = 2, 5, 8 12.2,
// 17.4, 17.1 -> 11.1, 14.7, 16.1.
//
// The 32 or 16 results of a lane are consecutive in memory, so storing them directly would be 16-byte
// pieces 128 or 64 bytes apart; they go through LDS (XOR-swizzled 16-byte slots, conflict free both
// ways) and leave as fully coalesced 16-byte stores.
//
// Each wavefront works out the units N/s of its own tensors.
//
// HBM traffic per output element: M(B+1)/8 bytes read, 4 bytes written.
//
// With a model vector x the epilogue also applies the update of Algorithm 1, x <- x - eta * g_hat
// (8 more bytes per element, read and written with the same coalesced 16-byte accesses).
#include "dq_reduce_core.h"

namespace {

// STREAM: the streaming hint on level loads that would not have it; ONCE: on the model (ur_stream, ur_model_once)
template <int B, bool UPDATE, bool STREAM, bool ONCE, int W>
__global__ __launch_bounds__(UR_THREADS, ur_min_waves<W>(B)) void k_unpack_dequant_reduce(
    const uint8_t* __restrict__ packed, int64_t packed_stride, int M, const float* __restrict__ norms,
    int32_t n_seg, const int32_t* __restrict__ granule_cseg, const int32_t* __restrict__ cseg_seg,
    const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems, float inv_M, float* __restrict__ out,
    float* __restrict__ x, float eta)
{
    extern __shared__ __align__(16) uint8_t lds_raw[];
    float4* lds_out = reinterpret_cast<float4*>(lds_raw); // [ur_tile<W> / 4]

    const int tid = threadIdx.x, lane = tid & 63;
    const wave_span span = wave_span_of<W>(tid, padded_elems, granule_cseg);
    const int64_t P0 = span.start + lane * ur_per_lane<W>;
    const bool active = lane < span.n_lanes;
    const uint8_t* level_plane = packed + (padded_elems >> 3);

    int64_t n_valid = 0;
    float* table = reinterpret_cast<float*>(lds_raw + ur_tile<W> * sizeof(float)) + (tid >> 6) * ur_wave_segs<W> * M;
    const float* unit_ptr = nullptr;
    auto make_table = [&] { // the row of the lane's tensor
        unit_ptr = wave_table(span, lane, M, P0, granule_cseg, cseg_valid_end, table, n_valid, [&](int w, int32_t c) {
            return ur_unit(norms[static_cast<int64_t>(w) * n_seg + cseg_seg[c]], B);
        });
    };
    if constexpr (ur_table_first(B)) {
        // past the layout's end too (the row of tensor 0, not used): behind a condition the load of n_valid would
        // be waited for ahead of the barrier (ResNet-18 shape, M = 8, b = 2 15.1 -> 15.9 us)
        make_table();
        // ... except that b = 3, with its 12-byte loads, is better off waiting: 17.5 -> 16.6 us there
        if constexpr (B == 3) asm volatile("" ::"v"(static_cast<uint32_t>(n_valid)));
        __syncthreads();
    }
    if (span.n_lanes <= 0) return; // the whole wavefront; there is no workgroup barrier below

    float acc[ur_per_lane<W>];
#pragma unroll
    for (int k = 0; k < ur_per_lane<W>; ++k) acc[k] = 0.0f;
    const uint8_t* level_wave = level_plane + (span.start >> 3) * B;
    accumulate_wave<B, W, ur_group_one_width<W>(B), STREAM>(
        packed + (span.start >> 3), [&](int w) { return level_wave + static_cast<int64_t>(w) * packed_stride; },
        packed_stride, M,
        [&] {
            if constexpr (!ur_table_first(B)) make_table();
        },
        [&](int w) { return unit_ptr[w]; }, span.n_lanes, acc, slots_of<W>(lds_out, tid));
    finish_tile<W, UPDATE, ONCE>(acc, active, n_valid, inv_M * ur_sum_scale(B), lds_out, tid, span.start, padded_elems, out, x, eta);
}

// Few tiles and many workers: the workgroup's four wavefronts share the 2048 elements of a span, each with `per_wave`
// consecutive blocks of UR_SUM_BLOCK workers (one or two).  The block sums are then added in block order, wavefront after
// wavefront through LDS -- the additions of k_unpack_dequant_reduce in the same order, bit for bit -- and the wavefronts
// write a quarter of the span each.
// What bounds the undivided kernel there is the vector ALU of a few SIMDs: 258 tiles are 1032 wavefronts on 1024 SIMDs, and
// one with two of them takes twice as long as the others with one.
constexpr int UR_SPLIT = UR_THREADS / 64;
template <int B, bool UPDATE>
__global__ __launch_bounds__(UR_THREADS, UR_MIN_WAVES) void k_unpack_dequant_reduce_split(
    const uint8_t* __restrict__ packed, int64_t packed_stride, int M, int per_wave, const float* __restrict__ norms,
    int32_t n_seg, const int32_t* __restrict__ granule_cseg, const int32_t* __restrict__ cseg_seg,
    const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems, float inv_M, float* __restrict__ out,
    float* __restrict__ x, float eta)
{
    constexpr int PIECES = 8 / UR_SPLIT; // of the span's eight pieces of 256 elements
    extern __shared__ __align__(16) uint8_t lds_raw[];
    float4* lds_out = reinterpret_cast<float4*>(lds_raw);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const wave_span span = wave_span_from<1>(static_cast<int64_t>(ur_tile_index<1>()) * ur_wave_elems<1>, padded_elems, granule_cseg);
    const int64_t P0 = span.start + lane * ur_per_lane<1>;
    const int w0 = wave * per_wave * UR_SUM_BLOCK;
    const int n_mine = M - w0 < per_wave * UR_SUM_BLOCK ? M - w0 : per_wave * UR_SUM_BLOCK; // <= 0: none
    const int last = (M - 1) / (per_wave * UR_SUM_BLOCK); // the last wavefront with workers

    const auto piece_at = [&](int j) { return span.start + 256 * (wave * PIECES + j) + 4 * lane; };
    float4 xv[PIECES]; // the model's pieces, in flight from the start
    ur_model<false> model;
    if constexpr (UPDATE) {
        model = ur_model<false>(x, span.start, ur_wave_elems<1>, padded_elems);
#pragma unroll
        for (int j = 0; j < PIECES; ++j) xv[j] = model.load(256 * (wave * PIECES + j) + 4 * lane);
    }

    float acc[ur_per_lane<1>];
#pragma unroll
    for (int k = 0; k < ur_per_lane<1>; ++k) acc[k] = 0.0f;
    const lane_slots<1> slots = slots_of<1>(lds_out, tid);
    int64_t n_valid = 0;
    if (n_mine > 0) { // a wavefront without workers still reaches the barriers and writes its quarter
        const uint8_t* mine = packed + static_cast<int64_t>(w0) * packed_stride;
        const uint8_t* level_wave = mine + (padded_elems >> 3) + (span.start >> 3) * B;
        float* table = reinterpret_cast<float*>(lds_raw + ur_tile<1> * sizeof(float)) + wave * ur_wave_segs<1> * per_wave * UR_SUM_BLOCK;
        const float* unit_ptr = wave_table(span, lane, n_mine, P0, granule_cseg, cseg_valid_end, table, n_valid, [&](int w, int32_t c) {
            return ur_unit(norms[static_cast<int64_t>(w0 + w) * n_seg + cseg_seg[c]], B);
        });
        accumulate_wave<B, 1, (B <= 4 ? 8 : 4), false, false>(
            mine + (span.start >> 3), [&](int w) { return level_wave + static_cast<int64_t>(w) * packed_stride; }, packed_stride,
            n_mine, [] {}, [&](int w) { return unit_ptr[w]; }, span.n_lanes, acc, slots);
    }
    for (int r = 0; r <= last; ++r) {
        if (wave == r) {
            const lane_slots<1> before{ lds_out + (wave - 1) * 512, lane };
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                float4 t = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
                if (n_mine > UR_SUM_BLOCK || r > 0) {
                    float4 o = n_mine > UR_SUM_BLOCK ? slots[q] : t;
                    if (r > 0) {
                        const float4 p = before[q];
                        o = make_float4(p.x + o.x, p.y + o.y, p.z + o.z, p.w + o.w);
                    }
                    if (n_mine > UR_SUM_BLOCK) o = make_float4(o.x + t.x, o.y + t.y, o.z + t.z, o.w + t.w);
                    t = o;
                }
                if (r == last) { // as in finish_tile
                    const int nv = n_valid >= ur_per_lane<1> ? ur_per_lane<1> : (n_valid > 0 ? static_cast<int>(n_valid) : 0);
                    const float scale = inv_M * ur_sum_scale(B);
                    t.x = 4 * q < nv ? t.x * scale : 0.0f;
                    t.y = 4 * q + 1 < nv ? t.y * scale : 0.0f;
                    t.z = 4 * q + 2 < nv ? t.z * scale : 0.0f;
                    t.w = 4 * q + 3 < nv ? t.w * scale : 0.0f;
                }
                slots[q] = t;
            }
        }
        __syncthreads();
    }
    const float4* sum = lds_out + last * 512;
#pragma unroll
    for (int j = 0; j < PIECES; ++j) {
        const int64_t P = piece_at(j);
        if (P >= padded_elems) continue;
        const int src = 8 * (wave * PIECES + j) + (lane >> 3), q = lane & 7;
        const float4 v = sum[src * 8 + (q ^ (src & 7))];
        if (!UPDATE || out) dq_store_stream(reinterpret_cast<float4*>(out + P), v);
        if constexpr (UPDATE) model.store(256 * (wave * PIECES + j) + 4 * lane, ur_step(xv[j], v, eta));
    }
}

// Few tiles and few workers: a lane owns 8 elements in place of 32, so that there are four times as many wavefronts, and
// the loads of messages, model and norms are issued together behind one lookup (the chunk table's) where the elements
// lie in one tensor.  The same products and the same additions in the same order as in k_unpack_dequant_reduce, bit for bit.
// What bounds it: launch and two memory latencies.
constexpr int UR_NARROW_PER_LANE = 8, UR_NARROW_WAVE = 64 * UR_NARROW_PER_LANE; // 512 elements, up to four tensors
constexpr int UR_NARROW_SEGS = UR_NARROW_WAVE / DQ_GRANULE;

template <int B, bool UPDATE>
__global__ __launch_bounds__(UR_THREADS) void k_unpack_dequant_reduce_narrow(
    const uint8_t* __restrict__ packed, int64_t packed_stride, int M, const float* __restrict__ norms, int32_t n_seg,
    const dq_chunk_tensor* __restrict__ chunk_tensor, const int32_t* __restrict__ granule_cseg,
    const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems, float inv_M,
    float* __restrict__ out, float* __restrict__ x, float eta)
{
    extern __shared__ __align__(16) uint8_t lds_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    wave_span span;
    span.start = (static_cast<int64_t>(blockIdx.x) * (UR_THREADS / 64) + wave) * UR_NARROW_WAVE;
    if (span.start >= padded_elems) return; // the whole wavefront; there is no workgroup barrier below
    const int64_t left = padded_elems - span.start;
    span.n_lanes = static_cast<int>(left < UR_NARROW_WAVE ? left : UR_NARROW_WAVE) / UR_NARROW_PER_LANE; // a multiple of 16
    const dq_chunk_tensor owner = dq_load_chunk_tensor(chunk_tensor, span.start >> 12);
    const int64_t P0 = span.start + lane * UR_NARROW_PER_LANE;
    const uint32_t own = lane < span.n_lanes ? lane : span.n_lanes - 1; // lanes past the end fetch the last one's bytes
    float4 xv[2];
    ur_model<false> model;
    if constexpr (UPDATE) {
        model = ur_model<false>(x, span.start, UR_NARROW_WAVE, padded_elems);
        xv[0] = model.load(own * UR_NARROW_PER_LANE);
        xv[1] = model.load(own * UR_NARROW_PER_LANE + 4);
    }

    const uint8_t* sign_wave = packed + (span.start >> 3);
    const uint8_t* level_wave = packed + (padded_elems >> 3) + (span.start >> 3) * B;
    float* table = reinterpret_cast<float*>(lds_raw) + wave * UR_NARROW_SEGS * M;
    const float* unit_ptr = nullptr;
    int64_t n_valid = UR_NARROW_PER_LANE;
    float acc[UR_NARROW_PER_LANE], total[UR_NARROW_PER_LANE];
#pragma unroll
    for (int k = 0; k < UR_NARROW_PER_LANE; ++k) acc[k] = total[k] = 0.0f;
    auto group = [&](auto g, int w) {
        constexpr int G = decltype(g)::value;
        uint32_t sg[G];
        uint64_t lv[G];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int64_t off = static_cast<int64_t>(w + i) * packed_stride;
            const uint8_t* lp = level_wave + off + own * B;
            sg[i] = sign_wave[off + own];
            lv[i] = 0;
            __builtin_memcpy(&lv[i], lp, B); // B bytes, at any byte address
        }
        if (w == 0) {
            if (owner.cseg >= 0) { // the same for the whole wavefront: one tensor, all of it data
                if (lane < M) table[lane] = ur_level_unit(norms[static_cast<int64_t>(lane) * n_seg + owner.seg], B);
                dq_wave_sync();
                unit_ptr = table;
            } else {
                span.first = granule_cseg[span.start >> 7];
                span.last = granule_cseg[(span.start + span.n_lanes * UR_NARROW_PER_LANE - 1) >> 7];
                unit_ptr = wave_table(span, lane, M, P0, granule_cseg, cseg_valid_end, table, n_valid, [&](int u, int32_t c) {
                    return ur_level_unit(norms[static_cast<int64_t>(u) * n_seg + cseg_seg[c]], B);
                });
            }
        }
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const float unit = unit_ptr[w + i];
#pragma unroll
            for (int k = 0; k < UR_NARROW_PER_LANE; ++k) {
                const uint32_t level = static_cast<uint32_t>(lv[i] >> (k * B)) & ((1u << B) - 1u);
                const float v = __uint_as_float(__float_as_uint(static_cast<float>(level)) | ((sg[i] << (31 - k)) & 0x80000000u));
                acc[k] = __builtin_fmaf(v, unit, acc[k]);
            }
            if (((w + i + 1) & (UR_SUM_BLOCK - 1)) == 0 && w + i + 1 < M) { // the block joins the total, as block_total does
#pragma unroll
                for (int k = 0; k < UR_NARROW_PER_LANE; ++k) {
                    total[k] = w + i + 1 > UR_SUM_BLOCK ? total[k] + acc[k] : acc[k];
                    acc[k] = 0.0f;
                }
            }
        }
    };
    int w = 0;
    for (; w + 8 <= M; w += 8) group(std::integral_constant<int, 8>{}, w);
    if (w + 4 <= M) { group(std::integral_constant<int, 4>{}, w); w += 4; }
    if (w + 2 <= M) { group(std::integral_constant<int, 2>{}, w); w += 2; }
    if (w < M) group(std::integral_constant<int, 1>{}, w);
    if (lane >= span.n_lanes) return;
    const int nv = n_valid >= UR_NARROW_PER_LANE ? UR_NARROW_PER_LANE : (n_valid > 0 ? static_cast<int>(n_valid) : 0);
#pragma unroll
    for (int k = 0; k < UR_NARROW_PER_LANE; ++k) {
        const float sum = M > UR_SUM_BLOCK ? total[k] + acc[k] : acc[k];
        acc[k] = k < nv ? sum * (inv_M * ur_sum_scale(B)) : 0.0f;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float4 v = make_float4(acc[4 * h], acc[4 * h + 1], acc[4 * h + 2], acc[4 * h + 3]);
        if (!UPDATE || out) *reinterpret_cast<float4*>(out + P0 + 4 * h) = v;
        if constexpr (UPDATE) model.store(lane * UR_NARROW_PER_LANE + 4 * h, ur_step(xv[h], v, eta));
    }
}

constexpr size_t UR_LDS_THREE_PER_CU = 41 * 1024; // of 160 KiB

// Up to how many tiles the workers are divided over wavefronts (k_unpack_dequant_reduce_split), measured with update against
// the undivided kernel for M = 28..64, 64..600 tiles, all widths, messages in no cache and read before (time undivided / time
// divided).  Undivided, a tile is one wavefront on each SIMD of a CU: 128 tiles leave half of the chip idle (M = 32 b = 1 +7 % and
// +17, b = 5 +34 and +41; M = 64 +28 and +33, +52 and +60), and beyond 256 some CUs have two tiles and the others wait for them
// (M = 64 at 256 and 258 tiles b = 5 33.0 and 41.0 us against 29.2 and 35.5).  What the division costs (LDS, barriers, a row of units per
// wavefront) is most at b = 1, 4 and 8.  Inside the lines it gains up to 100 %.  Beyond them fresh messages lose, at some sizes all do:
// M = 28 at 192 tiles b = 1 3 %, M = 32 at 256 b = 7 5 %, M = 48 at 258 b = 4 2 and b = 8 12 %; M = 60 at 361 and 400 b = 2, 3, 5 3 to 4 %
// gained and 3 to 6 lost, M = 57 at 320 and 400 b = 6, 7 2 to 3 gained and 10 lost; at 514 and 600 b = 5 3 and 7 % lost (read before 9 and 2
// gained), b = 4 16 and 18.
// Against two workers to a word (W = 2), which came later, messages in no cache / read before (time with W = 2 / divided): M = 64 at 64 tiles 1.1 to 1.5 / 1.1 to 1.7, at 150
// b >= 2 1.02 to 1.24 / 1.05 to 1.28, at 200 b = 5 1.06 / 1.09, b = 4 0.91 / 0.93, at 258 b = 2, 3, 5 1.0 to 1.03 / 1.0 to 1.13, b = 6 and 7 0.89 / 0.97; M = 48 b = 5 to 7 at 200
// 1.03 / 1.08, at 258 0.82 / 0.84, b <= 4 at 96 - / 0.93; M = 32 b >= 5 at 160 1.05 to 1.14, at 200 0.88, b <= 4 at 128 0.91.
inline int64_t ur_split_max_tiles(int b, int M)
{
    if (M > 56) return b == 1 ? 128 : b == 4 || b == 8 ? 170 : b == 5 ? 300 : b <= 3 ? 260 : 230;
    if (M >= 40) return b >= 5 && b <= 7 ? 220 : b == 8 ? 170 : 80;
    if (M > 24) return b >= 5 ? 170 : 64;
    return 0;
}
// Up to how many tiles a lane owns 8 elements (k_unpack_dequant_reduce_narrow), measured against the kernels above for
// M = 1..64, 0.5..768 tiles, all widths, with and without update (kernel trace).  4096 elements, M = 8, b = 8 with update
// 4.44 -> 3.32 us; 2^20, M = 4, b = 4 4.84 -> 4.24.  Inside the lines 0 to 60 % gained; beyond them its plain extraction
// of every level costs more than the idle lanes: M = 1 at 192 tiles 0 %, at 256 up to 9 % lost, M = 8 at 192 b = 1 7 %, 3.0 M ragged
// values, M = 5 b = 1 7 %; M = 32 b = 7 at 64 tiles 5 %, M = 64 b = 1 at any size 10 %.
// Against W = 2, messages in no cache / read before (time with W = 2 / a lane's 8): 64 tiles without update 0.94 to 1.25 / 1.0 to 1.6, with update b <= 4 0.93 to
// 1.04 / 0.95 to 1.15; 128 tiles without update M = 1 to 4 0.91 to 1.09 / 0.98 to 1.06, M = 8 to 24 b <= 4 0.78 to 0.9 / 0.86 to 0.97, b >= 5 0.85 to 1.09 / 0.99 to
// 1.25, with update b <= 4 0.72 to 0.9 / 0.79 to 0.89, b >= 5 0.8 to 0.95 / 0.81 to 0.9 up to twelve workers and 0.86 to 1.0 / 0.94 to 1.19 with more; b = 8 at
// 150 0.84 to 1.05 / 0.86 to 1.21.
inline int64_t ur_narrow_max_tiles(int b, int M, bool update)
{
    if (b == 8 && M >= 4) return 192;
    if (M > 24) return M <= 40 && b != 3 && b != 7 ? 64 : 0;
    if (update) return b >= 5 && M > 12 ? 128 : 80;
    return b >= 5 || M <= 4 ? 128 : 96;
}

template <int B>
int launch(const dq_plan* plan, const uint8_t* packed, int64_t packed_stride, int M, const float* norms,
           float* out, float* x, float eta, hipStream_t stream)
{
    const int64_t n_tiles = (plan->padded_elems + ur_tile<1> - 1) / ur_tile<1>;
    if (n_tiles > INT32_MAX) return DQ_ERR_INVALID_ARG;
    const float inv_M = 1.0f / static_cast<float>(M);
    if (n_tiles <= ur_narrow_max_tiles(B, M, x != nullptr)) {
        const dim3 grid(static_cast<unsigned>((plan->padded_elems + 4 * UR_NARROW_WAVE - 1) / (4 * UR_NARROW_WAVE))), block(UR_THREADS);
        const size_t lds = static_cast<size_t>(UR_THREADS / 64) * UR_NARROW_SEGS * M * sizeof(float);
#define DQ_LAUNCH_NARROW(UPDATE)                                                                                          \
    hipLaunchKernelGGL((k_unpack_dequant_reduce_narrow<B, UPDATE>), grid, block, lds, stream, packed, packed_stride, M, norms, \
                       plan->n_seg, plan->d_chunk_tensor, plan->d_granule_cseg, plan->d_cseg_seg, plan->d_cseg_valid_end, \
                       plan->padded_elems, inv_M, out, x, eta)
        if (x) DQ_LAUNCH_NARROW(true);
        else DQ_LAUNCH_NARROW(false);
#undef DQ_LAUNCH_NARROW
        return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
    }
    if (n_tiles <= ur_split_max_tiles(B, M)) {
        const int per_wave = (M + UR_SPLIT * UR_SUM_BLOCK - 1) / (UR_SPLIT * UR_SUM_BLOCK); // blocks of workers
        const dim3 grid(static_cast<unsigned>((plan->padded_elems + ur_wave_elems<1> - 1) / ur_wave_elems<1>)), block(UR_THREADS);
        const size_t lds = ur_tile<1> * sizeof(float) + static_cast<size_t>(ur_max_local_seg<1>) * per_wave * UR_SUM_BLOCK * sizeof(float);
#define DQ_LAUNCH_SPLIT(UPDATE)                                                                                           \
    hipLaunchKernelGGL((k_unpack_dequant_reduce_split<B, UPDATE>), grid, block, lds, stream, packed, packed_stride, M,    \
                       per_wave, norms, plan->n_seg, plan->d_granule_cseg, plan->d_cseg_seg, plan->d_cseg_valid_end,       \
                       plan->padded_elems, inv_M, out, x, eta)
        if (x) DQ_LAUNCH_SPLIT(true);
        else DQ_LAUNCH_SPLIT(false);
#undef DQ_LAUNCH_SPLIT
        return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
    }
    const ur_form form = ur_form_of(plan, B, M, x != nullptr);
    if (form.two) {
        const dim3 grid(static_cast<unsigned>((plan->padded_elems + ur_tile<2> - 1) / ur_tile<2>)), block(UR_THREADS);
        const size_t lds = ur_tile<2> * sizeof(float) + static_cast<size_t>(ur_max_local_seg<2>) * M * sizeof(float);
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, block, lds, stream, packed, packed_stride, M, norms, plan->n_seg, plan->d_granule_cseg,
                               plan->d_cseg_seg, plan->d_cseg_valid_end, plan->padded_elems, inv_M, out, x, eta);
        };
        if (!x && form.stream)
            go(k_unpack_dequant_reduce<B, false, ur_may_stream(B), false, 2>);
        else if (!x)
            go(k_unpack_dequant_reduce<B, false, false, false, 2>);
        else if (form.once) // (a model of that size is most of what form.stream asks for: it is set at the widths that look)
            go(k_unpack_dequant_reduce<B, true, ur_may_stream(B), true, 2>);
        else if (form.stream)
            go(k_unpack_dequant_reduce<B, true, ur_may_stream(B), false, 2>);
        else
            go(k_unpack_dequant_reduce<B, true, false, false, 2>);
        return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
    }
    size_t lds_bytes = ur_tile<1> * sizeof(float) + static_cast<size_t>(ur_max_local_seg<1>) * M * sizeof(float);
    // Where thousands of tiles stream wide messages, three workgroups per CU move more than four (W = 1; six to thirteen or sixteen workers without update take W = 2).  Measured for
    // M = 1..32, 2048..16384 tiles, b = 4..8, inputs in no cache and inputs read before, as a factor on the time:
    // M = 16 b = 4..8 0.98, 0.98, 0.97, 0.98, 0.99 at 4096 tiles and 0.95, 0.94, 0.95, 0.97, 0.99 at 16384; M = 8 0.98..1.0 at
    // 4096, 0.97..0.99 at 8192; M = 32 0.96..0.99 at 8192.  Below 4096 tiles or eight workers four are as good or better (M = 16
    // at 3072 tiles 0.98..1.02, at 2048 1.0..1.03; M = 4 b = 5 1.03..1.1, M = 1 1.01..1.16).  With update b = 5 to 7 lose 1 to
    // 4 % at any size, and 4 and 8 gain from 8192 tiles on (1.0, 16384 tiles 0.97..0.99).  b = 2 and 3 lose (471 -> 492 us, 549 ->
    // 563 at 2^28 x 16).
    const bool three = B >= 4 && M >= 8 && (x ? !ur_may_stream(B) && n_tiles >= 8192 : n_tiles >= 4096);
    if (three && lds_bytes < UR_LDS_THREE_PER_CU) lds_bytes = UR_LDS_THREE_PER_CU;
    const dim3 grid(static_cast<unsigned>(n_tiles)), block(UR_THREADS);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, lds_bytes, stream, packed, packed_stride, M, norms, plan->n_seg, plan->d_granule_cseg,
                           plan->d_cseg_seg, plan->d_cseg_valid_end, plan->padded_elems, inv_M, out, x, eta);
    };
    if (!x)
        go(k_unpack_dequant_reduce<B, false, false, false, 1>);
    else if (form.once) // (form.stream: such calls take W = 2)
        go(k_unpack_dequant_reduce<B, true, false, true, 1>);
    else
        go(k_unpack_dequant_reduce<B, true, false, false, 1>);
    return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
}

int reduce_entry(const dq_plan_t* plan, const uint8_t* packed_dev, int64_t packed_worker_stride_bytes, int M,
                 const float* norms_dev, int b, float* out_dev, float* x_dev, float eta, void* hip_stream)
{
    if (!plan || !packed_dev || !norms_dev || (!out_dev && !x_dev)) return DQ_ERR_INVALID_ARG;
    if (M < 1 || M > DQ_MAX_WORKERS || b < 1 || b > 8) return DQ_ERR_INVALID_ARG;
    if (packed_worker_stride_bytes < dq_packed_bytes(plan, b) || (packed_worker_stride_bytes & 15))
        return DQ_ERR_INVALID_ARG;
    if (!dq_aligned16(packed_dev) || !dq_aligned16(out_dev) || !dq_aligned16(x_dev) ||
        (reinterpret_cast<uintptr_t>(norms_dev) & 3u))
        return DQ_ERR_INVALID_ARG;
    if (x_dev && !(eta == eta)) return DQ_ERR_INVALID_ARG; // NaN learning rate
    const int rc = dq_plan_check_device(plan);
    if (rc != DQ_OK) return rc;
    if (plan->padded_elems == 0) return DQ_OK;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    switch (b) {
    case 1: return launch<1>(plan, packed_dev, packed_worker_stride_bytes, M, norms_dev, out_dev, x_dev, eta, stream);
    case 2: return launch<2>(plan, packed_dev, packed_worker_stride_bytes, M, norms_dev, out_dev, x_dev, eta, stream);
    case 3: return launch<3>(plan, packed_dev, packed_worker_stride_bytes, M, norms_dev, out_dev, x_dev, eta, stream);
    case 4: return launch<4>(plan, packed_dev, packed_worker_stride_bytes, M, norms_dev, out_dev, x_dev, eta, stream);
    case 5: return launch<5>(plan, packed_dev, packed_worker_stride_bytes, M, norms_dev, out_dev, x_dev, eta, stream);
    case 6: return launch<6>(plan, packed_dev, packed_worker_stride_bytes, M, norms_dev, out_dev, x_dev, eta, stream);
    case 7: return launch<7>(plan, packed_dev, packed_worker_stride_bytes, M, norms_dev, out_dev, x_dev, eta, stream);
    default: return launch<8>(plan, packed_dev, packed_worker_stride_bytes, M, norms_dev, out_dev, x_dev, eta, stream);
    }
}

} // namespace

extern "C" int dq_unpack_dequant_reduce(const dq_plan_t* plan, const uint8_t* packed_dev,
                                        int64_t packed_worker_stride_bytes, int M, const float* norms_dev,
                                        int b, float* out_dev, void* hip_stream)
{
    if (!out_dev) return DQ_ERR_INVALID_ARG;
    return reduce_entry(plan, packed_dev, packed_worker_stride_bytes, M, norms_dev, b, out_dev, nullptr, 0.0f,
                        hip_stream);
}

extern "C" int dq_unpack_dequant_reduce_update(const dq_plan_t* plan, const uint8_t* packed_dev,
                                               int64_t packed_worker_stride_bytes, int M,
                                               const float* norms_dev, int b, float eta, float* x_dev,
                                               float* ghat_dev, void* hip_stream)
{
    if (!x_dev) return DQ_ERR_INVALID_ARG;
    return reduce_entry(plan, packed_dev, packed_worker_stride_bytes, M, norms_dev, b, ghat_dev, x_dev, eta,
                        hip_stream);
}
