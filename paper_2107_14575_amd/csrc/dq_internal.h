// Internal declarations shared by the translation units of libdq (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "dq.h"

// One piece of a segment handed to one workgroup of the norm kernel: `count` valid elements
// starting at padded index `start` (a multiple of 128), all inside segment `seg`.
struct dq_norm_item {
    int64_t start;
    int32_t count;
    int32_t seg;
};

constexpr int DQ_NORM_CHUNK = 4096; // elements per norm item (one workgroup, 4 float4 per lane)

// Which tensor a 4096-element chunk of the padded index space belongs to: cseg (compact index, see
// below) and seg when all of its elements are there and are data of that one tensor; otherwise cseg = -1
// and seg is the tensor of its first element.
// Almost every chunk of a gradient of large tensors is of the first kind, and a kernel then gets by
// with two scalar loads in place of the granule table (32 entries per chunk and worker).
struct __align__(8) dq_chunk_tensor {
    int32_t cseg;
    int32_t seg;
};
// both words in one scalar load (k is the same for the whole workgroup)
__device__ __forceinline__ dq_chunk_tensor dq_load_chunk_tensor(const dq_chunk_tensor* __restrict__ table, int64_t k)
{
    const uint64_t v = reinterpret_cast<const uint64_t*>(table)[k];
    return dq_chunk_tensor{ static_cast<int32_t>(static_cast<uint32_t>(v)), static_cast<int32_t>(v >> 32) };
}

// Up to this many workgroups the norms take one launch (k_norm_partial<., true>): a small call is its launches.  Norms, quantize and
// reduce, us: 5000 values, M = 4 16.7 -> 13.3 (100 000, 100 workgroups 16.8 -> 13.2; 2^19, M = 1, 128 of them 16.7 -> 13.2), with the rule on the
// device 22.8 -> 19.4, with it on the host 32.2 -> 29.9.  Every arrival writes its XCD's cache back, one after the other, some
// 50 ns each: 200 workgroups 16.5 -> 15.4, 400 16.8 -> 19.8, 1024 16.5 -> 36.
constexpr int DQ_ARRIVE_WORKGROUPS = 160;

// A gradient cut into buckets of 128 << log values, log <= 3, with a last tensor of any length: the first `chunks` chunks hold nothing but whole buckets, so
// that granule g belongs to tensor g >> log and no table has to say so.  chunks = 0: another kind of plan.
struct dq_buckets {
    uint32_t chunks;
    int32_t log;
};

// Kernels that stream the gradient keep more requests in flight than the memory needs when all the workgroups that fit a CU are resident, and
// lose some of its rate.  A launch of many rounds of workgroups asks for so much LDS that fewer are: DQ_LDS_PER_CU / n less what rounding takes.
constexpr int64_t DQ_LDS_PER_CU = 160 * 1024;
// Four rounds of 2048: iterations with 8192 workgroups a pass 73.6 -> 73.2 us, with 16 000 to 82 000 1 to 2.5 % less, with 4300 0.8 % more.
constexpr int64_t DQ_MANY_WORKGROUPS = 8192;
inline constexpr size_t dq_lds_for(int per_cu) { return static_cast<size_t>(DQ_LDS_PER_CU / per_cu - 512); }

struct dq_plan {
    int32_t n_seg;
    int64_t padded_elems; // D'
    int64_t* seg_len;     // host [n_seg]
    int64_t* seg_start;   // host [n_seg + 1]
    int32_t n_items;      // norm work items
    int device;           // HIP device the tables live on, -1 if none
    int32_t n_cseg;       // number of non-empty segments
    bool chunk_local;     // no segment crosses a multiple of 4096 in the padded index space
    // At least a quarter of the chunks are of one tensor: the quantize kernels then look for them (see
    // quantize_pack_chunk).  Against the form that does not, b = 1, 4, 6 take 1.02, 1.0, 1.04 of its time with no such
    // chunk (tensors of 3000), 0.98, 0.96, 1.03 at 13 % (4700), 0.95, 0.94, 0.99 at 32 % (6000).
    bool many_whole;
    bool mostly_whole; // dq_mostly_whole
    dq_buckets buckets;
    void* d_tables;       // the one device allocation that holds all of the tables below
    // device tables.  Kernels address segments through a compact index c that counts only the
    // non-empty ones, so consecutive granules differ by at most one in c.
    dq_chunk_tensor* d_chunk_tensor; // [ceil(D'/4096)]
    int32_t* d_granule_cseg;       // [D'/128]  compact segment index of each 128-element granule
    int32_t* d_cseg_seg;           // [n_nonempty] segment l of compact index c
    int64_t* d_cseg_valid_end;     // [n_nonempty] P_l + len_l: first padded index past the data
    int64_t* d_cseg_start;         // [n_nonempty] P_l
    int32_t* d_span_cseg;          // [n_span] compact indices of the tensors that cross a multiple of 4096
    int32_t n_span;                //          padded elements (all others lie inside one chunk)
    int64_t span_chunks;           // the most chunks that one of them touches
    dq_norm_item* d_items;         // [n_items]
    int32_t* d_seg_item_begin;     // [n_seg + 1] items of segment l are [begin[l], begin[l+1])
    int32_t* d_finish_seg;         // [n_finish] segments whose norm needs the finishing kernel: all but
    int32_t n_finish;              //            those of exactly one item (the first kernel finishes these)
    // [DQ_ARRIVE_WORKGROUPS], of which [M][n_seg] are used: items of a segment that have arrived, zero between calls; null where one
    // worker has more items than that or a segment none (every segment having one, M * n_seg counters are no more than M * n_items).
    // The one part of a plan that a kernel writes: only for calls on the default stream, which run one after the other
    // whatever thread makes them and cannot be captured (see dq_norm.hip).
    uint32_t* d_arrived;
};

// Per-tensor bit-widths (dq_widths_*): one entry per non-empty segment, indexed like the plan's
// compact tables.
struct dq_cseg_width {
    int64_t level_start; // byte offset of the segment's level fields inside the level plane (multiple of 16)
    int64_t seg_start;   // P_l
    int32_t b;           // level bits of the segment, 1..8
    int32_t reserved;
};

struct dq_widths {
    const dq_plan* plan;
    int32_t n_workers;       // 1: the workers share the widths; M: one row of the table per worker
    dq_cseg_width* d_table;  // device [n_workers][plan->n_cseg]
    dq_cseg_width* h_stage;  // pinned host staging of the same size
    hipEvent_t uploaded;     // recorded after the last upload; the staging is reused only after it
    double* d_worker_sq;     // device [DQ_MAX_WORKERS]: per-worker squared norms between the rule's kernels
    int64_t packed_bytes;    // message size for the widths last set (the longest worker's), -1 before the first set
    int64_t* worker_bytes;   // [n_workers] message size of each row
    int32_t* b_host;         // [n_workers][n_seg] widths last set
};

// Workspace of dq_norm_quantize_pack_bracketed, four parts, each starting on a multiple of 256 bytes:
//   partial sums of squares, one binary64 slot per (worker, chunk, tensor in the chunk) at index
//     chunk + c (c = the tensor's compact index: both grow along the layout, so the sum is unique
//     and a tensor's slots are contiguous);
//   one 512-byte block per (worker, chunk) with the elements whose level the bracket left open;
//   one byte per (worker, non-empty tensor): 1 if the norm came out inside its bracket;
//   one bit per (worker, chunk), 64 chunks to a word: chunks that have to be quantized again.
constexpr int DQ_BRACKET_CAP = 63; // records per block
struct dq_bracket_block {
    uint32_t count; // open elements found (may exceed DQ_BRACKET_CAP: then the chunk is redone)
    uint32_t flags; // bit 0: a tensor in the chunk had no usable bracket, nothing was quantized;
                    // bit 1: the chunk was quantized again in full
    uint2 rec[DQ_BRACKET_CAP]; // .x = element index inside the chunk, .y = the gradient value's bits
};
static_assert(sizeof(dq_bracket_block) == 512, "one block per (worker, chunk), 512 bytes");

struct dq_bracket_layout {
    int64_t n_chunks, n_slots, n_words;
    int64_t blocks_at, inside_at, redo_at, total; // byte offsets into the workspace
};
static inline dq_bracket_layout dq_bracket_layout_of(const dq_plan* plan, int M)
{
    auto up = [](int64_t v) { return (v + 255) / 256 * 256; };
    dq_bracket_layout L;
    L.n_chunks = (plan->padded_elems + 4095) / 4096;
    L.n_slots = L.n_chunks + plan->n_cseg;
    L.n_words = (L.n_chunks + 63) / 64;
    L.blocks_at = up(static_cast<int64_t>(M) * L.n_slots * 8);
    L.inside_at = L.blocks_at + static_cast<int64_t>(M) * L.n_chunks * static_cast<int64_t>(sizeof(dq_bracket_block));
    L.redo_at = L.inside_at + up(static_cast<int64_t>(M) * plan->n_cseg);
    L.total = L.redo_at + up(static_cast<int64_t>(M) * L.n_words * 8);
    return L;
}

// Whether the norm pass runs with fewer workgroups resident and its partial sums written through: many workgroups that stream, i.e. whose items
// are nearly full.  Small tensors are an item each, and a workgroup with a few hundred values is latency and no stream: six workgroups per CU for
// eight took 1.15 to 1.4 of the time there (129 000 tensors of 1 to 400 values, M = 32, max norm 2866 -> 4016 us), items of 2500 to 3000 values on average
// 1.04 to 1.11, of 3500 0.97 to 1.04, of 3750 and more 0.91 to 1.02 (9000 to 40 000 items).
static inline bool dq_norm_streams(int64_t workgroups, int64_t padded_elems, int64_t n_items)
{
    return workgroups >= DQ_MANY_WORKGROUPS && padded_elems >= n_items * (DQ_NORM_CHUNK / 8 * 7);
}

// At least half of a layout's chunks are of one tensor: which form k_sign_pack has.
static inline bool dq_mostly_whole(int64_t n_whole, int64_t n_chunks) { return 2 * n_whole >= n_chunks; }

static inline bool dq_aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// sum_l N_l^2 of one worker's row of norms in binary64: blocks of DQ_SUM_BLOCK tensors, each added
// in index order, then the block sums in index order (the plain running sum up to 1024 tensors).
// Host and device rules share this order so that they agree bit for bit.
constexpr int DQ_SUM_BLOCK = 1024;
static inline double dq_worker_squared_norm(const float* row, int32_t n_seg)
{
    double total = 0.0;
    for (int32_t base = 0; base < n_seg; base += DQ_SUM_BLOCK) {
        double block = 0.0;
        for (int32_t l = base; l < n_seg && l < base + DQ_SUM_BLOCK; ++l)
            block += static_cast<double>(row[l]) * static_cast<double>(row[l]);
        total += block;
    }
    return total;
}

// Looks up this GPU's copy of dq_norm_static_scratch's scratch array (`device` is the current
// device), so that the entry point itself finds it ready.
void dq_norm_static_scratch_prepare(int device);

// Fills n floats with +0 (a kernel, not a memset: callers may capture the entry points in a graph).
int dq_zero_floats(float* dst_dev, int64_t n, hipStream_t stream);

// Checks shared by the device entry points; returns DQ_OK when `plan` can launch work on its GPU
// and makes that GPU current.
int dq_plan_check_device(const dq_plan* plan);

// Launches are checked through the thread's last runtime error.  One that an earlier call of the program left there
// (hipErrorInvalidDevice was seen where torch had just allocated new blocks) is not this call's: it is dropped
// before the first launch, and dq_plan_check_device does so.
inline void dq_forget_earlier_errors() { (void)hipGetLastError(); }

// Streaming accesses: data that passes through once (a gradient or a message being read, a message or the averaged
// gradient being written) is loaded and stored with the non-temporal hint, so it does not displace what the caches
// could keep.  Measured at D = 2^28, M = 16, b = 4: quantize+pack 3.67 -> 3.48 ms with such stores, the reduce
// 0.68 -> 0.59 ms with such loads and stores, the norm pass 2.69 -> 2.57 ms with such loads.  The hint pays where one
// load instruction covers whole cache lines (dq_load_wave_tile); where a line is met by several it costs instead
// (quantize+pack with two 16-byte loads per lane 4 %; the level loads of widths 5 to 7 in the reduce).
typedef uint32_t dq_v4u __attribute__((ext_vector_type(4)));
typedef float dq_v4f __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void dq_store_stream(uint4* dst, const uint4& v)
{
    const dq_v4u t = { v.x, v.y, v.z, v.w };
    __builtin_nontemporal_store(t, reinterpret_cast<dq_v4u*>(dst));
}
__device__ __forceinline__ void dq_store_stream(float4* dst, const float4& v)
{
    const dq_v4f t = { v.x, v.y, v.z, v.w };
    __builtin_nontemporal_store(t, reinterpret_cast<dq_v4f*>(dst));
}
// A buffer over `bytes` bytes at an address that is the same for the whole wavefront.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dq_bytes_buffer(const void* at, uint32_t bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(at);
    const uint64_t uniform = (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(a >> 32)))) << 32) |
                             static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(a)));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(uniform), 0, static_cast<int>(bytes), 0x00020000);
}
// Stores of data that passes through once carry the streaming hint (STREAM); otherwise they go through the XCD's own cache
// to the last-level one, where the next kernel finds the data.  A plain store leaves its line dirty in the XCD's cache instead; the
// next kernel then waits for up to 32 MB of such lines to be written back, or fetches them from another XCD one by one.
// Past the buffer's end nothing is stored, and loads give zero.
template <bool STREAM>
__device__ __forceinline__ void dq_store_buffer(const __amdgpu_buffer_rsrc_t buffer, uint32_t byte, const uint4& v)
{
    constexpr int NON_TEMPORAL = 2, DEVICE_SCOPE = 16; // nt, sc1
    const dq_v4u t = { v.x, v.y, v.z, v.w };
    __builtin_amdgcn_raw_buffer_store_b128(t, buffer, static_cast<int>(byte), 0, STREAM ? NON_TEMPORAL : DEVICE_SCOPE);
}
template <bool STREAM>
__device__ __forceinline__ float4 dq_load_buffer(const __amdgpu_buffer_rsrc_t buffer, uint32_t byte)
{
    constexpr int NON_TEMPORAL = 2;
    const dq_v4u t = __builtin_amdgcn_raw_buffer_load_b128(buffer, static_cast<int>(byte), 0, STREAM ? NON_TEMPORAL : 0);
    return make_float4(__uint_as_float(t.x), __uint_as_float(t.y), __uint_as_float(t.z), __uint_as_float(t.w));
}
__device__ __forceinline__ float4 dq_load_stream(const float4* src)
{
    const dq_v4f t = __builtin_nontemporal_load(reinterpret_cast<const dq_v4f*>(src));
    return make_float4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ uint32_t dq_load_stream(const uint32_t* src) { return __builtin_nontemporal_load(src); }

// Runs f with a width as a compile-time constant (widths outside 1..8 are never uploaded).
template <typename F>
__device__ __forceinline__ void dq_with_width(int b, F&& f)
{
    switch (b) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    default: break;
    }
}

// What the wavefront's lanes wrote to LDS becomes visible to its other lanes (no other wavefront takes
// part, so no workgroup barrier).
__device__ __forceinline__ void dq_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wavefront's tile of 512 consecutive elements, lane l receiving elements [8l, 8l + 8) in lo, hi.
// Two 16-byte loads per lane of eight consecutive elements each would use half of every cache line
// per instruction, so that the line has to be kept for the second one: the streaming hint then costs
// 4 %.  Instead each instruction covers 1 KiB in full -- the first one elements [0, 256) of the tile:
// lanes 0..31 the first four elements of lanes 0..31's eight, lanes 32..63 the last four; the second
// one [256, 512) the same way for lanes 32..63 -- with the streaming hint, and four swaps between the
// halves of the wavefront put every lane's own elements in place.
// The loads are buffer loads over the workgroup's n_elems elements: one address register serves all of a lane's tiles
// (the rest is the instruction's immediate offset), and what lies past the end reads as zero.  As global loads with
// clamped offsets a lane's four loads took fourteen instructions more.
//   base       the tile's first element, relative to the buffer
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dq_elems_buffer(const float* g, uint32_t n_elems)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g), 0, static_cast<int>(n_elems * 4u), 0x00020000);
}
__device__ __forceinline__ void dq_load_wave_tile(const __amdgpu_buffer_rsrc_t buffer, uint32_t base, uint32_t lane,
                                                  float4& lo, float4& hi)
{
    const uint32_t at = (base + (lane & 31u) * 8u + (lane >> 5) * 4u) * 4u;
    lo = dq_load_buffer<true>(buffer, at);
    hi = dq_load_buffer<true>(buffer, at + 1024u);
}
__device__ __forceinline__ void dq_swap_halves(float& a, float& b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
// the second half of the load: call it where the values are first used
__device__ __forceinline__ void dq_arrange_wave_tile(float4& lo, float4& hi)
{
    dq_swap_halves(lo.x, hi.x);
    dq_swap_halves(lo.y, hi.y);
    dq_swap_halves(lo.z, hi.z);
    dq_swap_halves(lo.w, hi.w);
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two 32x32->64 multiplies, key
// bumped by the Weyl constants between rounds.  The three-input XOR is one v_bitop3_b32.
__device__ __forceinline__ uint32_t dq_xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ void dq_philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                 uint32_t k0, uint32_t k1, uint32_t (&out)[4])
{
    constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = static_cast<uint64_t>(M0) * c0;
        const uint64_t p1 = static_cast<uint64_t>(M1) * c2;
        const uint32_t n0 = dq_xor3(static_cast<uint32_t>(p1 >> 32), c1, k0);
        const uint32_t n2 = dq_xor3(static_cast<uint32_t>(p0 >> 32), c3, k1);
        c1 = static_cast<uint32_t>(p1);
        c3 = static_cast<uint32_t>(p0);
        c0 = n0;
        c2 = n2;
        k0 += W0;
        k1 += W1;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}
