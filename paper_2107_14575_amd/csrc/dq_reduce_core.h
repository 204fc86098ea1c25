// What the server's reduce kernels share: decoding of a lane's fields, the sum over the workers, and the way out through LDS.
#pragma once
#include <utility>

#include "dq_internal.h"

namespace {

constexpr int UR_THREADS = 256;
// W workers share a decoded word: a lane owns 32 / W elements of each.
//   W = 1: 32 elements, 94 to 128 registers, four wavefronts per SIMD.
//   W = 2: 16 elements, half of a word one worker's and half the next one's, so that the decoding below is the same and as cheap; 62 to 80
//   registers and half the LDS: six wavefronts per SIMD, twice as many in all, which hide the latency of tables, messages and model, and the last
//   round of workgroups is half as long.  See ur_two_workers for where it pays.
template <int W> constexpr int ur_per_lane = 32 / W;
template <int W> constexpr int ur_tile = UR_THREADS * ur_per_lane<W>; // 8192 or 4096 elements
template <int W> constexpr int ur_wave_elems = 64 * ur_per_lane<W>;
template <int W> constexpr int ur_wave_segs = ur_wave_elems<W> / DQ_GRANULE;
template <int W> constexpr int ur_max_local_seg = ur_tile<W> / DQ_GRANULE;

// Widths 1 to 4 take the sign-and-level route below: the byte (sign << 7) | level, level <= 15,
// read as an 8-bit float (E4M3: 4 exponent bits with bias 7, 3 fraction bits) is exactly
// +-level * 2^-9 -- its subnormals and its first binade of normal numbers share one spacing -- so
// one conversion instruction turns two such bytes into two signed binary32 levels, with no
// separate sign handling per element.  Sums formed this way carry the factor 2^-9; the caller
// takes it out together with 1/M (UR_FP8_SCALE).
__host__ __device__ constexpr bool ur_fp8_width(int b) { return b >= 1 && b <= 4; }
constexpr float UR_FP8_SCALE = 512.0f;
// the 32 KiB output tile in LDS allows four workgroups per CU, i.e. four wavefronts per SIMD: the register
// budget is held to what keeps that many resident
constexpr int UR_MIN_WAVES = 4;
constexpr int UR_SUM_BLOCK = 8; // workers per block of the two-level sum (a power of two)
// workers whose loads are issued together (measured per width at D = 2^28, M = 16)
// (b = 3, 4: with eight the kernels that hold all widths need no spills)
__host__ __device__ constexpr int ur_group(int b) { return b <= 2 ? 16 : b <= 4 ? 8 : 4; }
// W = 2, six wavefronts per SIMD: eight workers' loads fit where their dwords are at most two.  M = 16, b = 4 at 2^26 155 (four) -> 150 us; b = 8 with eight
// spills (transformer shape 51 -> 64).
template <int W> __host__ __device__ constexpr int ur_group_of(int b) { return W == 1 ? ur_group(b) : b <= 4 ? 8 : 4; }
// The same in the kernel of one width, where sixteen fit at b = 4 too: 2^28 x 16 607 -> 587 us (b = 3: 524 -> 520
// there, but 17.2 -> 18.0 us on the ResNet-18 shape, M = 8, so it stays at eight).
template <int W> __host__ __device__ constexpr int ur_group_one_width(int b) { return W == 1 && b == 4 ? 16 : ur_group_of<W>(b); }
// (W = 2, b = 7 with update spills three registers at six)
template <int W> __host__ __device__ constexpr int ur_min_waves(int b) { return W == 1 ? UR_MIN_WAVES : b == 7 ? 5 : 6; }
// Whether the wavefront's table of units comes before the first group's loads.  One width: the message bytes do
// not depend on the tensors, so those loads can go ahead, and at b >= 5 they do.  But loads return in order, and
// the table's own then wait for the whole group, which costs more than it hides where a worker's bytes are few:
// at b <= 4 the table comes first, and a barrier after it lets the workgroup's wavefronts start on their
// neighbouring bytes together.  Measured against the loads first, in us: 2^28 x 16 b = 1 397 -> 381, b = 2
// 455 -> 444; 2^26 x 16 b = 1 110.6 -> 99.2; ResNet-18 shape, M = 8, b = 1, 2, 3 17.4, 18.3, 18.9 -> 14.2, 15.3,
// 17.2 (without the barrier 15.0, 15.7, 17.2).  At b = 8 it is the other way round: that shape with update
// 29.3 -> 31.8.
__host__ __device__ constexpr bool ur_table_first(int b) { return b <= 4; }

// Widths whose level loads carry the streaming hint in some calls only (ur_stream).
__host__ __device__ constexpr bool ur_may_stream(int b) { return b >= 5 && b <= 7; }

// bytes of {hi, lo} picked by the four selector bytes of sel: 0..3 = bytes of lo, 4..7 = bytes of hi
__device__ __forceinline__ uint32_t byte_perm(uint32_t hi, uint32_t lo, uint32_t sel)
{
    return __builtin_amdgcn_perm(hi, lo, sel);
}

// t holds the levels (<= 15) of elements e, e+8, e+16, e+24 of the lane, one per byte; the sign bits
// of those elements are bits e, e+8, e+16, e+24 of sg.  acc[.] += sgn * level * 2^-9 * unit.
template <int W>
struct ur_units { float of[W]; };
template <int E, int W>
__device__ __forceinline__ void fma_signed_bytes(uint32_t t, uint32_t sg, const ur_units<W>& unit, float (&acc)[ur_per_lane<W>])
{
    const uint32_t coded = ((sg << (7 - E)) & 0x80808080u) | t; // sign bits onto bit 7 of each byte
    const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(coded), false); // bytes 0, 1
    const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(coded), true);  // bytes 2, 3
    constexpr int H = W == 1 ? 16 : 0;
    acc[E] = __builtin_fmaf(lo[0], unit.of[0], acc[E]);
    acc[E + 8] = __builtin_fmaf(lo[1], unit.of[0], acc[E + 8]);
    acc[E + H] = __builtin_fmaf(hi[0], unit.of[W - 1], acc[E + H]);
    acc[E + 8 + H] = __builtin_fmaf(hi[1], unit.of[W - 1], acc[E + 8 + H]);
}

// Width 3: y[i] holds byte i of each of the lane's four 24-bit runs (eight 3-bit fields each); the
// levels of elements E, E+8, E+16, E+24 one per byte.  Fields 2 and 5 of a run straddle two bytes.
template <int E>
__device__ __forceinline__ uint32_t level_bytes_b3(const uint32_t (&y)[3])
{
    constexpr int bit = 3 * E, word = bit >> 3, off = bit & 7;
    if constexpr (off + 3 <= 8) {
        return (y[word] >> off) & 0x07070707u;
    } else {
        constexpr uint32_t lo_mask = ((1u << (8 - off)) - 1u) * 0x01010101u;
        constexpr uint32_t hi_mask = ((1u << (off + 3 - 8)) - 1u) * 0x01010101u;
        return ((y[word] >> off) & lo_mask) | ((y[word + 1] & hi_mask) << (8 - off));
    }
}

template <int B, int W, int... E>
__device__ __forceinline__ void accumulate_words_fp8(uint32_t sg, const uint32_t (&wd)[B], const ur_units<W>& unit,
                                                     float (&acc)[ur_per_lane<W>], std::integer_sequence<int, E...>)
{
    static_assert(sizeof...(E) == 8, "eight groups of four elements");
    if constexpr (B == 1) {
        // bit e + 8j of the one level dword is bit e of its byte j
        (fma_signed_bytes<E, W>((wd[0] >> E) & 0x01010101u, sg, unit, acc), ...);
    } else if constexpr (B == 2) {
        // byte r of dword q holds elements 16q + 4r .. + 3: gather bytes r, r+2 of both dwords
        const uint32_t q[2] = { byte_perm(wd[1], wd[0], 0x06040200u), byte_perm(wd[1], wd[0], 0x07050301u) };
        (fma_signed_bytes<E, W>((q[E / 4] >> (2 * (E % 4))) & 0x03030303u, sg, unit, acc), ...);
    } else if constexpr (B == 3) {
        // the lane's 96 level bits are four runs of 24 (elements 8j .. 8j+7): gather byte i of every run
        const uint32_t y[3] = { byte_perm(wd[2], byte_perm(wd[1], wd[0], 0x00060300u), 0x05020100u),
                                byte_perm(wd[2], byte_perm(wd[1], wd[0], 0x00070401u), 0x06020100u),
                                byte_perm(wd[2], byte_perm(wd[1], wd[0], 0x00000502u), 0x07040100u) };
        (fma_signed_bytes<E, W>(level_bytes_b3<E>(y), sg, unit, acc), ...);
    } else {
        // byte r of dword j holds elements 8j + 2r, 8j + 2r + 1: transpose the 4x4 bytes so that word r
        // holds byte r of every dword
        const uint32_t ab_lo = byte_perm(wd[1], wd[0], 0x05010400u), ab_hi = byte_perm(wd[1], wd[0], 0x07030602u);
        const uint32_t cd_lo = byte_perm(wd[3], wd[2], 0x05010400u), cd_hi = byte_perm(wd[3], wd[2], 0x07030602u);
        const uint32_t p[4] = { byte_perm(cd_lo, ab_lo, 0x05040100u), byte_perm(cd_lo, ab_lo, 0x07060302u),
                                byte_perm(cd_hi, ab_hi, 0x05040100u), byte_perm(cd_hi, ab_hi, 0x07060302u) };
        (fma_signed_bytes<E, W>((p[E / 2] >> (4 * (E % 2))) & 0x0F0F0F0Fu, sg, unit, acc), ...);
    }
}

// Widths 5 to 8: the half-word (sign << 15) | level << (8 - B), read as a 16-bit float, is a subnormal
// number (its exponent field is zero): exactly +-level * 2^(-16-B).  One mixed-precision FMA
// (v_fma_mix_f32) takes it as it is, so that two elements share the extraction and the sign handling.
// With the unit times 2^(B-1) every product is the true one times 2^-17, which the caller takes out
// together with 1/M (UR_FP16_SCALE): at most 0.52 N, so nothing overflows that did not before, and at
// least 2^-125 for a usable norm (2^-100), so every product is a normal number and rounds as the true
// one does -- the sums are bit for bit those of convert, sign merge and FMA in binary32.
// About 3.4 vector instructions per worker and element at B = 5, 6, 7 and 2.5 at B = 8, one of them (the FMA)
// at half rate, against 5 and 4.
// The pairs are elements (E, E + 16) of the lane: 16 fields are B half-words, so the words
// p[i] = {half-word i + B, half-word i} hold both elements' fields at the same place, and bits E and
// E + 16 of the sign dword are as far apart as the half-words' sign bits.
typedef _Float16 ur_half2 __attribute__((ext_vector_type(2)));
__host__ __device__ constexpr float ur_unit_factor(int b) { return ur_fp8_width(b) ? 1.0f : static_cast<float>(1 << (b - 1)); }
constexpr float UR_FP16_SCALE = 131072.0f;
__host__ __device__ constexpr float ur_sum_scale(int b) { return ur_fp8_width(b) ? UR_FP8_SCALE : UR_FP16_SCALE; }

template <int D> // shift left by D, or right by -D
__device__ __forceinline__ uint32_t shift_by(uint32_t v)
{
    if constexpr (D >= 0)
        return v << D;
    else
        return v >> -D;
}

template <int B, int E, int W>
__device__ __forceinline__ void fma_signed_halves(const uint32_t (&p)[B], uint32_t sg, const ur_units<W>& unit, float (&acc)[ur_per_lane<W>])
{
    constexpr int word = (E * B) >> 4, off = (E * B) & 15, J = 8 - B;
    const uint32_t sign = (sg << (15 - E)) & 0x80008000u;
    uint32_t coded;
    if constexpr (off + B <= 16) {
        constexpr uint32_t MASK = (((1u << B) - 1u) << J) * 0x00010001u;
        coded = (shift_by<J - off>(p[word]) & MASK) | sign;
    } else { // the field straddles two half-words
        constexpr int LOW = 16 - off; // bits of it in the first one
        constexpr uint32_t MASK_LO = (((1u << LOW) - 1u) << J) * 0x00010001u;
        constexpr uint32_t MASK_HI = (((1u << (B - LOW)) - 1u) << (J + LOW)) * 0x00010001u;
        coded = (shift_by<J - off>(p[word]) & MASK_LO) | sign;
        coded = ((p[word + 1 < B ? word + 1 : word] << (J + LOW)) & MASK_HI) | coded;
    }
    const ur_half2 h = __builtin_bit_cast(ur_half2, coded);
    constexpr int H = W == 1 ? 16 : 0;
    acc[E] = __builtin_fmaf(static_cast<float>(h[0]), unit.of[0], acc[E]);
    acc[E + H] = __builtin_fmaf(static_cast<float>(h[1]), unit.of[W - 1], acc[E + H]);
}

template <int E, int W> // B = 8: the two bytes come out by one permute each pair
__device__ __forceinline__ void fma_signed_halves_b8(const uint32_t (&wd)[8], uint32_t sg, const ur_units<W>& unit, float (&acc)[ur_per_lane<W>])
{
    constexpr uint32_t SEL = 0x0C000C00u | (E % 4) | ((4u + E % 4) << 16); // 0x0C: a zero byte
    const uint32_t coded = byte_perm(wd[E / 4 + 4], wd[E / 4], SEL) | ((sg << (15 - E)) & 0x80008000u);
    const ur_half2 h = __builtin_bit_cast(ur_half2, coded);
    constexpr int H = W == 1 ? 16 : 0;
    acc[E] = __builtin_fmaf(static_cast<float>(h[0]), unit.of[0], acc[E]);
    acc[E + H] = __builtin_fmaf(static_cast<float>(h[1]), unit.of[W - 1], acc[E + H]);
}

template <int B, int W, int... E>
__device__ __forceinline__ void accumulate_words_fp16(uint32_t sg, const uint32_t (&wd)[B], const ur_units<W>& unit,
                                                      float (&acc)[ur_per_lane<W>], std::integer_sequence<int, E...>)
{
    static_assert(sizeof...(E) == 16, "sixteen pairs of elements");
    if constexpr (B == 8) {
        (fma_signed_halves_b8<E, W>(wd, sg, unit, acc), ...);
    } else {
        uint32_t p[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const uint32_t lo = wd[i >> 1], hi = wd[(i + B) >> 1];
            const uint32_t sel = ((i & 1) ? 0x0302u : 0x0100u) | (((i + B) & 1) ? 0x07060000u : 0x05040000u);
            p[i] = byte_perm(hi, lo, sel);
        }
        (fma_signed_halves<B, E, W>(p, sg, unit, acc), ...);
    }
}

// One worker's contribution to a lane's 32 elements from the worker's sign dword and its B level
// dwords: acc[k] += sgn_k * level_k * unit, divided by ur_sum_scale(B); unit is N/s times
// ur_unit_factor(B).
template <int B, int W>
__device__ __forceinline__ void accumulate_words(uint32_t sg, const uint32_t (&wd)[B], const ur_units<W>& unit,
                                                 float (&acc)[ur_per_lane<W>])
{
    if constexpr (ur_fp8_width(B))
        accumulate_words_fp8<B, W>(sg, wd, unit, acc, std::make_integer_sequence<int, 8>{});
    else
        accumulate_words_fp16<B, W>(sg, wd, unit, acc, std::make_integer_sequence<int, 16>{});
}

// A lane's 8 / W 16-byte slots of the workgroup's output tile in LDS (XOR-swizzled: conflict free for
// the lane's own accesses and for the transposed read of finish_tile).  Before that read a lane's
// slots are its own, so it also keeps the running total of its block sums there.
template <int W>
struct lane_slots {
    static constexpr int N = 8 / W; // slots a lane
    float4* wave_out; // this wavefront's 64 * N slots
    int lane;
    static __device__ __forceinline__ int at(int lane, int q) { return lane * N + (q ^ (W == 1 ? lane & 7 : (lane >> 1) & 3)); }
    __device__ __forceinline__ float4& operator[](int q) const { return wave_out[at(lane, q)]; }
};
template <int W>
__device__ __forceinline__ lane_slots<W> slots_of(float4* lds_out, int tid)
{
    return lane_slots<W>{ lds_out + (tid >> 6) * (64 * lane_slots<W>::N), tid & 63 };
}

// Sum of blocks, kept without a second set of 32 registers: every block but the last is added to the
// lane's slots (the first one stored), and the accumulators start the next block from zero.
template <int W>
struct block_total {
    lane_slots<W> slots;
    int n_flushed = 0;
    __device__ __forceinline__ void flush(float (&acc)[ur_per_lane<W>])
    {
#pragma unroll
        for (int q = 0; q < 8 / W; ++q) {
            float4 t = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
            if (n_flushed) {
                const float4 o = slots[q];
                t = make_float4(o.x + t.x, o.y + t.y, o.z + t.z, o.w + t.w);
            }
            slots[q] = t;
            acc[4 * q] = acc[4 * q + 1] = acc[4 * q + 2] = acc[4 * q + 3] = 0.0f;
        }
        ++n_flushed;
    }
    // total of the flushed blocks plus the block still in the accumulators
    __device__ __forceinline__ void finish(float (&acc)[ur_per_lane<W>]) const
    {
        if (!n_flushed) return;
#pragma unroll
        for (int q = 0; q < 8 / W; ++q) {
            const float4 o = slots[q];
            acc[4 * q] = o.x + acc[4 * q];
            acc[4 * q + 1] = o.y + acc[4 * q + 1];
            acc[4 * q + 2] = o.z + acc[4 * q + 2];
            acc[4 * q + 3] = o.w + acc[4 * q + 3];
        }
    }
};

// A lane's B level dwords of one worker, by the widest loads their size allows (a global load needs no
// more than dword alignment).  Where one load takes them all (b <= 4), the lanes' loads cover whole cache lines
// and the streaming hint pays at the largest sizes.  Where a line is met by several loads (5 to 7) it has to
// stay unless they are many (STREAM; see ur_stream): with the hint b = 7 took 36.7 instead of 32.5 us on 11 M elements, M = 8.
typedef uint32_t ur_v4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t ur_v3u __attribute__((ext_vector_type(3), aligned(4)));
typedef uint32_t ur_v2u __attribute__((ext_vector_type(2), aligned(4)));
#define UR_GLOBAL __attribute__((address_space(1)))
typedef const UR_GLOBAL uint8_t* ur_bytes;
// An address that is the same for the whole wavefront, kept as one pair of scalar registers: left alone the
// compiler adds the lane's offset first and carries a vector register pair per load around the loop over
// the workers (22 to 41 of them spilled at B = 2, 3, 4).
__device__ __forceinline__ ur_bytes scalar_address(const uint8_t* at)
{
    uint64_t a = reinterpret_cast<uint64_t>(at);
    asm("" : "+s"(a));
    return reinterpret_cast<ur_bytes>(a);
}
__device__ __forceinline__ ur_bytes global_address(const uint8_t* at)
{
    return reinterpret_cast<ur_bytes>(reinterpret_cast<uint64_t>(at));
}
template <bool STREAM, typename T>
__device__ __forceinline__ T load_dwords(ur_bytes at)
{
    if constexpr (STREAM)
        return __builtin_nontemporal_load(reinterpret_cast<const UR_GLOBAL T*>(at));
    else
        return *reinterpret_cast<const UR_GLOBAL T*>(at);
}
template <int B, bool STREAM>
__device__ __forceinline__ void load_levels(ur_bytes at, uint32_t (&wd)[B])
{
#pragma unroll
    for (int q = 0; q + 4 <= B; q += 4) {
        const ur_v4u t = load_dwords<STREAM, ur_v4u>(at + 4 * q);
        wd[q] = t.x; wd[q + 1] = t.y; wd[q + 2] = t.z; wd[q + 3] = t.w;
    }
    constexpr int Q = B & ~3;
    if constexpr ((B & 3) == 3) {
        const ur_v3u t = load_dwords<STREAM, ur_v3u>(at + 4 * Q);
        wd[Q] = t.x; wd[Q + 1] = t.y; wd[Q + 2] = t.z;
    } else if constexpr ((B & 3) == 2) {
        const ur_v2u t = load_dwords<STREAM, ur_v2u>(at + 4 * Q);
        wd[Q] = t.x; wd[Q + 1] = t.y;
    } else if constexpr ((B & 3) == 1) {
        wd[Q] = load_dwords<STREAM, uint32_t>(at + 4 * Q);
    }
}

// a worker's dwords as a lane loads them: its 32 / W fields, at odd widths and W = 2 with the half-word before or after them
template <int B, int W> constexpr int ur_raw = W == 1 ? B : (B + 1) / 2;

// W = 2: the two workers' sixteen fields one after the other, as 32 fields of one lane.  Odd widths: a lane's fields are B half-words, and
// the odd lanes' start with the second half of their first dword.
template <int B>
__device__ __forceinline__ void join_pair(const uint32_t (&a)[ur_raw<B, 2>], const uint32_t (&b)[ur_raw<B, 2>], int lane, uint32_t (&wd)[B])
{
    constexpr int m = B / 2;
    if constexpr (B % 2 == 0) {
#pragma unroll
        for (int k = 0; k < m; ++k) {
            wd[k] = a[k];
            wd[m + k] = b[k];
        }
    } else {
        const bool odd = (lane & 1) != 0;
        wd[m] = byte_perm(b[0], a[m], odd ? 0x07060302u : 0x05040100u);
        const uint32_t first = odd ? 0x05040302u : 0x03020100u, second = odd ? 0x07060504u : 0x05040302u;
#pragma unroll
        for (int k = 0; k < m; ++k) {
            wd[k] = byte_perm(a[k + 1], a[k], first);
            wd[m + 1 + k] = byte_perm(b[k + 1], b[k], second);
        }
    }
}

// The same from eight loaded dwords of which the first B count (per-worker widths).
template <int B>
__device__ __forceinline__ void accumulate_first_words(uint32_t sg, const uint32_t (&wd8)[8], float unit,
                                                       float (&acc)[ur_per_lane<1>])
{
    uint32_t wd[B];
#pragma unroll
    for (int q = 0; q < B; ++q) wd[q] = wd8[q];
    accumulate_words<B, 1>(sg, wd, ur_units<1>{ { unit } }, acc);
}

// The M workers' contributions to a lane's elements: acc[k] += sgn * level * unit, workers in
// ascending order.  load(w, sg, wd) fetches worker w's sign dword and B level dwords of the lane,
// unit(w) is its unit for the lane's tensor.  WAVE: called by accumulate_wave.  prepare() runs once, when
// the first group's loads are on their way: what unit(w) needs and those loads do not belongs there.
//
// Workers in groups whose loads are all issued before the first is used: the pass is bound by
// memory latency once the arithmetic is cheap, so narrow widths (few registers per worker) take
// large groups.  Groups halve towards the end, so any M keeps its loads batched.
//
// Order of the additions: workers ascending inside blocks of UR_SUM_BLOCK workers (an FMA chain
// from zero), the block sums added in block order.  However the loads are grouped, a value
// passes through at most 7 + ceil(M/8) roundings: 15 at M = 64, where a single chain over all
// workers would take 63 (and measurably leaves the 1e-6 tolerance when one worker's norm
// dominates).  Up to eight workers nothing is flushed: the plain chain.
// JOIN: the last block joins the total; otherwise the flushed blocks' total stays in the slots and the last block in acc.
template <int B, int W, bool WAVE, int GROUP, bool JOIN = true, typename Load, typename Prepare, typename Unit>
__device__ __forceinline__ void accumulate_workers(int M, Load&& load, Prepare&& prepare, Unit&& unit,
                                                   float (&acc)[ur_per_lane<W>], lane_slots<W> slots)
{
    block_total<W> total{ slots };
    auto group = [&](auto g, int w) { // w is a multiple of G
        constexpr int G = decltype(g)::value;
        uint32_t sg[G], raw[G][ur_raw<B, W>];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            load(w + i, sg[i], raw[i]);
            // Narrow fields: the loads in the order of their use.  Left to itself the compiler puts most sign
            // dwords behind the levels, and the second worker waits for six loads: b = 1 at 2^28 x 16 380 -> 374
            // us, b = 2 and 3 on 2^24 values in tensors of 512, M = 8 23.1 -> 22.4 and 25.1 -> 24.5.  With
            // wider ones its order is the better one (2^28 x 16: b = 4 586 against 629 us, b = 7 877 against 957).
            if constexpr (B <= 3) __builtin_amdgcn_sched_barrier(0);
        }
        if (w == 0) prepare();
        if constexpr (W == 1) {
#pragma unroll
            for (int i = 0; i < G; ++i) {
                if constexpr (WAVE && B == 8) { // halves of the wavefront trade pieces (accumulate_wave)
#pragma unroll
                    for (int q = 0; q < B / 2; ++q) {
                        const auto t = __builtin_amdgcn_permlane32_swap(raw[i][q], raw[i][q + B / 2], false, false);
                        raw[i][q] = t[0];
                        raw[i][q + B / 2] = t[1];
                    }
                }
                accumulate_words<B, 1>(sg[i], raw[i], ur_units<1>{ { unit(w + i) } }, acc);
                if constexpr (G >= UR_SUM_BLOCK) {
                    if ((i + 1) % UR_SUM_BLOCK == 0 && w + i + 1 < M) total.flush(acc);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < G; i += 2) {
                uint32_t wd[B], sign;
                ur_units<2> u;
                u.of[0] = unit(w + i);
                if constexpr (G == 1) { // nobody to share with: a second worker of unit zero adds nothing
                    const uint32_t none[ur_raw<B, 2>] = {};
                    join_pair<B>(raw[0], none, slots.lane, wd);
                    sign = sg[0];
                    u.of[1] = 0.0f;
                } else {
                    join_pair<B>(raw[i], raw[i + 1], slots.lane, wd);
                    sign = sg[i] | (sg[i + 1] << 16);
                    u.of[1] = unit(w + i + 1);
                }
                accumulate_words<B, 2>(sign, wd, u, acc);
                if constexpr (G >= UR_SUM_BLOCK) {
                    if ((i + 2) % UR_SUM_BLOCK == 0 && w + i + 2 < M) total.flush(acc);
                }
            }
        }
        if constexpr (G < UR_SUM_BLOCK) {
            if (((w + G) & (UR_SUM_BLOCK - 1)) == 0 && w + G < M) total.flush(acc);
        }
    };
    int w = 0;
    for (; w + GROUP <= M; w += GROUP) group(std::integral_constant<int, GROUP>{}, w);
    if constexpr (GROUP > 8) if (w + 8 <= M) { group(std::integral_constant<int, 8>{}, w); w += 8; }
    if constexpr (GROUP > 4) if (w + 4 <= M) { group(std::integral_constant<int, 4>{}, w); w += 4; }
    if constexpr (GROUP > 2) if (w + 2 <= M) { group(std::integral_constant<int, 2>{}, w); w += 2; }
    if (w < M) group(std::integral_constant<int, 1>{}, w);
    if constexpr (JOIN) total.finish(acc);
}

// Lanes of different tensors: sign_ptr / level_ptr address worker 0's sign dword and level dwords of the
// lane, unit_ptr[w] (LDS) is worker w's unit for the lane's tensor.
template <int W>
__device__ __forceinline__ uint32_t load_sign(ur_bytes at)
{
    if constexpr (W == 1)
        return load_dwords<true, uint32_t>(at);
    else
        return __builtin_nontemporal_load(reinterpret_cast<const UR_GLOBAL uint16_t*>(at));
}
template <int B, int W>
__device__ __forceinline__ void accumulate_lane(const uint8_t* __restrict__ sign_ptr,
                                                const uint8_t* __restrict__ level_ptr, int64_t packed_stride,
                                                int M, const float* unit_ptr, float (&acc)[ur_per_lane<W>],
                                                lane_slots<W> slots)
{
    if constexpr (W == 2 && B % 2 != 0) level_ptr -= (slots.lane & 1) * 2;
    accumulate_workers<B, W, false, ur_group_of<W>(B) / 2>(
        M,
        [&](int w, uint32_t& sg, uint32_t (&wd)[ur_raw<B, W>]) {
            int64_t off = static_cast<int64_t>(w) * packed_stride; // scalar, for the reason given at scalar_address
            asm("" : "+s"(off));
            sg = load_sign<W>(global_address(sign_ptr + off));
            load_levels<ur_raw<B, W>, B <= 4 || (W == 2 && B == 8)>(global_address(level_ptr + off), wd);
        },
        [] {}, [&](int w) { return unit_ptr[w]; }, acc, slots);
}

// All lanes of a wavefront with one place for their level bytes: sign_wave addresses worker 0's sign bytes
// of the wavefront's first element and level_wave(w) worker w's level bytes of it, the same for all lanes,
// so a worker's address is scalar arithmetic.  Lanes past the end (n_lanes, a multiple of 4 W, exist) fetch
// the last ones' bytes.
// W = 2: one load takes a worker's fields whatever the width.  The streaming hint stays off at B = 5 to 7 all the same unless STREAM says otherwise: with it on,
// reduces of messages in no cache gain 1 to 2 % and iterations whose messages are still there lose (2^25 to 2^26 values, M = 3 b = 7 without update 172 -> 186 us).
// W = 1: at B = 8 a lane's dwords are two 16-byte pieces: each load instruction covers 1 KiB in full (lanes
// 0..31 and 32..63 take the first and second pieces of 32 lanes) and swaps between the halves of the
// wavefront put the pieces in place, so that the streaming hint can stay on.
template <int B, int W, int GROUP, bool STREAM, bool JOIN = true, typename LevelWave, typename Prepare, typename Unit>
__device__ __forceinline__ void accumulate_wave(const uint8_t* __restrict__ sign_wave, LevelWave&& level_wave,
                                                int64_t packed_stride, int M, Prepare&& prepare, Unit&& unit, int n_lanes,
                                                float (&acc)[ur_per_lane<W>], lane_slots<W> slots)
{
    const uint32_t lane = slots.lane < n_lanes ? slots.lane : n_lanes - 1;
    uint32_t at0 = lane * (4u * B / W), at1 = 0;
    if constexpr (W == 2 && B % 2 != 0) at0 -= (lane & 1u) * 2u;
    if constexpr (W == 1 && B == 8) {
        const uint32_t end = n_lanes * 32u - 16u;
        at0 = (slots.lane & 31) * 32u + (slots.lane >> 5) * 16u;
        at1 = at0 + 1024u < end ? at0 + 1024u : end;
        at0 = at0 < end ? at0 : end;
    }
    accumulate_workers<B, W, true, GROUP, JOIN>(
        M,
        [&](int w, uint32_t& sg, uint32_t (&wd)[ur_raw<B, W>]) {
            const ur_bytes lp = scalar_address(level_wave(w));
            sg = load_sign<W>(scalar_address(sign_wave + static_cast<int64_t>(w) * packed_stride) + lane * (4u / W));
            if constexpr (W == 1 && B == 8) {
                const ur_v4u a = load_dwords<true, ur_v4u>(lp + at0);
                const ur_v4u b = load_dwords<true, ur_v4u>(lp + at1);
                wd[0] = a.x; wd[1] = a.y; wd[2] = a.z; wd[3] = a.w;
                wd[4] = b.x; wd[5] = b.y; wd[6] = b.z; wd[7] = b.w;
            } else {
                load_levels<ur_raw<B, W>, STREAM || !ur_may_stream(B)>(lp + at0, wd);
            }
        },
        prepare, unit, acc, slots);
}

// The model's elements [first, first + n) of a wavefront (first is the same for all its lanes), by their index from `first`.
// What lies past the layout's end is read as zero and not written.
// ONCE: it passes through with the streaming hint; otherwise it is left in the last-level cache for the next iteration.
template <bool ONCE>
struct ur_model {
    __amdgpu_buffer_rsrc_t buffer;
    ur_model() = default;
    __device__ __forceinline__ ur_model(float* x, int64_t first, int n, int64_t padded_elems)
        : buffer(dq_bytes_buffer(x + first, static_cast<uint32_t>(padded_elems - first < n ? padded_elems - first : n) * 4u))
    {
    }
    __device__ __forceinline__ float4 load(int at) const { return dq_load_buffer<ONCE>(buffer, at * 4u); }
    __device__ __forceinline__ void store(int at, const float4& v) const
    {
        dq_store_buffer<ONCE>(buffer, at * 4u, make_uint4(__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)));
    }
};

// x - eta * g_hat (pads: g_hat is +0, x unchanged)
__device__ __forceinline__ float4 ur_step(float4 x, const float4& g, float eta)
{
    x.x = __builtin_fmaf(-eta, g.x, x.x);
    x.y = __builtin_fmaf(-eta, g.y, x.y);
    x.z = __builtin_fmaf(-eta, g.z, x.z);
    x.w = __builtin_fmaf(-eta, g.w, x.w);
    return x;
}

// Scales a lane's sums by 1/M (zero beyond the tensor's end), transposes the wavefront's elements
// (from padded index wave0 on) through LDS and writes them out; with UPDATE it also applies the model update to x (and then
// `out` may be null).
template <int W, bool UPDATE, bool ONCE = false>
__device__ __forceinline__ void finish_tile(float (&acc)[ur_per_lane<W>], bool active, int64_t n_valid, float inv_M,
                                            float4* lds_out, int tid, int64_t wave0, int64_t padded_elems,
                                            float* __restrict__ out, float* __restrict__ x, float eta)
{
    constexpr int N = 8 / W, PL = ur_per_lane<W>; // 16-byte pieces and elements of a lane
    if (active) {
        const int nv = n_valid >= PL ? PL : (n_valid > 0 ? static_cast<int>(n_valid) : 0);
#pragma unroll
        for (int k = 0; k < PL; ++k) acc[k] = k < nv ? acc[k] * inv_M : 0.0f;
    }
    const int lane = tid & 63;
    // the model's pieces, all in flight before the first is used (each load behind the store before it cost a
    // memory latency apiece)
    float4 xv[N];
    ur_model<ONCE> model;
    if constexpr (UPDATE) {
        model = ur_model<ONCE>(x, wave0, ur_wave_elems<W>, padded_elems);
#pragma unroll
        for (int j = 0; j < N; ++j) xv[j] = model.load(256 * j + 4 * lane);
    }
    const lane_slots<W> slots = slots_of<W>(lds_out, tid);
#pragma unroll
    for (int q = 0; q < N; ++q) slots[q] = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    // the transposition stays inside the wavefront's own slots: its lanes only have to see one
    // another's LDS writes, no other wavefront's
    dq_wave_sync();
    // piece j of the wave covers its elements [256j, 256j + 256); this lane takes 4 of them
    auto piece = [&](int j) { return slots.wave_out[lane_slots<W>::at((64 / N) * j + lane / N, lane % N)]; };
    if constexpr (!UPDATE) {
        // one after the other behind their bounds checks: eight stores in one go took 161 instead of 152 us at
        // D = 2^26, M = 16, b = 4
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int64_t P = wave0 + 256 * j + 4 * lane;
            if (P < padded_elems) dq_store_stream(reinterpret_cast<float4*>(out + P), piece(j));
        }
    } else { // model update of Algorithm 1: x <- x - eta * g_hat (pads: g_hat is +0, x unchanged)
        float4 v[N];
#pragma unroll
        for (int j = 0; j < N; ++j) v[j] = piece(j);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int64_t P = wave0 + 256 * j + 4 * lane;
            if (out && P < padded_elems) dq_store_stream(reinterpret_cast<float4*>(out + P), v[j]);
            model.store(256 * j + 4 * lane, ur_step(xv[j], v[j], eta));
        }
    }
}

// Which tile a workgroup takes.  Consecutive workgroups go to the eight XCDs in turn; four consecutive
// tiles are given to one XCD (32 tiles, the last 0..31 left as they are), so that a worker's stretch of the
// message is read in pieces of four times a tile's bytes by one of them.  Measured at D = 2^28, M = 16:
// b = 4 with update 905 -> 836 us, without 634 -> 610; b = 8 at 2^26 256 -> 248; groups of two or eight, or
// one contiguous range per XCD, gave less.  (W = 2: eight of its smaller tiles.)
template <int W>
__device__ __forceinline__ uint32_t ur_tile_index()
{
    constexpr uint32_t T = 4u * W;
    const uint32_t i = blockIdx.x;
    return i < gridDim.x / (8u * T) * (8u * T) ? i / (8u * T) * (8u * T) + (i % 8u) * T + i / 8u % T : i;
}

// The elements of a wavefront (2048 or 1024) and the tensors they belong to (compact indices first..last).
struct wave_span {
    int64_t start;  // first padded index
    int n_lanes;    // lanes whose 32 elements exist (a multiple of 4; <= 0: none)
    int32_t first, last;
};
template <int W>
__device__ __forceinline__ wave_span wave_span_from(int64_t start, int64_t padded_elems, const int32_t* __restrict__ granule_cseg)
{
    wave_span s;
    s.start = start;
    s.n_lanes = 0;
    s.first = s.last = 0;
    if (s.start < padded_elems) {
        const int64_t left = padded_elems - s.start;
        s.n_lanes = static_cast<int>(left < ur_wave_elems<W> ? left : ur_wave_elems<W>) / ur_per_lane<W>;
        s.first = granule_cseg[s.start >> 7];
        s.last = granule_cseg[(s.start + s.n_lanes * ur_per_lane<W> - 1) >> 7];
    }
    return s;
}
template <int W>
__device__ __forceinline__ wave_span wave_span_of(int tid, int64_t padded_elems, const int32_t* __restrict__ granule_cseg)
{
    return wave_span_from<W>(static_cast<int64_t>(ur_tile_index<W>()) * ur_tile<W> +
                                 __builtin_amdgcn_readfirstlane(tid >> 6) * ur_wave_elems<W>,
                          padded_elems, granule_cseg);
}

__device__ __forceinline__ float ur_unit(float N, int b)
{
    return N >= DQ_MIN_NORM ? N / static_cast<float>((1 << b) - 1) * ur_unit_factor(b) : 0.0f;
}

// The unit of levels that are whole numbers: the products carry 1 / ur_sum_scale(b) as everywhere (a power of two), so that
// a sum passes the largest value where the other kernels' sums do and not M times sooner.
__device__ __forceinline__ float ur_level_unit(float N, int b)
{
    return N >= DQ_MIN_NORM ? N / static_cast<float>((1 << b) - 1) * (1.0f / ur_sum_scale(b)) : 0.0f;
}

// Worker w's value out of the one each lane holds (M <= 64).
__device__ __forceinline__ float lane_value(float of_lane, int w)
{
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(of_lane), w));
}

// The wavefront's table [tensor of the span][worker] in LDS, value(w, c) of worker w and compact tensor c;
// returns the row of the lane's own tensor and the end of its data relative to P0.  A wavefront inside
// one tensor (nearly every one of a gradient of large tensors) fills one row, a lane each.
template <typename Value>
__device__ __forceinline__ const float* wave_table(const wave_span& span, int lane, int M, int64_t P0,
                                                   const int32_t* __restrict__ granule_cseg,
                                                   const int64_t* __restrict__ cseg_valid_end, float* table,
                                                   int64_t& n_valid, Value&& value)
{
    const int32_t first = __builtin_amdgcn_readfirstlane(span.first), last = __builtin_amdgcn_readfirstlane(span.last);
    int32_t c = first;
    if (first == last) {
        if (lane < M) table[lane] = value(lane, first);
    } else {
        c = granule_cseg[(lane < span.n_lanes ? P0 : span.start) >> 7]; // lanes past the end: the first one's
        const int n_local = last - first + 1; // <= UR_WAVE_SEGS: compact indices grow by <= 1 per granule
        for (int i = lane; i < n_local * M; i += 64) {
            const int local = i / M, w = i - local * M;
            table[i] = value(w, first + local);
        }
    }
    n_valid = cseg_valid_end[c] - P0;
    dq_wave_sync();
    return table + (c - first) * M;
}
// Whether the level loads of widths 5 to 7 carry the streaming hint although several of them meet a cache line: with the
// update, where messages and model together are more than half of the last-level cache, so that the messages do not push the model
// out.  Measured over 1 to 270 M values, M = 1..31: the reduce alone, messages from memory, 16.8 M, M = 16 b = 5 65 -> 55 us, 20 M,
// M = 4 b = 7 44.5 -> 40.2; whole iterations (norm, quantize, reduce) 11.2 M, M = 16 b = 7 315 -> 303; below, where an iteration's
// messages are still in the cache, it costs (ResNet-18 shape, M = 8 28.8 -> 30.1).  Without update it gains 3 to 7 % of iterations with 200
// to 400 MB of messages and loses up to 9 % where they come from memory.  With more than 32 workers and W = 1 (three workgroups per CU, the
// vector ALU as much as the loads) it loses there too: 4.2 M ragged elements, M = 64 b = 5 56 -> 62, transformer shape, M = 62 b = 5 113 -> 128; with W = 2
// it gains: 11 to 20 M, M = 47 and 64 b = 5 to 7 1.0 -> 0.88 of the time with W = 1.  There the line lies at 100 MB: without the hint iterations in which neither model nor messages
// are in the cache at the start take 1.0 to 1.04 of the time at 100 to 128 MB and 0.97 to 1.0 below, those in which both are from the last iteration
// 0.96 to 0.99 at 60 to 128 MB and 0.99 to 1.04 below.
// Without update and with W = 2 it is for messages of more than 640 MB, of which next to nothing is in the cache: 2^28 values, M = 16 b = 5, 6, 7 0.71, 0.82, 0.90 ->
// 0.69, 0.80, 0.88 ms; iterations are the same with and without it from 400 MB on, and up to 260 MB they lose 1 to 10 % by it.
constexpr int64_t UR_LAST_LEVEL_CACHE = 256 << 20, UR_STREAM_FROM = 100 << 20, UR_STREAM_MESSAGES_FROM = 640 << 20;
inline bool ur_stream(const dq_plan* plan, int M, int b, bool two, bool update)
{
    if (!ur_may_stream(b)) return false;
    const int64_t messages = M * dq_packed_bytes(plan, b);
    if (!update) return two && messages > UR_STREAM_MESSAGES_FROM;
    return (two || M <= 32) && messages + plan->padded_elems * 4 > (two ? UR_STREAM_FROM : UR_LAST_LEVEL_CACHE / 2);
}
// Whether the model passes through with the hint: a large one would not be in the cache when it is next read, and takes the
// messages' place.  Iterations with b = 2 and 8, us, model left in the cache / passing through: 2^24, M = 2 73 / 77, M = 8 (b = 8) 233 / 230;
// 21 M, M = 2 92 / 95, M = 32 969 / 929; 2^25, M = 2 149 / 141, M = 32 1500 / 1474; 2^26, M = 2 288 / 271.  The reduce alone: 22 M, M = 16 b = 8
// 91 / 97, 28 M 134 / 125.  Where the line lies depends on the workers too (with 32 of them passing through gains from 21 M on already); by
// elements alone it lies where few and many are even.  Left plainly, in the XCDs' own caches, models of 14 to 24 M took 1 to 9 % of an
// iteration longer (21 M, b = 2, M = 2 113 us against 105, M = 32 969 against 946).
constexpr int64_t UR_ONCE_ELEMS = 24 << 20;
inline bool ur_model_once(const dq_plan* plan) { return plan->padded_elems > UR_ONCE_ELEMS; }

// Runs f(STREAM, ONCE) with the two as compile-time constants.
template <bool MAY_STREAM, typename F>
inline void ur_with_policy(bool stream, bool once, F&& f)
{
    using yes = std::true_type;
    using no = std::false_type;
    using streamed = std::integral_constant<bool, MAY_STREAM>;
    if (stream && once) f(streamed{}, yes{});
    else if (stream) f(streamed{}, no{});
    else if (once) f(no{}, yes{});
    else f(no{}, no{});
}

// Whether two workers share a decoded word (W = 2).  b = 0: a widths table, which the GPU may have filled.  A tile is 8192 elements: one workgroup at W = 1,
// two at W = 2.  Measured with 6 to 32 768 tiles, M = 1 to 64, all widths, messages in no cache (time with W = 2 / with W = 1):
//   up to 384 tiles 0.76 to 1.04, all together 0.94;
//   up to 1280 (five to a CU; tables with update 768) what counts is whether the fullest CU has less to do with half tiles, 2 n / 256 rounded up against n / 256: where it
//   does (an odd number of 128 tiles) b >= 5 from four workers on (from six where one round of W = 1, 1024 tiles, takes all and one of W = 2, 768, does not: M = 4 and 5 1.03
//   to 1.1 there) and b <= 4 and tables from ten on 0.83 to 1.0; where it does not 0.96 to 1.16 (512 tiles, M = 16 b = 4
//   1.16), b = 5 to 7 with update from six workers on 0.85 to 0.99.  With fewer workers the wavefronts' start and the decoding, twice for an odd one, decide: 0.98 to 1.36;
//   beyond, without update b = 2 and b >= 4 for six to thirteen workers 0.93 to 1.0, b = 4 to 7 for sixteen 0.95 to 1.0 where the planes are on cache lines and 0.98 to
//   1.04 where they are not (tables with b = 2, 4, 6, 8 1.0 to 1.05, 0.96 to 1.02, 0.95 to 0.99, 0.97 to 1.0), the others 0.98 to 1.24 (b = 3: M = 1 1.24, M = 16 1.03; b = 8, M = 16 0.99 to 1.03);
//   with update 0.85 to 1.0 for six to sixteen workers (b = 8 from three on), with a table for three to 32, at b = 5 to 7 for one to 32; with more, whose messages are read in pieces of half the size,
//   1.0 to 1.08, but b = 5 to 7 and tables 0.87 to 0.96 while the model stays in the cache; with fewer, or b = 1, 0.96 to 1.12 there and 0.93 to 0.99 where it passes through.
// Whole iterations say the same, less sharply (b = 3, 2^26 to 2^28 values, M = 1 to 4, no update: 1.04 to 1.12 with W = 2).
inline bool ur_two_workers(int64_t n_tiles, int b, int M, bool update, bool once)
{
    const bool halves = b >= 5 && b <= 7;
    if (n_tiles <= 384) return true;
    if (n_tiles <= (update && b == 0 ? 768 : 1280)) {
        const bool less = (n_tiles + 127) / 128 % 2 != 0; // for the fullest CU with half tiles
        if (!less) return halves && update && M >= 6;
        return M >= (b < 5 ? 10 : n_tiles > 768 && n_tiles <= 1024 ? 6 : 4);
    }
    if (!update) return M >= 6 && M <= (b == 2 || b == 8 ? 13 : 16) && b != 1 && b != 3;
    if (!once && !halves && (M < (b == 0 || b == 8 ? 3 : 6) || b == 1)) return false;
    return M <= (!halves && b != 0 ? 16 : once ? 32 : 64);
}

// The form that a call takes.  b as above.
struct ur_form {
    bool two;    // W = 2
    bool stream; // the hint on the level loads of widths 5 to 7
    bool once;   // with update: the hint on the model
};
// rows: a widths table with a row per worker (W = 1 only)
inline ur_form ur_form_of(const dq_plan* plan, int b, int M, bool update, bool rows = false)
{
    const int64_t n_tiles = (plan->padded_elems + ur_tile<1> - 1) / ur_tile<1>;
    ur_form f;
    f.once = update && ur_model_once(plan);
    f.two = !rows && ur_two_workers(n_tiles, b, M, update, f.once);
    f.stream = ur_stream(plan, M, b ? b : 6, f.two, update); // six bits stand for widths that the GPU may have set
    return f;
}

} // namespace
