// dq_unpack_dequant_reduce: the server average of Algorithm 1 / Eq. (2),
//     out_P = (1/M) sum_i sgn_{i,P} * level_{i,P} * (N_{i,l} / s),
// with every worker's message read exactly once.
//
// Work split.  One workgroup (256 lanes) owns 8192 consecutive padded elements; a lane owns 32 of
// them, so per worker it reads one sign dword and B level dwords -- every load is dword aligned
// for every B -- and keeps 32 binary32 accumulators.
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
// 15.0, 15.4, 16.9 -> 14.6, 15.3, 16.7 (see ur_table_first).
//
// The 32 results of a lane are consecutive in memory, so storing them directly would be 16-byte
// pieces 128 bytes apart; they go through LDS (XOR-swizzled 16-byte slots, conflict free both
// ways) and leave as fully coalesced 16-byte stores.
//
// Each wavefront works out the units N/s of its own tensors.
//
// HBM traffic per output element: M(B+1)/8 bytes read, 4 bytes written.
//
// With a model vector x the epilogue also applies the update of Algorithm 1, x <- x - eta * g_hat
// (8 more bytes per element, read and written with the same coalesced 16-byte accesses).
#include <utility>

#include "dq_internal.h"

namespace {

constexpr int UR_THREADS = 256;
constexpr int UR_PER_LANE = 32;
constexpr int UR_TILE = UR_THREADS * UR_PER_LANE; // 8192 elements
constexpr int UR_MAX_LOCAL_SEG = UR_TILE / DQ_GRANULE;
constexpr int UR_WAVE_ELEMS = 64 * UR_PER_LANE; // 2048 elements
constexpr int UR_WAVE_SEGS = UR_WAVE_ELEMS / DQ_GRANULE;

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
// The same in the kernel of one width, where sixteen fit at b = 4 too: 2^28 x 16 607 -> 587 us (b = 3: 524 -> 520
// there, but 17.2 -> 18.0 us on the ResNet-18 shape, M = 8, so it stays at eight).
__host__ __device__ constexpr int ur_group_one_width(int b) { return b == 4 ? 16 : ur_group(b); }
// Whether the wavefront's table of units comes before the first group's loads.  One width: the message bytes do
// not depend on the tensors, so those loads can go ahead, and at b >= 5 they do.  But loads return in order, and
// the table's own then wait for the whole group, which costs more than it hides where a worker's bytes are few:
// at b <= 4 the table comes first, and a barrier after it lets the workgroup's wavefronts start on their
// neighbouring bytes together.  Measured against the loads first, in us: 2^28 x 16 b = 1 397 -> 381, b = 2
// 455 -> 444; 2^26 x 16 b = 1 110.6 -> 99.2; ResNet-18 shape, M = 8, b = 1, 2, 3 17.4, 18.3, 18.9 -> 14.2, 15.3,
// 17.2 (without the barrier 15.0, 15.7, 17.2).  At b = 8 it is the other way round: that shape with update
// 29.3 -> 31.8.
__host__ __device__ constexpr bool ur_table_first(int b) { return b <= 4; }

// bytes of {hi, lo} picked by the four selector bytes of sel: 0..3 = bytes of lo, 4..7 = bytes of hi
__device__ __forceinline__ uint32_t byte_perm(uint32_t hi, uint32_t lo, uint32_t sel)
{
    return __builtin_amdgcn_perm(hi, lo, sel);
}

// t holds the levels (<= 15) of elements e, e+8, e+16, e+24 of the lane, one per byte; the sign bits
// of those elements are bits e, e+8, e+16, e+24 of sg.  acc[.] += sgn * level * 2^-9 * unit.
template <int E>
__device__ __forceinline__ void fma_signed_bytes(uint32_t t, uint32_t sg, float unit, float (&acc)[UR_PER_LANE])
{
    const uint32_t coded = ((sg << (7 - E)) & 0x80808080u) | t; // sign bits onto bit 7 of each byte
    const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(coded), false); // bytes 0, 1
    const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(coded), true);  // bytes 2, 3
    acc[E] = __builtin_fmaf(lo[0], unit, acc[E]);
    acc[E + 8] = __builtin_fmaf(lo[1], unit, acc[E + 8]);
    acc[E + 16] = __builtin_fmaf(hi[0], unit, acc[E + 16]);
    acc[E + 24] = __builtin_fmaf(hi[1], unit, acc[E + 24]);
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

template <int B, int... E>
__device__ __forceinline__ void accumulate_words_fp8(uint32_t sg, const uint32_t (&wd)[B], float unit,
                                                     float (&acc)[UR_PER_LANE], std::integer_sequence<int, E...>)
{
    static_assert(sizeof...(E) == 8, "eight groups of four elements");
    if constexpr (B == 1) {
        // bit e + 8j of the one level dword is bit e of its byte j
        (fma_signed_bytes<E>((wd[0] >> E) & 0x01010101u, sg, unit, acc), ...);
    } else if constexpr (B == 2) {
        // byte r of dword q holds elements 16q + 4r .. + 3: gather bytes r, r+2 of both dwords
        const uint32_t q[2] = { byte_perm(wd[1], wd[0], 0x06040200u), byte_perm(wd[1], wd[0], 0x07050301u) };
        (fma_signed_bytes<E>((q[E / 4] >> (2 * (E % 4))) & 0x03030303u, sg, unit, acc), ...);
    } else if constexpr (B == 3) {
        // the lane's 96 level bits are four runs of 24 (elements 8j .. 8j+7): gather byte i of every run
        const uint32_t y[3] = { byte_perm(wd[2], byte_perm(wd[1], wd[0], 0x00060300u), 0x05020100u),
                                byte_perm(wd[2], byte_perm(wd[1], wd[0], 0x00070401u), 0x06020100u),
                                byte_perm(wd[2], byte_perm(wd[1], wd[0], 0x00000502u), 0x07040100u) };
        (fma_signed_bytes<E>(level_bytes_b3<E>(y), sg, unit, acc), ...);
    } else {
        // byte r of dword j holds elements 8j + 2r, 8j + 2r + 1: transpose the 4x4 bytes so that word r
        // holds byte r of every dword
        const uint32_t ab_lo = byte_perm(wd[1], wd[0], 0x05010400u), ab_hi = byte_perm(wd[1], wd[0], 0x07030602u);
        const uint32_t cd_lo = byte_perm(wd[3], wd[2], 0x05010400u), cd_hi = byte_perm(wd[3], wd[2], 0x07030602u);
        const uint32_t p[4] = { byte_perm(cd_lo, ab_lo, 0x05040100u), byte_perm(cd_lo, ab_lo, 0x07060302u),
                                byte_perm(cd_hi, ab_hi, 0x05040100u), byte_perm(cd_hi, ab_hi, 0x07060302u) };
        (fma_signed_bytes<E>((p[E / 2] >> (4 * (E % 2))) & 0x0F0F0F0Fu, sg, unit, acc), ...);
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

template <int B, int E>
__device__ __forceinline__ void fma_signed_halves(const uint32_t (&p)[B], uint32_t sg, float unit, float (&acc)[UR_PER_LANE])
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
    acc[E] = __builtin_fmaf(static_cast<float>(h[0]), unit, acc[E]);
    acc[E + 16] = __builtin_fmaf(static_cast<float>(h[1]), unit, acc[E + 16]);
}

template <int E> // B = 8: the two bytes come out by one permute each pair
__device__ __forceinline__ void fma_signed_halves_b8(const uint32_t (&wd)[8], uint32_t sg, float unit, float (&acc)[UR_PER_LANE])
{
    constexpr uint32_t SEL = 0x0C000C00u | (E % 4) | ((4u + E % 4) << 16); // 0x0C: a zero byte
    const uint32_t coded = byte_perm(wd[E / 4 + 4], wd[E / 4], SEL) | ((sg << (15 - E)) & 0x80008000u);
    const ur_half2 h = __builtin_bit_cast(ur_half2, coded);
    acc[E] = __builtin_fmaf(static_cast<float>(h[0]), unit, acc[E]);
    acc[E + 16] = __builtin_fmaf(static_cast<float>(h[1]), unit, acc[E + 16]);
}

template <int B, int... E>
__device__ __forceinline__ void accumulate_words_fp16(uint32_t sg, const uint32_t (&wd)[B], float unit,
                                                      float (&acc)[UR_PER_LANE], std::integer_sequence<int, E...>)
{
    static_assert(sizeof...(E) == 16, "sixteen pairs of elements");
    if constexpr (B == 8) {
        (fma_signed_halves_b8<E>(wd, sg, unit, acc), ...);
    } else {
        uint32_t p[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const uint32_t lo = wd[i >> 1], hi = wd[(i + B) >> 1];
            const uint32_t sel = ((i & 1) ? 0x0302u : 0x0100u) | (((i + B) & 1) ? 0x07060000u : 0x05040000u);
            p[i] = byte_perm(hi, lo, sel);
        }
        (fma_signed_halves<B, E>(p, sg, unit, acc), ...);
    }
}

// One worker's contribution to a lane's 32 elements from the worker's sign dword and its B level
// dwords: acc[k] += sgn_k * level_k * unit, divided by ur_sum_scale(B); unit is N/s times
// ur_unit_factor(B).
template <int B>
__device__ __forceinline__ void accumulate_words(uint32_t sg, const uint32_t (&wd)[B], float unit,
                                                 float (&acc)[UR_PER_LANE])
{
    if constexpr (ur_fp8_width(B))
        accumulate_words_fp8<B>(sg, wd, unit, acc, std::make_integer_sequence<int, 8>{});
    else
        accumulate_words_fp16<B>(sg, wd, unit, acc, std::make_integer_sequence<int, 16>{});
}

// The same from eight loaded dwords of which the first B count (per-worker widths).
template <int B>
__device__ __forceinline__ void accumulate_first_words(uint32_t sg, const uint32_t (&wd8)[8], float unit,
                                                       float (&acc)[UR_PER_LANE])
{
    uint32_t wd[B];
#pragma unroll
    for (int q = 0; q < B; ++q) wd[q] = wd8[q];
    accumulate_words<B>(sg, wd, unit, acc);
}

// A lane's eight 16-byte slots of the workgroup's output tile in LDS (XOR-swizzled: conflict free for
// the lane's own accesses and for the transposed read of finish_tile).  Before that read a lane's
// slots are its own, so it also keeps the running total of its block sums there.
struct lane_slots {
    float4* wave_out; // this wavefront's 512 slots
    int lane;
    __device__ __forceinline__ float4& operator[](int q) const { return wave_out[lane * 8 + (q ^ (lane & 7))]; }
};
__device__ __forceinline__ lane_slots slots_of(float4* lds_out, int tid)
{
    return lane_slots{ lds_out + (tid >> 6) * 512, tid & 63 };
}

// Sum of blocks, kept without a second set of 32 registers: every block but the last is added to the
// lane's slots (the first one stored), and the accumulators start the next block from zero.
struct block_total {
    lane_slots slots;
    int n_flushed = 0;
    __device__ __forceinline__ void flush(float (&acc)[UR_PER_LANE])
    {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
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
    __device__ __forceinline__ void finish(float (&acc)[UR_PER_LANE]) const
    {
        if (!n_flushed) return;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
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

// The M workers' contributions to a lane's 32 elements: acc[k] += sgn * level * unit, workers in
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
template <int B, bool WAVE, int GROUP, bool JOIN = true, typename Load, typename Prepare, typename Unit>
__device__ __forceinline__ void accumulate_workers(int M, Load&& load, Prepare&& prepare, Unit&& unit,
                                                   float (&acc)[UR_PER_LANE], lane_slots slots)
{
    block_total total{ slots };
    auto group = [&](auto g, int w) { // w is a multiple of G
        constexpr int G = decltype(g)::value;
        uint32_t sg[G], wd[G][B];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            load(w + i, sg[i], wd[i]);
            // Narrow fields: the loads in the order of their use.  Left to itself the compiler puts most sign
            // dwords behind the levels, and the second worker waits for six loads: b = 1 at 2^28 x 16 380 -> 374
            // us, b = 2 and 3 on 2^24 values in tensors of 512, M = 8 23.1 -> 22.4 and 25.1 -> 24.5.  With
            // wider ones its order is the better one (2^28 x 16: b = 4 586 against 629 us, b = 7 877 against 957).
            if constexpr (B <= 3) __builtin_amdgcn_sched_barrier(0);
        }
        if (w == 0) prepare();
#pragma unroll
        for (int i = 0; i < G; ++i) {
            if constexpr (WAVE && B == 8) { // halves of the wavefront trade pieces (accumulate_wave)
#pragma unroll
                for (int q = 0; q < B / 2; ++q) {
                    const auto t = __builtin_amdgcn_permlane32_swap(wd[i][q], wd[i][q + B / 2], false, false);
                    wd[i][q] = t[0];
                    wd[i][q + B / 2] = t[1];
                }
            }
            accumulate_words<B>(sg[i], wd[i], unit(w + i), acc);
            if constexpr (G >= UR_SUM_BLOCK) {
                if ((i + 1) % UR_SUM_BLOCK == 0 && w + i + 1 < M) total.flush(acc);
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
template <int B>
__device__ __forceinline__ void accumulate_lane(const uint8_t* __restrict__ sign_ptr,
                                                const uint8_t* __restrict__ level_ptr, int64_t packed_stride,
                                                int M, const float* unit_ptr, float (&acc)[UR_PER_LANE],
                                                lane_slots slots)
{
    accumulate_workers<B, false, ur_group(B) / 2>(
        M,
        [&](int w, uint32_t& sg, uint32_t (&wd)[B]) {
            int64_t off = static_cast<int64_t>(w) * packed_stride; // scalar, for the reason given at scalar_address
            asm("" : "+s"(off));
            sg = load_dwords<true, uint32_t>(global_address(sign_ptr + off));
            load_levels<B, B <= 4>(global_address(level_ptr + off), wd);
        },
        [] {}, [&](int w) { return unit_ptr[w]; }, acc, slots);
}

// All lanes of a wavefront with one place for their level bytes: sign_wave addresses worker 0's sign bytes
// of the wavefront's first element and level_wave(w) worker w's level bytes of it, the same for all lanes,
// so a worker's address is scalar arithmetic.  Lanes past the end (n_lanes, a multiple of 4, exist) fetch
// the last ones' bytes.
// At B = 8 a lane's dwords are two 16-byte pieces: each load instruction covers 1 KiB in full (lanes
// 0..31 and 32..63 take the first and second pieces of 32 lanes) and swaps between the halves of the
// wavefront put the pieces in place, so that the streaming hint can stay on.
template <int B, int GROUP, bool STREAM, bool JOIN = true, typename LevelWave, typename Prepare, typename Unit>
__device__ __forceinline__ void accumulate_wave(const uint8_t* __restrict__ sign_wave, LevelWave&& level_wave,
                                                int64_t packed_stride, int M, Prepare&& prepare, Unit&& unit, int n_lanes,
                                                float (&acc)[UR_PER_LANE], lane_slots slots)
{
    const uint32_t lane = slots.lane < n_lanes ? slots.lane : n_lanes - 1;
    uint32_t at0 = lane * (4u * B), at1 = 0;
    if constexpr (B == 8) {
        const uint32_t end = n_lanes * 32u - 16u;
        at0 = (slots.lane & 31) * 32u + (slots.lane >> 5) * 16u;
        at1 = at0 + 1024u < end ? at0 + 1024u : end;
        at0 = at0 < end ? at0 : end;
    }
    accumulate_workers<B, true, GROUP, JOIN>(
        M,
        [&](int w, uint32_t& sg, uint32_t (&wd)[B]) {
            const ur_bytes lp = scalar_address(level_wave(w));
            sg = load_dwords<true, uint32_t>(scalar_address(sign_wave + static_cast<int64_t>(w) * packed_stride) + lane * 4u);
            if constexpr (B == 8) {
                const ur_v4u a = load_dwords<true, ur_v4u>(lp + at0);
                const ur_v4u b = load_dwords<true, ur_v4u>(lp + at1);
                wd[0] = a.x; wd[1] = a.y; wd[2] = a.z; wd[3] = a.w;
                wd[4] = b.x; wd[5] = b.y; wd[6] = b.z; wd[7] = b.w;
            } else {
                load_levels<B, STREAM || B <= 4>(lp + at0, wd);
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

// Scales a lane's sums by 1/M (zero beyond the tensor's end), transposes the wavefront's 2048 elements
// (from padded index wave0 on) through LDS and writes them out; with UPDATE it also applies the model update to x (and then
// `out` may be null).
template <bool UPDATE, bool ONCE = false>
__device__ __forceinline__ void finish_tile(float (&acc)[UR_PER_LANE], bool active, int64_t n_valid, float inv_M,
                                            float4* lds_out, int tid, int64_t wave0, int64_t padded_elems,
                                            float* __restrict__ out, float* __restrict__ x, float eta)
{
    if (active) {
        const int nv = n_valid >= UR_PER_LANE ? UR_PER_LANE : (n_valid > 0 ? static_cast<int>(n_valid) : 0);
#pragma unroll
        for (int k = 0; k < UR_PER_LANE; ++k) acc[k] = k < nv ? acc[k] * inv_M : 0.0f;
    }
    // lane t of wave v holds elements [v*2048 + 32t, +32): slot (t, q) -> t*8 + (q ^ (t & 7))
    const int wave = tid >> 6, lane = tid & 63;
    // the model's pieces, all eight in flight before the first is used (each load behind the store before it cost a
    // memory latency apiece)
    float4 xv[8];
    ur_model<ONCE> model;
    if constexpr (UPDATE) {
        model = ur_model<ONCE>(x, wave0, UR_WAVE_ELEMS, padded_elems);
#pragma unroll
        for (int j = 0; j < 8; ++j) xv[j] = model.load(256 * j + 4 * lane);
    }
    float4* wave_out = lds_out + wave * 512;
#pragma unroll
    for (int q = 0; q < 8; ++q)
        wave_out[lane * 8 + (q ^ (lane & 7))] = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    // the transposition stays inside the wavefront's own 512 slots: its lanes only have to see one
    // another's LDS writes, no other wavefront's
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // piece j of the wave covers its elements [256j, 256j + 256); this lane takes 4 of them
    auto piece = [&](int j) {
        const int src_lane = 8 * j + (lane >> 3), q = lane & 7;
        return wave_out[src_lane * 8 + (q ^ (src_lane & 7))];
    };
    if constexpr (!UPDATE) {
        // one after the other behind their bounds checks: eight stores in one go took 161 instead of 152 us at
        // D = 2^26, M = 16, b = 4
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t P = wave0 + 256 * j + 4 * lane;
            if (P < padded_elems) dq_store_stream(reinterpret_cast<float4*>(out + P), piece(j));
        }
    } else { // model update of Algorithm 1: x <- x - eta * g_hat (pads: g_hat is +0, x unchanged)
        float4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = piece(j);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
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
// one contiguous range per XCD, gave less.
__device__ __forceinline__ uint32_t ur_tile_index()
{
    const uint32_t i = blockIdx.x;
    return i < gridDim.x / 32u * 32u ? i / 32u * 32u + (i % 8u) * 4u + i / 8u % 4u : i;
}

// The 2048 elements of a wavefront and the tensors they belong to (compact indices first..last).
struct wave_span {
    int64_t start;  // first padded index
    int n_lanes;    // lanes whose 32 elements exist (a multiple of 4; <= 0: none)
    int32_t first, last;
};
__device__ __forceinline__ wave_span wave_span_from(int64_t start, int64_t padded_elems, const int32_t* __restrict__ granule_cseg)
{
    wave_span s;
    s.start = start;
    s.n_lanes = 0;
    s.first = s.last = 0;
    if (s.start < padded_elems) {
        const int64_t left = padded_elems - s.start;
        s.n_lanes = static_cast<int>(left < UR_WAVE_ELEMS ? left : UR_WAVE_ELEMS) / UR_PER_LANE;
        s.first = granule_cseg[s.start >> 7];
        s.last = granule_cseg[(s.start + s.n_lanes * UR_PER_LANE - 1) >> 7];
    }
    return s;
}
__device__ __forceinline__ wave_span wave_span_of(int tid, int64_t padded_elems, const int32_t* __restrict__ granule_cseg)
{
    return wave_span_from(static_cast<int64_t>(ur_tile_index()) * UR_TILE +
                              __builtin_amdgcn_readfirstlane(tid >> 6) * UR_WAVE_ELEMS,
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

// STREAM: the streaming hint on level loads that would not have it; ONCE: on the model (ur_stream, ur_model_once)
template <int B, bool UPDATE, bool STREAM, bool ONCE>
__global__ __launch_bounds__(UR_THREADS, UR_MIN_WAVES) void k_unpack_dequant_reduce(
    const uint8_t* __restrict__ packed, int64_t packed_stride, int M, const float* __restrict__ norms,
    int32_t n_seg, const int32_t* __restrict__ granule_cseg, const int32_t* __restrict__ cseg_seg,
    const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems, float inv_M, float* __restrict__ out,
    float* __restrict__ x, float eta)
{
    extern __shared__ __align__(16) uint8_t lds_raw[];
    float4* lds_out = reinterpret_cast<float4*>(lds_raw); // [UR_TILE / 4]

    const int tid = threadIdx.x, lane = tid & 63;
    const wave_span span = wave_span_of(tid, padded_elems, granule_cseg);
    const int64_t P0 = span.start + lane * UR_PER_LANE;
    const bool active = lane < span.n_lanes;
    const uint8_t* level_plane = packed + (padded_elems >> 3);

    int64_t n_valid = 0;
    float* table = reinterpret_cast<float*>(lds_raw + UR_TILE * sizeof(float)) + (tid >> 6) * UR_WAVE_SEGS * M;
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

    float acc[UR_PER_LANE];
#pragma unroll
    for (int k = 0; k < UR_PER_LANE; ++k) acc[k] = 0.0f;
    const uint8_t* level_wave = level_plane + (span.start >> 3) * B;
    accumulate_wave<B, ur_group_one_width(B), STREAM>(
        packed + (span.start >> 3), [&](int w) { return level_wave + static_cast<int64_t>(w) * packed_stride; },
        packed_stride, M,
        [&] {
            if constexpr (!ur_table_first(B)) make_table();
        },
        [&](int w) { return unit_ptr[w]; }, span.n_lanes, acc, slots_of(lds_out, tid));
    finish_tile<UPDATE, ONCE>(acc, active, n_valid, inv_M * ur_sum_scale(B), lds_out, tid, span.start, padded_elems, out, x, eta);
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
    const wave_span span = wave_span_from(static_cast<int64_t>(ur_tile_index()) * UR_WAVE_ELEMS, padded_elems, granule_cseg);
    const int64_t P0 = span.start + lane * UR_PER_LANE;
    const int w0 = wave * per_wave * UR_SUM_BLOCK;
    const int n_mine = M - w0 < per_wave * UR_SUM_BLOCK ? M - w0 : per_wave * UR_SUM_BLOCK; // <= 0: none
    const int last = (M - 1) / (per_wave * UR_SUM_BLOCK); // the last wavefront with workers

    const auto piece_at = [&](int j) { return span.start + 256 * (wave * PIECES + j) + 4 * lane; };
    float4 xv[PIECES]; // the model's pieces, in flight from the start
    ur_model<false> model;
    if constexpr (UPDATE) {
        model = ur_model<false>(x, span.start, UR_WAVE_ELEMS, padded_elems);
#pragma unroll
        for (int j = 0; j < PIECES; ++j) xv[j] = model.load(256 * (wave * PIECES + j) + 4 * lane);
    }

    float acc[UR_PER_LANE];
#pragma unroll
    for (int k = 0; k < UR_PER_LANE; ++k) acc[k] = 0.0f;
    const lane_slots slots = slots_of(lds_out, tid);
    int64_t n_valid = 0;
    if (n_mine > 0) { // a wavefront without workers still reaches the barriers and writes its quarter
        const uint8_t* mine = packed + static_cast<int64_t>(w0) * packed_stride;
        const uint8_t* level_wave = mine + (padded_elems >> 3) + (span.start >> 3) * B;
        float* table = reinterpret_cast<float*>(lds_raw + UR_TILE * sizeof(float)) + wave * UR_WAVE_SEGS * per_wave * UR_SUM_BLOCK;
        const float* unit_ptr = wave_table(span, lane, n_mine, P0, granule_cseg, cseg_valid_end, table, n_valid, [&](int w, int32_t c) {
            return ur_unit(norms[static_cast<int64_t>(w0 + w) * n_seg + cseg_seg[c]], B);
        });
        accumulate_wave<B, (B <= 4 ? 8 : 4), false, false>(
            mine + (span.start >> 3), [&](int w) { return level_wave + static_cast<int64_t>(w) * packed_stride; }, packed_stride,
            n_mine, [] {}, [&](int w) { return unit_ptr[w]; }, span.n_lanes, acc, slots);
    }
    for (int r = 0; r <= last; ++r) {
        if (wave == r) {
            const lane_slots before{ lds_out + (wave - 1) * 512, lane };
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
                    const int nv = n_valid >= UR_PER_LANE ? UR_PER_LANE : (n_valid > 0 ? static_cast<int>(n_valid) : 0);
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

// Per-tensor widths: a wavefront inside one tensor takes its b and the place of its level dwords from the
// widths table (scalar) and runs the accumulation specialised for that b.  Elsewhere each lane does: its
// 32 elements lie in one 128-element granule, hence in one segment.
template <bool UPDATE, bool STREAM, bool ONCE> // as in k_unpack_dequant_reduce
__global__ __launch_bounds__(UR_THREADS, UR_MIN_WAVES) void k_unpack_dequant_reduce_v(
    const uint8_t* __restrict__ packed, int64_t packed_stride, int M, const float* __restrict__ norms,
    int32_t n_seg, const int32_t* __restrict__ granule_cseg, const int32_t* __restrict__ cseg_seg,
    const int64_t* __restrict__ cseg_valid_end, const dq_cseg_width* __restrict__ widths, int64_t padded_elems,
    float inv_M, float* __restrict__ out, float* __restrict__ x, float eta)
{
    extern __shared__ __align__(16) uint8_t lds_raw[];
    float4* lds_out = reinterpret_cast<float4*>(lds_raw);

    const int tid = threadIdx.x, lane = tid & 63;
    const wave_span span = wave_span_of(tid, padded_elems, granule_cseg);
    if (span.n_lanes <= 0) return;
    const int64_t P0 = span.start + lane * UR_PER_LANE;
    const bool active = lane < span.n_lanes;
    const uint8_t* level_plane = packed + (padded_elems >> 3);

    float acc[UR_PER_LANE];
#pragma unroll
    for (int k = 0; k < UR_PER_LANE; ++k) acc[k] = 0.0f;
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
            accumulate_wave<decltype(width)::value, ur_group(decltype(width)::value), STREAM>(
                packed + (span.start >> 3), [&](int w) { return level_wave + static_cast<int64_t>(w) * packed_stride; },
                packed_stride, M, [] {}, [&](int w) { return lane_value(unit, w); }, span.n_lanes, acc, slots_of(lds_out, tid));
        });
    } else {
        // the lane's own tensor, fetched beside the table (lanes past the end: the first one's)
        const int32_t c = granule_cseg[(active ? P0 : span.start) >> 7];
        n_valid = cseg_valid_end[c] - P0;
        const dq_cseg_width e = widths[c];
        float* lds_unit = reinterpret_cast<float*>(lds_raw + UR_TILE * sizeof(float)) + (tid >> 6) * UR_WAVE_SEGS * M;
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
                accumulate_lane<decltype(width)::value>(packed + (P0 >> 3), level_ptr, packed_stride, M, unit_ptr, acc,
                                                        slots_of(lds_out, tid));
            });
        }
    }
    finish_tile<UPDATE, ONCE>(acc, active, n_valid, inv_M * ur_sum_scale(b), lds_out, tid, span.start, padded_elems, out, x, eta);
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
    const wave_span span = wave_span_of(tid, padded_elems, granule_cseg);
    if (span.n_lanes <= 0) return;
    const int64_t P0 = span.start + lane * UR_PER_LANE;
    const bool active = lane < span.n_lanes;
    const uint8_t* level_plane = packed + (padded_elems >> 3);

    float acc[UR_PER_LANE];
#pragma unroll
    for (int k = 0; k < UR_PER_LANE; ++k) acc[k] = 0.0f;
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
                accumulate_wave<decltype(width)::value, ur_group(decltype(width)::value), STREAM>(
                    packed + (span.start >> 3),
                    [&](int w) {
                        const uint64_t off = (static_cast<uint64_t>(__builtin_amdgcn_readlane(at_hi, w)) << 32) |
                                             static_cast<uint32_t>(__builtin_amdgcn_readlane(at_lo, w));
                        return level_plane + (static_cast<int64_t>(w) * packed_stride + static_cast<int64_t>(off));
                    },
                    packed_stride, M, [] {}, [&](int w) { return lane_value(unit, w); }, span.n_lanes, acc, slots_of(lds_out, tid));
            });
            // This route ends here.  Joined with the general one ahead of finish_tile, the kernel spilled 18 registers,
            // and the general one paid: widths mixed, 4.2 M ragged elements, M = 64 152 us before there were two routes,
            // 206 joined, 137 now; one width in buckets of 512, M = 8, b = 2 33, 42, 31; this route, ResNet-18 shape, M = 8, b = 4
            // 24.0 joined, 21.2 now.
            finish_tile<UPDATE, ONCE>(acc, active, n_valid, inv_M * ur_sum_scale(b), lds_out, tid, span.start, padded_elems, out, x, eta);
            return;
        }
    }

    // the lane's own tensor, fetched beside the table (lanes past the end: the first one's)
    const int32_t c = granule_cseg[(active ? P0 : span.start) >> 7];
    n_valid = cseg_valid_end[c] - P0;
    worker_entry* lds_entry = reinterpret_cast<worker_entry*>(lds_raw + UR_TILE * sizeof(float)) +
                              (tid >> 6) * UR_WAVE_SEGS * M; // [local seg][M]
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
        block_total total{ slots_of(lds_out, tid) }; // the block sums of accumulate_workers: same order of additions
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
    finish_tile<UPDATE, ONCE>(acc, active, n_valid, inv_M * UR_FP16_SCALE, lds_out, tid, span.start, padded_elems, out, x, eta);
}

// acc[k] += sgn_k * scale for a lane's 32 elements: the scale with its sign flipped where the bit is set.
// (Conversion routes were measured here too and the integer form stays: (sign << 7) | 0x38 as an 8-bit
// float 0.40 ms against 0.35 ms at D = 2^28, M = 16; (sign << 15) | 0x3C00 as the 16-bit operand of a
// mixed-precision FMA, which issues at half rate, 33.8 against 30.8 us on 4.2 M elements at M = 64.)
__device__ __forceinline__ void add_signed_scale(uint32_t sg, float scale, float (&acc)[UR_PER_LANE])
{
    const uint32_t unit = __float_as_uint(scale);
#pragma unroll
    for (int k = 0; k < UR_PER_LANE; ++k) acc[k] += __uint_as_float(unit ^ ((sg << (31 - k)) & 0x80000000u));
}

// The workers in ascending order, eight loads in flight.
template <typename Load, typename Scale>
__device__ __forceinline__ void accumulate_signs(int M, Load&& load, Scale&& scale, float (&acc)[UR_PER_LANE])
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
        for (int i = 0; i < G; ++i) add_signed_scale(sg[i], scale(w + i), acc);
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
__global__ __launch_bounds__(UR_THREADS) void k_sign_reduce_scaled(
    const uint8_t* __restrict__ packed, int64_t packed_stride, int M, const float* __restrict__ scales,
    int32_t n_seg, const int32_t* __restrict__ granule_cseg, const int32_t* __restrict__ cseg_seg,
    const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems, float inv_M, float* __restrict__ out)
{
    extern __shared__ __align__(16) uint8_t lds_raw[];
    float4* lds_out = reinterpret_cast<float4*>(lds_raw);

    const int tid = threadIdx.x, lane = tid & 63;
    const wave_span span = wave_span_of(tid, padded_elems, granule_cseg);
    const int64_t P0 = span.start + lane * UR_PER_LANE;
    const bool active = lane < span.n_lanes;

    // The scales first, then the messages, as at the narrow widths of the quantized average (ur_table_first).
    // Against the first loads ahead of the scales, in us: 2^24 values, M = 4, 8, 16 18.0, 21.1, 27.4 -> 16.8, 18.4,
    // 25.8; 2^28 x 16 340 -> 334; 2^24 values in tensors of 512, M = 8 21.8 -> 19.1; 2^24 x 64 68.5 -> 70.6.
    int64_t n_valid = 0;
    float* table = reinterpret_cast<float*>(lds_raw + UR_TILE * sizeof(float)) + (tid >> 6) * UR_WAVE_SEGS * M;
    const float* scale_ptr = nullptr;
    if (span.n_lanes > 0)
        scale_ptr = wave_table(span, lane, M, P0, granule_cseg, cseg_valid_end, table, n_valid, [&](int w, int32_t c) {
            return scales[static_cast<int64_t>(w) * n_seg + cseg_seg[c]];
        });
    __syncthreads();
    if (span.n_lanes <= 0) return; // the whole wavefront; there is no workgroup barrier below

    float acc[UR_PER_LANE];
#pragma unroll
    for (int k = 0; k < UR_PER_LANE; ++k) acc[k] = 0.0f;
    const uint8_t* sign_wave = packed + (span.start >> 3);
    const uint32_t at = (active ? lane : span.n_lanes - 1) * 4u;
    accumulate_signs(
        M,
        [&](int w) {
            return load_dwords<true, uint32_t>(scalar_address(sign_wave + static_cast<int64_t>(w) * packed_stride) + at);
        },
        [&](int w) { return scale_ptr[w]; }, acc);
    finish_tile<false>(acc, active, n_valid, inv_M, lds_out, tid, span.start, padded_elems, out, nullptr, 0.0f);
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
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * UR_TILE;
    const int64_t tile_end = tile0 + UR_TILE < padded_elems ? tile0 + UR_TILE : padded_elems;
    const int64_t P0 = tile0 + tid * UR_PER_LANE;
    const bool active = P0 < tile_end;

    float acc[UR_PER_LANE];
#pragma unroll
    for (int k = 0; k < UR_PER_LANE; ++k) acc[k] = 0.0f;
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
        for (int k = 0; k < UR_PER_LANE; ++k) {
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
    finish_tile<false>(acc, active, n_valid, MAJORITY ? 1.0f : inv_M, lds_out, tid, tile0 + (tid >> 6) * UR_WAVE_ELEMS,
                       padded_elems, out, nullptr, 0.0f);
}

constexpr size_t UR_LDS_THREE_PER_CU = 41 * 1024; // of 160 KiB

// Whether the level loads of widths 5 to 7 carry the streaming hint although several of them meet a cache line: with the
// update, where messages and model together are more than half of the last-level cache, so that the messages do not push the model
// out.  Measured over 1 to 270 M values, M = 1..31: the reduce alone, messages from memory, 16.8 M, M = 16 b = 5 65 -> 55 us, 20 M,
// M = 4 b = 7 44.5 -> 40.2; whole iterations (norm, quantize, reduce) 11.2 M, M = 16 b = 7 315 -> 303; below, where an iteration's
// messages are still in the cache, it costs (ResNet-18 shape, M = 8 28.8 -> 30.1).  Without update it gains 3 to 7 % of iterations with 200
// to 400 MB of messages and loses up to 9 % where they come from memory.  With more than 32 workers (three workgroups per CU, the
// vector ALU as much as the loads) it loses there too: 4.2 M ragged elements, M = 64 b = 5 56 -> 62, transformer shape, M = 62 b = 5 113 -> 128.
constexpr int64_t UR_LAST_LEVEL_CACHE = 256 << 20;
constexpr bool ur_may_stream(int b) { return b >= 5 && b <= 7; }
inline bool ur_stream(const dq_plan* plan, int M, int b)
{
    return ur_may_stream(b) && M <= 32 && M * dq_packed_bytes(plan, b) + plan->padded_elems * 4 > UR_LAST_LEVEL_CACHE / 2;
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

// Up to how many tiles the workers are divided over wavefronts (k_unpack_dequant_reduce_split), measured with update against
// the undivided kernel for M = 28..64, 64..600 tiles, all widths, messages in no cache and read before (time undivided / time
// divided).  Undivided, a tile is one wavefront on each SIMD of a CU: 128 tiles leave half of the chip idle (M = 32 b = 1 +7 % and
// +17, b = 5 +34 and +41; M = 64 +28 and +33, +52 and +60), and beyond 256 some CUs have two tiles and the others wait for them
// (M = 64 at 256 and 258 tiles b = 5 33.0 and 41.0 us against 29.2 and 35.5).  What the division costs (LDS, barriers, a row of units per
// wavefront) is most at b = 1, 4 and 8.  Inside the lines it gains up to 100 %.  Beyond them fresh messages lose, at some sizes all do:
// M = 28 at 192 tiles b = 1 3 %, M = 32 at 256 b = 7 5 %, M = 48 at 258 b = 4 2 and b = 8 12 %; M = 60 at 361 and 400 b = 2, 3, 5 3 to 4 %
// gained and 3 to 6 lost, M = 57 at 320 and 400 b = 6, 7 2 to 3 gained and 10 lost; at 514 and 600 b = 5 3 and 7 % lost (read before 9 and 2
// gained), b = 4 16 and 18.
inline int64_t ur_split_max_tiles(int b, int M)
{
    if (M > 56 && b != 1 && b != 4 && b != 8) return b <= 5 ? 380 : 320;
    if (M >= 40 && b >= 4 && b <= 7) return 256;
    if (M >= 32 && b >= 3) return 192;
    return M > 24 ? 128 : 0;
}
// Up to how many tiles a lane owns 8 elements (k_unpack_dequant_reduce_narrow), measured against the kernels above for
// M = 1..64, 0.5..768 tiles, all widths, with and without update (kernel trace).  4096 elements, M = 8, b = 8 with update
// 4.44 -> 3.32 us; 2^20, M = 4, b = 4 4.84 -> 4.24.  Inside the lines 0 to 60 % gained; beyond them its plain extraction
// of every level costs more than the idle lanes: M = 1 at 192 tiles 0 %, at 256 up to 9 % lost, M = 8 at 192 b = 1 7 %, 3.0 M ragged
// values, M = 5 b = 1 7 %; M = 32 b = 7 at 64 tiles 5 %, M = 64 b = 1 at any size 10 %.
inline int64_t ur_narrow_max_tiles(int b, int M)
{
    if (b == 8 && M >= 4) return 192;
    if (M <= 24) return 128;
    return M <= 40 && b != 3 && b != 7 ? 64 : 0;
}

template <int B>
int launch(const dq_plan* plan, const uint8_t* packed, int64_t packed_stride, int M, const float* norms,
           float* out, float* x, float eta, hipStream_t stream)
{
    const int64_t n_tiles = (plan->padded_elems + UR_TILE - 1) / UR_TILE;
    if (n_tiles > INT32_MAX) return DQ_ERR_INVALID_ARG;
    const float inv_M = 1.0f / static_cast<float>(M);
    if (n_tiles <= ur_narrow_max_tiles(B, M)) {
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
        const dim3 grid(static_cast<unsigned>((plan->padded_elems + UR_WAVE_ELEMS - 1) / UR_WAVE_ELEMS)), block(UR_THREADS);
        const size_t lds = UR_TILE * sizeof(float) + static_cast<size_t>(UR_MAX_LOCAL_SEG) * per_wave * UR_SUM_BLOCK * sizeof(float);
#define DQ_LAUNCH_SPLIT(UPDATE)                                                                                           \
    hipLaunchKernelGGL((k_unpack_dequant_reduce_split<B, UPDATE>), grid, block, lds, stream, packed, packed_stride, M,    \
                       per_wave, norms, plan->n_seg, plan->d_granule_cseg, plan->d_cseg_seg, plan->d_cseg_valid_end,       \
                       plan->padded_elems, inv_M, out, x, eta)
        if (x) DQ_LAUNCH_SPLIT(true);
        else DQ_LAUNCH_SPLIT(false);
#undef DQ_LAUNCH_SPLIT
        return hipGetLastError() == hipSuccess ? DQ_OK : DQ_ERR_HIP;
    }
    size_t lds_bytes = UR_TILE * sizeof(float) + static_cast<size_t>(UR_MAX_LOCAL_SEG) * M * sizeof(float);
    // Where thousands of tiles stream wide messages, three workgroups per CU move more than four.  Measured for
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
    if (x)
        ur_with_policy<ur_may_stream(B)>(ur_stream(plan, M, B), ur_model_once(plan), [&](auto s, auto once) {
            go(k_unpack_dequant_reduce<B, true, decltype(s)::value, decltype(once)::value>);
        });
    else
        go(k_unpack_dequant_reduce<B, false, false, false>);
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
    const int64_t n_tiles = (plan->padded_elems + UR_TILE - 1) / UR_TILE;
    if (n_tiles > INT32_MAX) return DQ_ERR_INVALID_ARG;
    // No fewer workgroups per CU here (as launch() has them for wide messages): the widths may be known to the GPU
    // only, and where it is b >= 5 that gains (1 to 4 % from 8192 tiles on), b = 2 loses (2 to 4 %) and so do small tensors
    // (16.8 M in buckets of 512, M = 16, b = 1 8 %).
    const size_t lds_bytes = UR_TILE * sizeof(float) + static_cast<size_t>(UR_MAX_LOCAL_SEG) * M * sizeof(float);
    const dim3 grid(static_cast<unsigned>(n_tiles)), block(UR_THREADS);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const float inv_M = 1.0f / static_cast<float>(M);
    const bool hint = ur_stream(plan, M, 6), once = ur_model_once(plan); // six bits stand for widths that the GPU may have set
    if (widths->n_workers != 1) {
        const size_t lds_w = UR_TILE * sizeof(float) + static_cast<size_t>(UR_MAX_LOCAL_SEG) * M * sizeof(worker_entry);
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
            ur_with_policy<true>(hint, once, [&](auto s, auto o) {
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
        hipLaunchKernelGGL(kernel, grid, block, lds_bytes, stream, packed_dev, packed_worker_stride_bytes, M, norms_dev, plan->n_seg,
                           plan->d_granule_cseg, plan->d_cseg_seg, plan->d_cseg_valid_end, widths->d_table, plan->padded_elems, inv_M,
                           out_dev, x_dev, eta);
    };
    if (x_dev)
        ur_with_policy<true>(hint, once, [&](auto s, auto o) {
            go(k_unpack_dequant_reduce_v<true, decltype(s)::value, decltype(o)::value>);
        });
    else
        go(k_unpack_dequant_reduce_v<false, false, false>);
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
    const int64_t n_tiles = (plan->padded_elems + UR_TILE - 1) / UR_TILE;
    if (n_tiles > INT32_MAX) return DQ_ERR_INVALID_ARG;
    const dim3 grid(static_cast<unsigned>(n_tiles)), block(UR_THREADS);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const float inv_M = 1.0f / static_cast<float>(M);
    const size_t tile_bytes = UR_TILE * sizeof(float);
    if (!majority && scales_dev) {
        const size_t lds_bytes = tile_bytes + static_cast<size_t>(UR_MAX_LOCAL_SEG) * M * sizeof(float);
        hipLaunchKernelGGL(k_sign_reduce_scaled, grid, block, lds_bytes, stream, packed_dev,
                           packed_worker_stride_bytes, M, scales_dev, plan->n_seg, plan->d_granule_cseg,
                           plan->d_cseg_seg, plan->d_cseg_valid_end, plan->padded_elems, inv_M, out_dev);
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
