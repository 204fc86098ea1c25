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

// Writes the low B bytes of v at dst (LDS, byte offset a multiple of B): even widths in pieces of 8, 4 and 2 bytes, which
// LDS takes at any byte address (the compiler checks that the target does), odd ones byte by byte: their pieces would lie
// at odd addresses, where a store takes longer than the bytes.  Pieces at odd widths against bytes, norms and messages in one
// pass, 16.8 M values in buckets of 512, M = 8: b = 3 126.6 -> 120.1 us, b = 7 134.3 -> 128.6; bracketed b = 5 168.4 -> 159.3; 64
// buckets, M = 2, b = 3 3.98 -> 3.76.  At b = 6 4 + 2 bytes against 2 + 2 + 2 124.2 against 126.6.
template <int B>
__device__ __forceinline__ void stage_bytes(uint8_t* dst, uint64_t v)
{
    if constexpr (B % 2 != 0) {
#pragma unroll
        for (int k = 0; k < B; ++k) dst[k] = static_cast<uint8_t>(v >> (8 * k));
    } else if constexpr (B == 8) {
        __builtin_memcpy(dst, &v, 8);
    } else {
        if constexpr ((B & 4) != 0) {
            const uint32_t piece = static_cast<uint32_t>(v);
            __builtin_memcpy(dst, &piece, 4);
        }
        if constexpr ((B & 2) != 0) {
            const uint16_t piece = static_cast<uint16_t>(v >> (8 * (B & 4)));
            __builtin_memcpy(dst + (B & 4), &piece, 2);
        }
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

// ---------------------------------------------------------------------------------------------
// Two quads (four consecutive elements each, one Philox block) of a lane.  Per element, with
// a = min(|g| * scale, s) in binary32 and u = (word >> 8) * 2^-24, the level of Eq. (5)-(6) is
// floor(a) + [u < a - floor(a)], which is the integer ceil(a - u): inside an integer interval of a the
// difference is above floor(a) exactly when u < a - floor(a), and never above floor(a) + 1 or at most floor(a) - 1.
// Rounding towards +infinity keeps the ceiling of a difference that binary32 cannot hold (no integer lies between
// the exact value and its rounding), and adding 1.5 * 2^23 in that mode takes the ceiling itself.  So with the
// mode set, fma(-(word >> 8), 2^-24, a) and one addition per element give the level in the low bits of a sum that
// also holds the levels packed before it (times 2^b by one exact fma).
//
// What bounds it: vector issue, where the norms are computed in the same pass; the plain pass is bound by memory.  Per
// element and beside the 9.3 instructions of Philox, 6.4 are issued: multiply, half a max3, shift, convert, fma, fma and
// addition (a quad's first needs no fma), half a sign (see quantize_exchange); with minimum (and the canonicalising maximum ahead of it), v_fract, two
// conversions, compare, add with carry and shift they were 12.5, and 8.5 in a form for wavefronts whose products are all
// below 1.  Fma and addition also issue twice as fast as those (2.4 against 4.3 cycles by themselves, less of a
// difference in a mixture).  Norms and messages in one pass, 16.8 M values in buckets of 512, M = 8, no input in a cache: b = 2
// (products below 1) 122.5 -> 117.6 us, b = 3 128.8 -> 120.1, b = 4 138.1 -> 118.9, b = 7 144.8 -> 128.6, b = 8 140.8 -> 121.6.
// The smallest calls pay for it at b = 1 and 2: one chunk, norms given, 2.3 -> 2.4 us.
// ---------------------------------------------------------------------------------------------

// s|g|/N of the lane's eight elements, one rounding each, and what the wavefront can conclude from the largest:
enum qp_range {
    QP_ALL_ZERO, // every product of the wavefront is +0 (exact-zero stretches, unusable norm): every level is 0
                 // whatever the random numbers, and none are drawn
    QP_BELOW_S,  // none above s: min(a, s) = a
    QP_CLAMP     // something above s, or a NaN
};
template <int B>
__device__ __forceinline__ qp_range quantize_products(const float4 x0, const float4 x1, const float scale, const float S_arg,
                                                      float (&a)[8])
{
    const float S = B > 0 ? static_cast<float>((1 << (B > 0 ? B : 1)) - 1) : S_arg;
    const float v[8] = { x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w };
    uint32_t n[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        a[k] = fabsf(v[k]) * scale;
        n[k] = __float_as_uint(a[k]); // never negative, so the patterns are in the values' order, a NaN above all
    }
    const uint32_t top = max(max(max(max(n[0], n[1]), n[2]), max(max(n[3], n[4]), n[5])), max(n[6], n[7]));
    if (__all(top == 0u)) return QP_ALL_ZERO;
    return __all(top <= __float_as_uint(S)) ? QP_BELOW_S : QP_CLAMP;
}

// min(a, s): a caller's norm may be too small, and |g|/N may round above 1.  A NaN goes to s, and an unusable norm
// (scale 0) to 0 whatever the elements are.
template <int B>
__device__ __forceinline__ void quantize_clamp(float (&a)[8], const float scale, const float S_arg)
{
    const float S = B > 0 ? static_cast<float>((1 << (B > 0 ? B : 1)) - 1) : S_arg;
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] = scale > 0.0f ? fminf(a[k], S) : 0.0f;
}

// word >> 8 of the two quads' random words, as binary32 (exact).
__device__ __forceinline__ void quantize_random(const uint32_t quad0, const uint32_t quad1, const uint32_t quad_hi,
                                                const uint32_t worker, const uint32_t step, const uint32_t key0,
                                                const uint32_t key1, float (&t)[8])
{
    uint32_t r[2][4];
    dq_philox4x32_10(quad0, quad_hi, worker, step, key0, key1, r[0]);
    dq_philox4x32_10(quad1, quad_hi, worker, step, key0, key1, r[1]);
#pragma unroll
    for (int k = 0; k < 8; ++k) t[k] = static_cast<float>(r[k >> 2][k & 3] >> 8);
}

// The two quads' levels, four fields of b bits each in the low 4 b bits of lv[h], from the clamped products and the random numbers.  Above
// the fields lv holds what the sum leaves there (B = 1 to 5; zero otherwise): whoever takes the fields masks them or drops the rest.
// The rounding mode is set and put back inside the one asm statement, so no other operation runs under it.
// Results are marked as written early: without that an operand still to be read may be given the register of a result
// that has the same value to begin with.
// b <= 5: a quad's 20 bits fit the sum's 22; above, pairs are summed and joined.  b: the width, where B = 0.
template <int B>
__device__ __forceinline__ void quantize_levels(const float (&a)[8], const float (&t)[8], const int b, uint32_t (&lv)[2])
{
    constexpr uint32_t MAGIC = 0x4B400000u; // 1.5 * 2^23: sums from here on are whole numbers, and the pattern counts them
    float c[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) c[k] = a[k];
    const float pw = B > 0 ? static_cast<float>(1 << B) : __uint_as_float(static_cast<uint32_t>(127 + b) << 23);
    const float back = 0x1.8p23f - 0x1.8p23f * pw; // y -> y * pw + back keeps 1.5 * 2^23 and multiplies the rest; exact
    if constexpr (B >= 1 && B <= 5) {
        asm("s_nop 1\n\t"
            "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 1\n\t"
            "v_fma_f32 %3, -%11, %16, %3\n\t"
            "v_fma_f32 %7, -%15, %16, %7\n\t"
            "v_fma_f32 %2, -%10, %16, %2\n\t"
            "v_fma_f32 %6, -%14, %16, %6\n\t"
            "v_add_f32 %3, %17, %3\n\t"
            "v_add_f32 %7, %17, %7\n\t"
            "v_fma_f32 %1, -%9, %16, %1\n\t"
            "v_fma_f32 %5, -%13, %16, %5\n\t"
            "v_fma_f32 %3, %3, %18, %19\n\t"
            "v_fma_f32 %7, %7, %18, %19\n\t"
            "v_fma_f32 %0, -%8, %16, %0\n\t"
            "v_fma_f32 %4, -%12, %16, %4\n\t"
            "v_add_f32 %3, %3, %2\n\t"
            "v_add_f32 %7, %7, %6\n\t"
            "v_fma_f32 %3, %3, %18, %19\n\t"
            "v_fma_f32 %7, %7, %18, %19\n\t"
            "v_add_f32 %3, %3, %1\n\t"
            "v_add_f32 %7, %7, %5\n\t"
            "v_fma_f32 %3, %3, %18, %19\n\t"
            "v_fma_f32 %7, %7, %18, %19\n\t"
            "v_add_f32 %3, %3, %0\n\t"
            "v_add_f32 %7, %7, %4\n\t"
            "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 0"
            : "+&v"(c[0]), "+&v"(c[1]), "+&v"(c[2]), "+&v"(c[3]), "+&v"(c[4]), "+&v"(c[5]), "+&v"(c[6]), "+&v"(c[7])
            : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]), "v"(t[6]), "v"(t[7]), "s"(0x1p-24f),
              "s"(0x1.8p23f), "s"(pw), "v"(back));
        lv[0] = __float_as_uint(c[3]);
        lv[1] = __float_as_uint(c[7]);
    } else {
        asm("s_nop 1\n\t"
            "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 1\n\t"
            "v_fma_f32 %1, -%9, %16, %1\n\t"
            "v_fma_f32 %3, -%11, %16, %3\n\t"
            "v_fma_f32 %5, -%13, %16, %5\n\t"
            "v_fma_f32 %7, -%15, %16, %7\n\t"
            "v_fma_f32 %0, -%8, %16, %0\n\t"
            "v_fma_f32 %2, -%10, %16, %2\n\t"
            "v_fma_f32 %4, -%12, %16, %4\n\t"
            "v_fma_f32 %6, -%14, %16, %6\n\t"
            "v_add_f32 %1, %17, %1\n\t"
            "v_add_f32 %3, %17, %3\n\t"
            "v_add_f32 %5, %17, %5\n\t"
            "v_add_f32 %7, %17, %7\n\t"
            "v_fma_f32 %1, %1, %18, %19\n\t"
            "v_fma_f32 %3, %3, %18, %19\n\t"
            "v_fma_f32 %5, %5, %18, %19\n\t"
            "v_fma_f32 %7, %7, %18, %19\n\t"
            "v_add_f32 %1, %1, %0\n\t"
            "v_add_f32 %3, %3, %2\n\t"
            "v_add_f32 %5, %5, %4\n\t"
            "v_add_f32 %7, %7, %6\n\t"
            "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 0"
            : "+&v"(c[0]), "+&v"(c[1]), "+&v"(c[2]), "+&v"(c[3]), "+&v"(c[4]), "+&v"(c[5]), "+&v"(c[6]), "+&v"(c[7])
            : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]), "v"(t[6]), "v"(t[7]), "s"(0x1p-24f),
              "s"(0x1.8p23f), "v"(pw), "v"(back));
        // (hi << 2b) + lo, less what the two patterns carry
        const int two = 2 * (B > 0 ? B : b);
        const uint32_t excess = (MAGIC << two) + MAGIC;
        lv[0] = (__float_as_uint(c[3]) << two) + __float_as_uint(c[1]) - excess;
        lv[1] = (__float_as_uint(c[7]) << two) + __float_as_uint(c[5]) - excess;
    }
}

// w moved up by four bits and a quad's sign bits below it (element 0 in bit 0): one instruction an element.
__device__ __forceinline__ uint32_t quantize_signs_below(uint32_t w, const float4 x)
{
    w = __builtin_amdgcn_alignbit(w, __float_as_uint(x.w), 31);
    w = __builtin_amdgcn_alignbit(w, __float_as_uint(x.z), 31);
    w = __builtin_amdgcn_alignbit(w, __float_as_uint(x.y), 31);
    return __builtin_amdgcn_alignbit(w, __float_as_uint(x.x), 31);
}
// the sign byte of a lane's eight consecutive elements
__device__ __forceinline__ uint32_t quantize_sign_byte(const float4 x0, const float4 x1)
{
    return quantize_signs_below(quantize_signs_below(0u, x1), x0);
}
// the fields of a quad, four of b bits
template <int B>
__device__ __forceinline__ constexpr uint32_t quad_fields(int b)
{
    return static_cast<uint32_t>((static_cast<uint64_t>(1) << (4 * (B > 0 ? B : b))) - 1u);
}

// Both quads: the levels.  The random numbers are left in t for a caller that
// quantizes the same elements again (QP_ALL_ZERO: none were drawn, every level is 0 for any smaller scale too).
template <int B>
__device__ __forceinline__ qp_range quantize_quads(const float4 x0, const float4 x1, const float scale, const float S,
                                                   const int b, const uint32_t quad0, const uint32_t quad1,
                                                   const uint32_t quad_hi, const uint32_t worker, const uint32_t step,
                                                   const uint32_t key0, const uint32_t key1, uint32_t (&lv)[2],
                                                   float (&t)[8])
{
    float a[8];
    lv[0] = lv[1] = 0u;
    const qp_range range = quantize_products<B>(x0, x1, scale, S, a);
    if (range != QP_ALL_ZERO) {
        quantize_random(quad0, quad1, quad_hi, worker, step, key0, key1, t);
        if (range == QP_CLAMP) quantize_clamp<B>(a, scale, S);
        quantize_levels<B>(a, t, b, lv);
    }
    return range;
}

// The same elements' levels with a smaller scale, for the random numbers and the range quantize_quads gave.
template <int B>
__device__ __forceinline__ void quantize_again(const qp_range range, const float4 x0, const float4 x1, const float scale,
                                               const float S, const int b, const float (&t)[8], uint32_t (&lv)[2])
{
    float a[8] = { fabsf(x0.x) * scale, fabsf(x0.y) * scale, fabsf(x0.z) * scale, fabsf(x0.w) * scale,
                   fabsf(x1.x) * scale, fabsf(x1.y) * scale, fabsf(x1.z) * scale, fabsf(x1.w) * scale };
    if (range == QP_CLAMP) quantize_clamp<B>(a, scale, S);
    quantize_levels<B>(a, t, b, lv);
}

// A lane's eight consecutive elements (Philox counters quad, quad + 1): the sign byte (element 0 in bit 0)
// and the 8*B level bits (element 0 in the low B bits).
// S, b: the level count and bits of the tensor (template argument B > 0 fixes them at compile time).
template <int B>
__device__ __forceinline__ qp_range quantize8(const float4 x_lo, const float4 x_hi, const float scale, const float S,
                                              const int b, const uint32_t quad, const uint32_t quad_hi,
                                              const uint32_t worker, const uint32_t step, const uint32_t key0,
                                              const uint32_t key1, uint32_t& sign, uint64_t& level, float (&t)[8])
{
    uint32_t lv[2];
    const qp_range range = quantize_quads<B>(x_lo, x_hi, scale, S, b, quad, quad + 1u, quad_hi, worker, step, key0, key1, lv, t);
    sign = quantize_sign_byte(x_lo, x_hi);
    level = static_cast<uint64_t>(lv[0] & quad_fields<B>(b)) | (static_cast<uint64_t>(lv[1] & quad_fields<B>(b)) << (4 * (B > 0 ? B : b)));
    return range;
}

// The codes of the two quads x0 and x1 that a lane loaded (dq_load_wave_tile, not arranged) change places between the halves of
// the wavefront, so that the lane has its eight consecutive elements' sign byte (in the low eight bits of `sign`) and level bits (in
// the low 8 b bits of `level`).  Up to seven bits the signs travel below the levels in one word: with a word of signs made by masks and
// merged above the levels, a tile took 8 instructions more: with that and what dq_row_sums_of_two saves, norms and messages in one pass, 16.8 M values in
// buckets of 4096, M = 8, b = 5 with the reduce 149.2 -> 143.3 us; of 512, b = 2 132.4 -> 128.9; bracketed 2^26, M = 16, b = 4 1053 -> 1039.
template <int B>
__device__ __forceinline__ void quantize_exchange(const float4 x0, const float4 x1, const uint32_t (&lv)[2], const int b,
                                                  uint32_t& sign, uint64_t& level)
{
    if constexpr (B >= 1 && B <= 7) {
        const auto w = __builtin_amdgcn_permlane32_swap(quantize_signs_below(lv[0], x0), quantize_signs_below(lv[1], x1), false, false);
        sign = __builtin_amdgcn_bitop3_b32(0xFu, w[0], w[1] << 4, 0xCA); // a ? b : c, bit by bit
        level = static_cast<uint64_t>((w[0] >> 4) & quad_fields<B>(B)) | (static_cast<uint64_t>((w[1] >> 4) & quad_fields<B>(B)) << (4 * B));
    } else {
        const auto s = __builtin_amdgcn_permlane32_swap(quantize_signs_below(0u, x0), quantize_signs_below(0u, x1), false, false);
        const auto l = __builtin_amdgcn_permlane32_swap(lv[0], lv[1], false, false);
        sign = s[0] | (s[1] << 4);
        level = static_cast<uint64_t>(l[0]) | (static_cast<uint64_t>(l[1]) << (4 * (B > 0 ? B : b)));
    }
}

// quantize8 for a wavefront's tile as dq_load_wave_tile loaded it (not arranged) when one scale serves
// the whole tile: every lane quantizes the two quads it loaded, and the codes change places instead of
// the values -- one or two swaps in place of eight.  quad_tile: the tile's first quad.
template <int B>
__device__ __forceinline__ void quantize_wave_tile(const float4 lo, const float4 hi, const float scale, const float S,
                                                   const int b, const uint32_t quad_tile, const uint32_t lane,
                                                   const uint32_t quad_hi, const uint32_t worker, const uint32_t step,
                                                   const uint32_t key0, const uint32_t key1, uint32_t& sign, uint64_t& level)
{
    uint32_t lv[2];
    float t[8];
    const uint32_t quad = quad_tile + (lane & 31u) * 2u + (lane >> 5);
    quantize_quads<B>(lo, hi, scale, S, b, quad, quad + 64u, quad_hi, worker, step, key0, key1, lv, t);
    quantize_exchange<B>(lo, hi, lv, b, sign, level);
}

// threadIdx.x for the body of a loop over chunks: what follows from it is not worked out ahead of the loop and held in
// registers (k_bracket_settle_redo 82 to 98 -> 66 to 72).
__device__ __forceinline__ uint32_t qp_tid_in_loop()
{
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid;
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
// past the end of a ragged last chunk get zeros; what they compute is never stored.
template <int TILES>
__device__ __forceinline__ void qp_load(const float* __restrict__ g, uint32_t tid, uint32_t n_elems, float4 (&x)[TILES][2])
{
    const __amdgpu_buffer_rsrc_t buffer = dq_elems_buffer(g, n_elems);
#pragma unroll
    for (int it = 0; it < TILES; ++it)
        dq_load_wave_tile(buffer, (tid >> 6) * (QP_WAVE_TILE * TILES) + it * QP_WAVE_TILE, tid & 63u, x[it][0], x[it][1]);
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

// A wavefront's staged bytes [0, bytes) (a multiple of 16) leave as 16-byte stores; dst is the same for the whole wavefront.
// KEEP: through to the last-level cache (dq_store_buffer); otherwise with the streaming hint.
template <bool KEEP = false>
__device__ __forceinline__ void qp_store_wave(uint8_t* __restrict__ dst, const uint8_t* src, uint32_t bytes, uint32_t lane)
{
    const uint4* f = reinterpret_cast<const uint4*>(src);
    if constexpr (KEEP) {
        const __amdgpu_buffer_rsrc_t buffer = dq_bytes_buffer(dst, bytes);
        for (uint32_t i = lane; i < bytes / 16; i += 64) dq_store_buffer<false>(buffer, i * 16u, f[i]);
    } else {
        uint4* d = reinterpret_cast<uint4*>(dst);
        for (uint32_t i = lane; i < bytes / 16; i += 64) dq_store_stream(d + i, f[i]);
    }
}

// The workgroup's staged bytes [0, bytes) (a multiple of 16), after a barrier.  The lanes are counted from the start of
// the cache line that holds the first byte, so that no line is shared by two store instructions.
template <bool KEEP = false>
__device__ __forceinline__ void qp_store_block(uint8_t* __restrict__ dst, const uint8_t* src, uint32_t bytes, uint32_t tid)
{
    const uint4* f = reinterpret_cast<const uint4*>(src);
    const uint32_t skew = (static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst)) & 127u) >> 4;
    if constexpr (KEEP) {
        const __amdgpu_buffer_rsrc_t buffer = dq_bytes_buffer(dst, bytes);
        for (uint32_t i = tid; i < bytes / 16 + skew; i += QP_THREADS)
            if (i >= skew) dq_store_buffer<false>(buffer, (i - skew) * 16u, f[i - skew]);
    } else {
        uint4* d = reinterpret_cast<uint4*>(dst);
        for (uint32_t i = tid; i < bytes / 16 + skew; i += QP_THREADS)
            if (i >= skew) dq_store_stream(d + (i - skew), f[i - skew]);
    }
}

// Whether a chunk's two stretches of the message start on cache lines; each wavefront's part then does too (its tiles
// give a multiple of 128 bytes of either plane).  Where they don't -- the planes follow one another at multiples of 16
// bytes only --, wavefronts that store for themselves write two parts of a line each, and the memory
// pays for every part: the workgroup stores together there.  2^26 + 12345 values, M = 16, b = 7 950 -> 933 us, 2^28 - 1000,
// b = 4 3518 -> 3467, bracketed ResNet-18 shape, M = 8, b = 3 92.9 -> 89.8.
__device__ __forceinline__ bool qp_on_lines(const uint8_t* sign, const uint8_t* level)
{
    return ((reinterpret_cast<uintptr_t>(sign) | reinterpret_cast<uintptr_t>(level)) & 127u) == 0;
}

// The chunk's staged bytes leave: by wavefronts (each after its own staging) or together after a barrier (see qp_on_lines),
// so all of the workgroup has to come here.
// n_elems: the chunk's elements; sign and level: where its stretches start; b: its width.
template <bool KEEP = false>
__device__ __forceinline__ void qp_store_chunk(uint8_t* sign, uint8_t* level, const uint8_t* lds_sign, const uint8_t* lds_level,
                                               uint32_t n_elems, uint32_t wave0, uint32_t b, uint32_t tid)
{
    if (qp_on_lines(sign, level)) {
        dq_wave_sync();
        if (wave0 < n_elems) {
            const uint32_t n_wave = n_elems - wave0 < QP_WAVE_TILE * QP_TILES ? n_elems - wave0 : QP_WAVE_TILE * QP_TILES;
            qp_store_wave<KEEP>(sign + (wave0 >> 3), lds_sign + (wave0 >> 3), n_wave >> 3, tid & 63u);
            qp_store_wave<KEEP>(level + (wave0 >> 3) * b, lds_level + (wave0 >> 3) * b, (n_wave >> 3) * b, tid & 63u);
        }
    } else {
        __syncthreads();
        qp_store_block<KEEP>(sign, lds_sign, n_elems >> 3, tid);
        qp_store_block<KEEP>(level, lds_level, (n_elems >> 3) * b, tid);
    }
}

// The norm of a chunk's tensor (segment seg) for one worker: at[seg] of what the caller gave.  A kernel that works norms out
// itself has a form of its own (k_bracket_settle_redo).
struct qp_norm_given {
    __device__ __forceinline__ float operator()(const float* row, int32_t seg) const { return row[seg]; }
};

// What bounds it: the memory system's rate at 4 bytes read to (B+1)/8 written (about 6.1-6.2 TB/s, what a
// kernel with the same accesses and no arithmetic reaches), with the vector ALU at 89 % beside it (b = 4).  A chunk
// that lies in one tensor (nearly all of a gradient of large tensors) takes the first route: two scalar
// loads and one division per wavefront in place of the granule table, LDS and a barrier, and the codes
// change places between the lanes instead of the values.  Measured at D = 2^28, M = 16 against the table
// route alone: b = 2 3.36 -> 3.06 ms (6.1 TB/s), b = 4 3.39 -> 3.28 ms; ResNet-18 shape, M = 8, b = 2
// 74.9 -> 66.9 us.  Chunks that hold a tensor's end or several tensors take the table.
// NORM != 0: WHOLE = with the route for buckets.
// WHOLE = false, NORM = 0: no such route, and the lanes' elements as qp_load_block has them, for layouts with
// few chunks of one tensor (dq_plan::many_whole).  Measured there against the form with the route, in us: 5.4 M
// values in tensors of 128, M = 8 b = 4 38.0 -> 36.6, 16.8 M in tensors of 512, M = 8 b = 6 121.8 -> 114.8 and, with a
// widths table, b = 7 130.9 -> 122.4; 30.7 M in tensors of 1000, M = 4 b = 6 112.0 -> 104.5.
//
// KEEP: the message's stores go through to the last-level cache (qp_keep_messages).
// tid: threadIdx.x, or qp_tid_in_loop() where a workgroup takes several chunks.
// NORM = 0: the norms are an input.  NORM = 1 (l2) or 2 (max): chunk-local plans only; the kernel
// computes the norms of its chunk's tensors itself, writes them to norms_out and quantizes from
// the registers it already holds -- one read of the gradient instead of two.
template <int B, int TILES, int NORM, bool WHOLE = true, bool KEEP = false, typename NormOf = qp_norm_given>
__device__ __forceinline__ void quantize_pack_chunk(
    const float* __restrict__ grads, int64_t worker_stride, const float* __restrict__ norms, int32_t n_seg,
    const dq_chunk_tensor* __restrict__ chunk_tensor, const int32_t* __restrict__ granule_cseg,
    const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_valid_end, int64_t padded_elems,
    uint32_t key0, uint32_t key1, uint32_t step, uint32_t worker_base, uint8_t* __restrict__ packed,
    int64_t packed_stride, float* __restrict__ norms_out, uint32_t chunk_index, uint32_t tid = threadIdx.x, NormOf norm_of = {},
    dq_buckets buckets = {})
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
        const float N = norm_of(norms + static_cast<int64_t>(w) * n_seg, whole.seg); // issued whatever cseg is: one wait less
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
            qp_store_chunk<KEEP>(msg + (chunk0 >> 3), msg + (padded_elems >> 3) + (chunk0 >> 3) * B, lds_sign, lds_level, CHUNK, wave0,
                           B, tid);
            return;
        }
    }

    // Buckets that a wavefront holds whole: no tables, and each wavefront goes its own way (one barrier, and only where the chunk's stretches are off the
    // cache lines) in place of three barriers with two lookups ahead of the first.  16.8 M values, M = 8 with the reduce, buckets of 128, 256, 512, 1024,
    // b = 8 158 -> 152, 156 -> 151, 156 -> 151, 155 -> 151 us; 4 M, M = 3, b = 5 24.9 -> 22.4.  A root and a division for every wavefront are
    // what it costs; buckets of 2048 and 4096 lie in several wavefronts and take the tables.
    if constexpr (NORM != 0 && WHOLE) {
        if (chunk_index < buckets.chunks) {
            __shared__ double lds_bucket[DQ_CHUNK_GRANULES];
            const uint32_t lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
            for (int it = 0; it < TILES; ++it) dq_arrange_wave_tile(x[it][0], x[it][1]);
            const float N = dq_wave_bucket_norms<NORM == 2>(x, static_cast<int>(lane), lds_bucket + wave * 8, buckets.log);
            const float scale_of = N >= DQ_MIN_NORM ? S / N : 0.0f;
            if (lane < 8u && (lane & ((1u << buckets.log) - 1u)) == 0)
                norms_out[static_cast<int64_t>(w) * n_seg + (((chunk0 >> 7) + wave * 8 + lane) >> buckets.log)] = N;
#pragma unroll
            for (int it = 0; it < TILES; ++it) {
                const uint32_t tile0 = wave0 + it * QP_WAVE_TILE, at = (tile0 >> 3) + lane;
                const float scale = __shfl(scale_of, it * 4 + (lane >> 4), 64);
                uint32_t sign;
                uint64_t level;
                float t[8];
                quantize8<B>(x[it][0], x[it][1], scale, 0.0f, 0, quad_lo0 + (tile0 >> 2) + 2u * lane, quad_hi, worker, step, key0, key1,
                             sign, level, t);
                lds_sign[at] = static_cast<uint8_t>(sign);
                stage_bytes<B>(&lds_level[at * B], level);
            }
            qp_store_chunk<KEEP>(msg + (chunk0 >> 3), msg + (padded_elems >> 3) + (chunk0 >> 3) * B, lds_sign, lds_level, CHUNK, wave0,
                                 B, tid);
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
            const float N = norm_of(norms + static_cast<int64_t>(w) * n_seg, cseg_seg[seg_first + tid]);
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
        __shared__ int32_t lds_seg[MAX_LOCAL_SEG]; // fetched with the tables: a load where the norm is written is waited for
        if (static_cast<int32_t>(tid) <= seg_last - seg_first) {
            const int64_t rel = cseg_valid_end[seg_first + tid] - chunk0;
            lds_seg[tid] = cseg_seg[seg_first + tid];
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
                                                 lds_scale[j] = N >= DQ_MIN_NORM ? S / N : 0.0f;
                                                 norms_out[static_cast<int64_t>(w) * n_seg + lds_seg[j]] = N;
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
            float t[8];
            quantize8<B>(x[it][0], x[it][1], scale, 0.0f, 0, quad, quad_hi, worker, step, key0, key1, sign, level, t);
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
        qp_store_block<KEEP>(msg + (chunk0 >> 3), lds_sign, n_elems >> 3, tid);
        qp_store_block<KEEP>(msg + (padded_elems >> 3) + (chunk0 >> 3) * B, lds_level, (n_elems >> 3) * B, tid);
        return;
    }
    // 16-byte stores; every plane of a wavefront's stretch is a whole number of 16-byte pieces because it holds a
    // multiple of 128 elements
    qp_store_chunk<KEEP>(msg + (chunk0 >> 3), msg + (padded_elems >> 3) + (chunk0 >> 3) * B, lds_sign, lds_level, n_elems, wave0,
                              B, tid);
}

// ---------------------------------------------------------------------------------------------
// Per-tensor widths.  Same work split; b, the level count and the place of the level bytes come
// from the widths table per segment instead of the template argument.  A wavefront's level bytes are
// still one contiguous stretch of the message (every segment's stretch is a whole number of
// 16-byte pieces per granule), so they are staged and stored the same way.
// ---------------------------------------------------------------------------------------------
template <int TILES, int NORM, bool WHOLE = true, bool KEEP = false, typename NormOf = qp_norm_given> // as in quantize_pack_chunk
__device__ __forceinline__ void quantize_pack_chunk_v(
    const float* __restrict__ grads, int64_t worker_stride, const float* __restrict__ norms, int32_t n_seg,
    const dq_chunk_tensor* __restrict__ chunk_tensor, const int32_t* __restrict__ granule_cseg,
    const int32_t* __restrict__ cseg_seg, const int64_t* __restrict__ cseg_valid_end,
    const dq_cseg_width* __restrict__ widths_table, int32_t widths_worker_stride, int64_t padded_elems,
    uint32_t key0, uint32_t key1, uint32_t step, uint32_t worker_base, uint8_t* __restrict__ packed,
    int64_t packed_stride, float* __restrict__ norms_out, uint32_t chunk_index, uint32_t tid = threadIdx.x, NormOf norm_of = {})
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
    __shared__ int32_t lds_seg[NORM == 0 ? 1 : MAX_LOCAL_SEG]; // as in quantize_pack_chunk
    __shared__ int32_t lds_level_base[MAX_LOCAL_SEG]; // byte offset, in the chunk's level bytes, the
                                                      // segment's fields would have at chunk element 0
    __shared__ int32_t lds_valid_end[MAX_LOCAL_SEG];
    __shared__ __align__(16) uint8_t lds_sign[TILES * QP_THREADS];
    __shared__ __align__(16) uint8_t lds_level[TILES * QP_THREADS * 8];

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
        const float N = norm_of(norms + static_cast<int64_t>(w) * n_seg, whole.seg);
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
            qp_store_chunk<KEEP>(msg + (chunk0 >> 3), msg + (padded_elems >> 3) + e.level_start + ((chunk0 - e.seg_start) >> 3) * e.b,
                           lds_sign, lds_level, CHUNK, wave0, e.b, tid);
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
        const int32_t own_seg = cseg_seg[seg_first + tid];
        if constexpr (NORM == 0) {
            const float N = norm_of(norms + static_cast<int64_t>(w) * n_seg, own_seg);
            lds_scale[tid] = N >= DQ_MIN_NORM ? S / N : 0.0f;
        } else {
            lds_seg[tid] = own_seg;
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
                                                 lds_scale[j] = N >= DQ_MIN_NORM ? lds_levels[j] / N : 0.0f;
                                                 norms_out[static_cast<int64_t>(w) * n_seg + lds_seg[j]] = N;
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
            uint32_t sign;
            uint64_t level;
            float t[8];
            quantize8<0>(x[it][0], x[it][1], scale, S, b, quad, quad_hi, worker, step, key0, key1, sign, level, t);
            if (n_valid < QP_PER_LANE) {
                const int nv = n_valid > 0 ? n_valid : 0;
                sign &= (1u << nv) - 1u;
                level &= (static_cast<uint64_t>(1) << (nv * b)) - 1u;
            }
            lds_sign[e >> 3] = static_cast<uint8_t>(sign);
            // b bytes at an offset that is a multiple of b past a 16-byte boundary (every tensor's
            // stretch of a chunk starts on one); stage_bytes takes any
            stage_bytes_v(&lds_level[lds_level_base[local] + static_cast<int32_t>(e >> 3) * b], level, b);
        }
    }
    __syncthreads();
    const int last = seg_last - seg_first;
    qp_store_block<KEEP>(msg + (chunk0 >> 3), lds_sign, n_elems >> 3, tid);
    qp_store_block<KEEP>(msg + (padded_elems >> 3) + chunk_level0, lds_level,
                              static_cast<uint32_t>(lds_level_base[last]) + (n_elems >> 3) * lds_b[last], tid);
}

} // namespace
