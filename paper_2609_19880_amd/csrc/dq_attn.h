// Device helpers shared by the attention kernels over D-Quant records: LDS
// addressing, fp16 header words, level packing and the int8 matrix-core
// contractions with three-digit fixed-point operands.
#pragma once

#include "dq_common.h"

namespace dq {

__device__ __forceinline__ float half_lo(uint32_t w) { return half_bits_to_f32((uint16_t)(w & 0xFFFFu)); }
__device__ __forceinline__ float half_hi(uint32_t w) { return half_bits_to_f32((uint16_t)(w >> 16)); }

// LDS access through a plain byte offset (no symbol relocation in the address).
#define LDS_PTR(T, off) reinterpret_cast<__attribute__((address_space(3))) T*>((uintptr_t)(off))

// Levels of four consecutive steps (top bytes of the table words) as one word.
__device__ __forceinline__ uint32_t pack4(uint32_t e0, uint32_t e1, uint32_t e2, uint32_t e3) {
    const uint32_t lo = __builtin_amdgcn_perm(e1, e0, 0x0c0c0703u);
    const uint32_t hi = __builtin_amdgcn_perm(e3, e2, 0x07030c0cu);
    return lo | hi;
}

// Fixed-point range of the query and of the softmax weights, in three signed 8-bit
// digits: 2^22, so that the weights' unit and its reciprocal scale exactly (an
// error common to all channels shows in the output's channel 0, where the offsets'
// sum and the levels' sums nearly cancel).
constexpr float kDigitMax = 4194304.0f;

// Rotates one query head held as channels l and l + 64 in lane l
// (unnormalized Hadamard, stages h = 1, 2, ..., 64 in the order of the
// definition), multiplies it by scale (the softmax's, for exponents of 2, so that
// the scores come out as such) and stores it into qt[g][128] fp32, with qscale[g] =
// max |q_rot| / kDigitMax and qsum[g] = sum of q_rot.  rotate = 0: keys arrive in the rotated
// basis, and so does the query: it is taken as it is.  v0, v1 end as the
// rotated channels; returns qscale[g].
__device__ __forceinline__ float rotate_query_head(float& v0, float& v1, int g, int lane, float* qt, float* qscale,
                                                   float* qsum, int rotate, float scale) {
    if (rotate) {
        hadamard_lanes(v0, v1, lane);
        const float r0 = v0 + v1, r1 = v0 - v1;
        v0 = r0;
        v1 = r1;
    }
    v0 *= scale;
    v1 *= scale;
    qt[g * 128 + lane] = v0;
    qt[g * 128 + lane + 64] = v1;
    const float mx = wave_max_f32(fmaxf(fabsf(v0), fabsf(v1)));
    const float sm = wave_sum_f32(v0 + v1);
    const float qs = mx * (1.0f / kDigitMax);
    if (lane == 0) {
        qscale[g] = qs;
        qsum[g] = sm;
    }
    return qs;
}

// All query heads of a workgroup, a wavefront per head: heads 0 .. nh - 1 of
// q, and qscale = qsum = 0 for the slots nh .. slots - 1.
__device__ __forceinline__ void rotate_query_heads(const uint16_t* q, int nh, int slots, int wave, int nw,
                                                   int lane, float* qt, float* qscale, float* qsum,
                                                   int rotate, float scale) {
    for (int g = wave; g < slots; g += nw) {
        if (g >= nh) {
            if (lane == 0) {
                qscale[g] = 0.f;
                qsum[g] = 0.f;
            }
            continue;
        }
        float v0 = bf16_to_f32(q[g * 128 + lane]), v1 = bf16_to_f32(q[g * 128 + lane + 64]);
        rotate_query_head(v0, v1, g, lane, qt, qscale, qsum, rotate, scale);
    }
}

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

// v_mfma_i32_16x16x64_i8: 16 bytes of K per lane; A and B are loaded alike, so
// which K a byte stands for does not matter.
__device__ __forceinline__ v4i mfma64(const v4i& a, const v4i& b, const v4i& c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// ds_read_b64_tr_b8 at LDS byte address off.  Within each group of 16 lanes,
// lane 8 h + i receives byte i of the 8-byte rows that the group's lanes h,
// h + 2, ..., h + 14 address (in that order): token-major rows come back
// K-major, as the 16x16x32 products take them.
__device__ __forceinline__ uint64_t lds_tr8(uint32_t off) {
    typedef int v2i __attribute__((ext_vector_type(2)));
    const v2i r = __builtin_amdgcn_ds_read_tr8_b64_v2i32(LDS_PTR(v2i, off));
    return (uint64_t)(uint32_t)r.x | ((uint64_t)(uint32_t)r.y << 32);
}

// ---- a 64-token tile's scores, softmax and weighted values
//
// Work layout.  Lane l serves query-head slot l / 16 of a group of four and
// token 16 tg + l % 16 of each 16-token group tg: the rows of the 16x16x64
// products are (slot, digit) with a zero fourth digit, their columns tokens (q .
// k) or channels (P . v), so that a lane receives the three digit sums of its
// slot.  The running maximum, sums and corrections are then one per lane, and a
// tile's maximum is four values and four DPP steps inside the row of 16 lanes.
// (With v_mfma_i32_4x4x4_16b_i8 on the levels as they appear, a lane held all
// four slots of its token: 96 products per tile instead of 8, four times the
// reductions, and 32 reads of query digits.)
constexpr int kRowT = 80;                 // bytes per row of a level tile (64 channels, then 16 bytes of row padding)
constexpr int kRowHdr = 64;               // the padding holds the headers of the row's token (no LDS of their own: it
                                          // would cost wavefronts); 16 rows' headers fall in different banks
constexpr int kQRow = 64;                 // bytes per row of a query-digit tile
constexpr int kQTile = 16 * kQRow;        // query digits of a group's 16 rows, one 64-channel slice
constexpr int kColGroup = 16 * kRowT;     // 16 token rows of a level tile

// Digits of rotated query head g (values r0, r1 of channels lane, lane + 64, unit
// qs) into the tiles [group][slice][row 4 slot + digit][kQRow].  The 16-byte
// pieces of a row are exchanged (piece ^ slot), so that the 16 rows' pieces that
// are read together fall in different banks without padding.
__device__ __forceinline__ void query_digits(uint8_t* tiles, int g, int lane, float r0, float r1, float qs) {
#pragma unroll
    for (int sl = 0; sl < 2; ++sl) {
        int v = 0;
        if (qs > 0.f) {
            v = (int)rintf((sl ? r1 : r0) / qs);
            v = max(-4194304, min(4194304, v));
        }
        // adding 128 to every byte and flipping its top bit leaves the signed digits
        const uint32_t w = ((uint32_t)v + 0x00808080u) ^ 0x00808080u;
        uint8_t* dst = tiles + ((g / 4) * 2 + sl) * kQTile + 4 * (g % 4) * kQRow + (lane ^ (16 * (g % 4)));
        dst[0] = (uint8_t)w;
        dst[kQRow] = (uint8_t)(w >> 8);
        dst[2 * kQRow] = (uint8_t)(w >> 16);
        dst[3 * kQRow] = 0;
    }
}

// Sixteen dwords (64 channels) of the lane's levels into its row.
__device__ __forceinline__ void store_levels(uint32_t row, const uint32_t* lev) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *LDS_PTR(v4i, row + 16 * q) =
            v4i{(int)lev[4 * q], (int)lev[4 * q + 1], (int)lev[4 * q + 2], (int)lev[4 * q + 3]};
}

// The lane's operands: bytes 16 (l / 16) .. of row l % 16, of a level tile and of
// a query tile.
__device__ __forceinline__ uint32_t level_operand(int lane) { return (lane & 15) * kRowT + 16 * (lane >> 4); }
__device__ __forceinline__ uint32_t query_operand(int lane) {
    return (lane & 15) * kQRow + 16 * ((lane >> 4) ^ ((lane >> 2) & 3));
}

// d[hg][tg] += query digits . levels over one 64-channel slice (col, qa: the
// lane's operands in the level tile and in the slice's query tile of group 0).
template <int HG>
__device__ __forceinline__ void qk_slice(uint32_t col, uint32_t qa, v4i (&d)[HG][4]) {
    v4i b[4], a[HG];
#pragma unroll
    for (int tg = 0; tg < 4; ++tg) b[tg] = *LDS_PTR(v4i, col + tg * kColGroup);
#pragma unroll
    for (int hg = 0; hg < HG; ++hg) a[hg] = *LDS_PTR(v4i, qa + hg * 2 * kQTile);
#pragma unroll
    for (int hg = 0; hg < HG; ++hg)
#pragma unroll
        for (int tg = 0; tg < 4; ++tg) d[hg][tg] = mfma64(a[hg], b[tg], d[hg][tg]);
}

// Maximum over each row of 16 lanes, in every lane of the row, of non-NaN
// floats (wait states as in wave_max_f32).
__device__ __forceinline__ float row_max16(float v) {
    asm("s_nop 4\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1"
        : "+v"(v));
    return v;
}
__device__ __forceinline__ float row_sum16(float v) {
    v += dpp0<0xB1, 0xF>(v);
    v += dpp0<0x4E, 0xF>(v);
    v += dpp0<0x141, 0xF>(v);
    return v + dpp0<0x140, 0xF>(v);
}

// The digit sums of a slot and token or channel as one number (each below 2^20 in
// magnitude, so the upper two meet exactly in int32).
__device__ __forceinline__ float digit_sum(const v4i& d) {
    return fmaf((float)((d[2] << 8) + d[1]), 256.0f, (float)d[0]);
}

constexpr float kLowest = -3.4028234663852886e38f;

// Softmax of the lane's four tokens for its slot (Eq. fold-key), the value scale
// folded into the weights (Eq. fold-value).
//   d: digit sums; h[tg]: scale and offset of the token's key and value, in fp32
//   or as the records' first words; qs, qsum, qm: the slot's digit unit, query sum and
//   q . mu, all with the softmax's scale in them, so that a score is an exponent of 2
//   (a scale that enters with the subtraction of the rounded maximum, as one fused
//   multiply-add, leaves the maximum itself an exponent of half a unit in the last
//   place: more than the range for scores beyond 2^30);
//   left: tokens from l % 16 to the sequence's end (token 16 tg is live while
//   16 tg < left); m: running maximum.
// Returns the correction of what was summed before; psum, osum: the lane's
// parts of sum p and sum p o_v; w: the weights' digits (fixed point relative to
// the tile's largest), wscale their unit.
struct SlotWeights {
    float corr, psum, osum, wscale;
    uint32_t w[4];
};
__device__ __forceinline__ float key_scale(const float4& h) { return h.x; }
__device__ __forceinline__ float key_offset(const float4& h) { return h.y; }
__device__ __forceinline__ float value_scale(const float4& h) { return h.z; }
__device__ __forceinline__ float value_offset(const float4& h) { return h.w; }
__device__ __forceinline__ float key_scale(const uint2& h) { return half_lo(h.x); }
__device__ __forceinline__ float key_offset(const uint2& h) { return half_hi(h.x); }
__device__ __forceinline__ float value_scale(const uint2& h) { return half_lo(h.y); }
__device__ __forceinline__ float value_offset(const uint2& h) { return half_hi(h.y); }

template <typename H>
__device__ __forceinline__ SlotWeights slot_softmax(const v4i (&d)[4], const H (&h)[4], float qs, float qsum,
                                                    float qm, int left, bool whole, float& m) {
    float s[4];
#pragma unroll
    for (int tg = 0; tg < 4; ++tg) {
        const float dot = digit_sum(d[tg]) * qs;
        s[tg] = fmaf(key_scale(h[tg]), dot, fmaf(key_offset(h[tg]), qsum, qm));
    }
    if (!whole) {
#pragma unroll
        for (int tg = 0; tg < 4; ++tg) s[tg] = 16 * tg < left ? s[tg] : -INFINITY;
    }
    SlotWeights r;
    const float mn = fmaxf(m, row_max16(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))));
    const float base = fmaxf(mn, kLowest);           // -inf - base stays -inf
    // v_exp_f32 directly: arguments are <= 0 and results that would be denormal
    // may flush to zero
    r.corr = __builtin_amdgcn_exp2f(m - base);
    m = mn;
    float p[4], pw[4];
#pragma unroll
    for (int tg = 0; tg < 4; ++tg) {
        p[tg] = __builtin_amdgcn_exp2f(s[tg] - base);
        pw[tg] = p[tg] * value_scale(h[tg]);           // >= 0: scales are non-negative
    }
    r.psum = (p[0] + p[1]) + (p[2] + p[3]);
    r.osum = 0.f;
#pragma unroll
    for (int tg = 0; tg < 4; ++tg) r.osum = fmaf(value_offset(h[tg]), p[tg], r.osum);
    const float top = fmaxf(row_max16(fmaxf(fmaxf(pw[0], pw[1]), fmaxf(pw[2], pw[3]))), 1e-30f);
    const float inv = kDigitMax * __builtin_amdgcn_rcpf(top);
    r.wscale = top * (1.0f / kDigitMax);
#pragma unroll
    for (int tg = 0; tg < 4; ++tg) {
        // 2^23 + v has v in its low bits, rounded to nearest even; the reciprocal
        // is good to 2^-23, so v ends at most one above 2^22
        const uint32_t v = __float_as_uint(fmaf(pw[tg], inv, 8388608.0f)) - 0x4B000000u;
        r.w[tg] = (v + 0x00808080u) ^ 0x00808080u;
    }
    return r;
}

// The lane's four weight words to byte 4 slot of their token rows (16 bytes
// each); at: tile + 16 (l % 16) + 4 (l / 16).
__device__ __forceinline__ void store_weights(uint32_t at, const uint32_t (&w)[4]) {
#pragma unroll
    for (int tg = 0; tg < 4; ++tg) *LDS_PTR(uint32_t, at + tg * 256) = w[tg];
}

// Weights of a tile as the A operand (rows (slot, digit), K = 64 tokens).
__device__ __forceinline__ v4i load_weights(uint32_t a_lane) {
    const uint64_t lo = lds_tr8(a_lane), hi = lds_tr8(a_lane + 32 * 16);
    return v4i{(int)(uint32_t)lo, (int)(uint32_t)(lo >> 32), (int)(uint32_t)hi, (int)(uint32_t)(hi >> 32)};
}
// 16 channels of the value tile as the B operand.
__device__ __forceinline__ v4i load_values(uint32_t b_lane) {
    const uint64_t lo = lds_tr8(b_lane), hi = lds_tr8(b_lane + 32 * kRowT);
    return v4i{(int)(uint32_t)lo, (int)(uint32_t)(lo >> 32), (int)(uint32_t)hi, (int)(uint32_t)(hi >> 32)};
}
}  // namespace dq
