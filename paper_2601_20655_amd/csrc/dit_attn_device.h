// Device helpers shared by the gfx950 kernels: 16-bit operand packing, MFMA wrappers,
// input widening and the 3-axis rotary rotation of eight consecutive channels.
#pragma once
#include "dit_attn_internal.h"

namespace dit {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4 mk4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) {
    u32x4 r = {x, y, z, w};
    return r;
}

// Two fp32 values -> one dword of two 16-bit operands, round to nearest even (low half = a).
template <int OP>
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    f32x2 f = {a, b};
    if constexpr (OP == OP_F16) {
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, f16x2));
    } else {
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
    }
}

// acc + lo + hi of one packed operand pair, summed in fp32 (one v_dot2c against (1, 1)).  Used for bf16
// probabilities only: the instruction does not overlap with a running MFMA.
template <int OP>
__device__ __forceinline__ float sum2(uint32_t packed, float acc) {
    if constexpr (OP == OP_F16) {
        const f16x2 one = {(_Float16)1.0f, (_Float16)1.0f};
        return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, packed), one, acc, false);
    } else {
        const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, packed), one, acc, false);
    }
}

// Two fp32 values -> one dword of two fp16 operands, SATURATING: a value beyond the largest finite fp16 number
// becomes +-65504 instead of an infinity that would turn the products into NaN (bf16 inputs can hold such values).
// NaN stays NaN (the IEEE minimum / maximum pass it on).  Clamped as a pair behind the conversion, two instructions
// a pair: rounding first gives the same numbers (whatever rounds past 65504 is clamped to it), and comparing and
// selecting the fp32 values took eight.
__device__ __forceinline__ uint32_t pack2_sat_f16(float a, float b) {
    const f32x2 f = {a, b};
    const f16x2 top = {(_Float16)65504.0f, (_Float16)65504.0f};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_maximum(
                                            __builtin_elementwise_minimum(__builtin_convertvector(f, f16x2), top), -top));
}

// Eight fp32 values -> four dwords of 16-bit operands, saturating for fp16.  Used where q', k' and v are
// rounded (prologue, pre-pack pass), never in the key loop: probabilities cannot overflow.
template <int OP>
__device__ __forceinline__ u32x4 pack8(const float x[8]) {
    if constexpr (OP == OP_F16) {
        return mk4(pack2_sat_f16(x[0], x[1]), pack2_sat_f16(x[2], x[3]), pack2_sat_f16(x[4], x[5]),
                   pack2_sat_f16(x[6], x[7]));
    } else {
        return mk4(pack2<OP>(x[0], x[1]), pack2<OP>(x[2], x[3]), pack2<OP>(x[4], x[5]), pack2<OP>(x[6], x[7]));
    }
}

// D(32x32, fp32) += A(32x16) * B(16x32).  Lane l supplies row (l % 32) of A and column
// (l % 32) of B, eight contraction indices each (group l / 32); it receives column (l % 32)
// of D, rows 8*(r/4) + 4*(l/32) + r%4 for r = 0..15.
template <int OP>
__device__ __forceinline__ f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c) {
    if constexpr (OP == OP_F16) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    } else {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
}

// ---- 8-bit (OCP e4m3) score operands ----
typedef int i32x8 __attribute__((ext_vector_type(8)));

// Exponent e such that amax * 2^e lies in [128, 256), inside e4m3's normal range (largest finite
// value 448); 0 for an all-zero row.  Clamped so that 127 - e stays a valid 8-bit scale code.
__device__ __forceinline__ int fp8_row_exponent(float amax) {
    const int be = (int)((__float_as_uint(amax) >> 23) & 255u);  // amax in [2^(be-127), 2^(be-126))
    if (be == 0) return 0;
    const int e = 134 - be;
    return e > 100 ? 100 : (e < -100 ? -100 : e);
}
__device__ __forceinline__ float pow2i(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }

// Eight fp32 values -> eight e4m3 bytes (round to nearest even), byte i = x[i].
__device__ __forceinline__ uint2 pack8_fp8(const float x[8]) {
    int lo = __builtin_amdgcn_cvt_pk_fp8_f32(x[0], x[1], 0, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(x[2], x[3], lo, true);
    int hi = __builtin_amdgcn_cvt_pk_fp8_f32(x[4], x[5], 0, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(x[6], x[7], hi, true);
    return make_uint2((uint32_t)lo, (uint32_t)hi);
}

// 16x16x32 form of the same instructions (half the issue time per instruction, same flops per cycle): lane
// 16 g + i supplies, for both operands, row i and contraction indices 8g .. 8g+7; result: column i, rows 4g .. 4g+3.
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int OP>
__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
    if constexpr (OP == OP_F16) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                      0);
    } else {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                       0, 0);
    }
}

// D(32x32, fp32) += 2^(sa-127) A(32x64, e4m3) * 2^(sb-127) B(64x32, e4m3).  Lane l supplies 32
// contraction indices of row (l % 32) of A and of column (l % 32) of B, the same 32 indices on
// both sides (group l / 32); sa and sb are the lane's own 8-bit scale codes for that row resp.
// column, and the two lanes of a row must carry the same code.  Result layout as mfma32.
__device__ __forceinline__ f32x16 mfma32_fp8(i32x8 a, i32x8 b, f32x16 c, int sa, int sb) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, sa, 0, sb);
}

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

__device__ __forceinline__ void widen8(u32x4 u, float x[8]) {
    x[0] = bf16_lo(u.x); x[1] = bf16_hi(u.x);
    x[2] = bf16_lo(u.y); x[3] = bf16_hi(u.y);
    x[4] = bf16_lo(u.z); x[5] = bf16_hi(u.z);
    x[6] = bf16_lo(u.w); x[7] = bf16_hi(u.w);
}

// Eight consecutive channels starting at element offset `off` (a multiple of 8) as fp32.
__device__ __forceinline__ void load8(const void* base, int64_t off, int in_f32, float x[8]) {
    if (in_f32) {
        const float4* p = reinterpret_cast<const float4*>(static_cast<const float*>(base) + off);
        float4 lo = p[0], hi = p[1];
        x[0] = lo.x; x[1] = lo.y; x[2] = lo.z; x[3] = lo.w;
        x[4] = hi.x; x[5] = hi.y; x[6] = hi.z; x[7] = hi.w;
    } else {
        widen8(*reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(base) + off), x);
    }
}

// Multiplier 1/sqrt(mean(x^2) + eps) of one q row.  The row's D channels are read by the lane
// pair (lane, lane ^ 32), lane half `half` taking chunks 2*ks + half; `base` is the element
// offset of the row's head, `stat` the row's index in the per-token table (mode 2).
template <int D>
__device__ __forceinline__ float q_row_rstd(const NormArgs& n, const void* q, int64_t base, int in_f32, int half,
                                            int64_t stat) {
    if (n.mode == 2) return n.rstd[stat];
    float ss = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        float x[8];
        load8(q, base + 8 * (2 * ks + half), in_f32, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) ss = fmaf(x[e], x[e], ss);
    }
    ss += __shfl_xor(ss, 32);
    return 1.0f / sqrtf(ss * (1.0f / D) + n.eps);
}

// x[0..8) = channels [8c, 8c+8) of head h: times the row multiplier and the channel weights
__device__ __forceinline__ void norm8(float x[8], const NormArgs& n, float rs, int h, int D, int c) {
    if (n.gamma) {
        const float4* g = reinterpret_cast<const float4*>(n.gamma + (int64_t)h * D + 8 * c);
        const float4 g0 = g[0], g1 = g[1];
        x[0] *= rs * g0.x; x[1] *= rs * g0.y; x[2] *= rs * g0.z; x[3] *= rs * g0.w;
        x[4] *= rs * g1.x; x[5] *= rs * g1.y; x[6] *= rs * g1.z; x[7] *= rs * g1.w;
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] *= rs;
    }
}

// angle = position * base^(-2i/d_a), d_a = 2 * hd.  base^x = 2^(x log2(base)), the exponent in two parts (log2(base)
// is, and the product's rounding is kept): as exact as pow() for every base and position that is accepted, and it and
// the joint sine and cosine are a third of the dependent fp64 instructions of pow(), cos() and sin() -- a table is a
// few hundred to a few thousand entries, so the time is a launch and one thread's latency: 2.8 -> 2.4 us for 212
// entries. (In one part the error of the power grows with |x log2(base)|: base 1e-10 at positions 3 to 7 gave four
// times the error that the last bits of the power and of the product with the position allow.)
__device__ __forceinline__ float2 rope_entry(const TableArgs& a, int idx) {
    int ax = 0;
    if (idx >= a.rg.off[2]) ax = 2;
    else if (idx >= a.rg.off[1]) ax = 1;
    const int local = idx - a.rg.off[ax];
    const int hd = a.rg.hd[ax];
    const int p = local / hd, i = local - p * hd;
    const double x = -(double)i / (double)hd;
    const double t = x * a.log2_base, rest = fma(x, a.log2_base, -t) + x * a.log2_base_lo;
    const double y = exp2(t);
    const double phi = (double)(a.origin[ax] + p) * fma(y, rest * 0.6931471805599453, y);
    double sn, cs;
    sincos(phi, &sn, &cs);
    return make_float2((float)cs, (float)sn);
}

// Token index -> position indices along (t, h, w), counted from the grid origin.
__device__ __forceinline__ void token_pos(int n, const RopeGeom& rg, int& pt, int& ph, int& pw) {
    const int hw = rg.Hg * rg.Wg;
    pt = n / hw;
    const int rem = n - pt * hw;
    ph = rem / rg.Wg;
    pw = rem - ph * rg.Wg;
}

// A pair (x0, x1) becomes (x0 cos - x1 sin, x1 cos + x0 sin); all in fp32.  Which product is rounded by itself is stated and
// not left to the compiler, whose choice differs from kernel to kernel: rows that the projection's epilogue rotates are
// to have the bits of those that the pre-pack rotates.
__device__ __forceinline__ float2 rotate_pair(float x0, float x1, float2 cs) {
    return make_float2(__builtin_fmaf(x0, cs.x, -(x1 * cs.y)), __builtin_fmaf(x1, cs.x, x0 * cs.y));
}

// Rotate channels [8c, 8c+8) = pairs 4c..4c+3 of a token at position indices (pt, ph, pw).
__device__ __forceinline__ void rope8(float x[8], int c, const RopeGeom& rg, const float2* tab,
                                      int pt, int ph, int pw) {
#pragma unroll
    for (int pp = 0; pp < 4; ++pp) {
        const int ip = 4 * c + pp;
        int idx;
        if (ip < rg.hd[0]) {
            idx = rg.off[0] + pt * rg.hd[0] + ip;
        } else if (ip < rg.hd[0] + rg.hd[1]) {
            idx = rg.off[1] + ph * rg.hd[1] + (ip - rg.hd[0]);
        } else {
            idx = rg.off[2] + pw * rg.hd[2] + (ip - rg.hd[0] - rg.hd[1]);
        }
        const float2 y = rotate_pair(x[2 * pp], x[2 * pp + 1], tab[idx]);
        x[2 * pp] = y.x;
        x[2 * pp + 1] = y.y;
    }
}

// The same in two stages, for code that requests the entries of several rows before it uses the first: two pairs a load
// (a load of scattered entries costs the address unit some thirty clocks whatever its width).
struct RopeRow {
    int b[3];  // axis a's table row at the token's position, less the axis's first pair: entry of pair i = tab[b[a] + i]
};

__device__ __forceinline__ RopeRow rope_row(const RopeGeom& rg, int pt, int ph, int pw) {
    RopeRow r;
    r.b[0] = rg.off[0] + pt * rg.hd[0];
    r.b[1] = rg.off[1] + ph * rg.hd[1] - rg.hd[0];
    r.b[2] = rg.off[2] + pw * rg.hd[2] - rg.hd[0] - rg.hd[1];
    return r;
}

__device__ __forceinline__ float2 rope_one(const float2* tab, const RopeGeom& rg, const RopeRow& r, int ip) {
    return tab[(uint32_t)((ip < rg.hd[0] ? r.b[0] : ip < rg.hd[0] + rg.hd[1] ? r.b[1] : r.b[2]) + ip)];
}

typedef float f32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));

// Entries of pairs ip, ip + 1 (ip even) as if both were of ip's axis.  Where they are not (an axis ends behind an odd
// number of pairs) the second one is whatever stands behind the row -- the next position's or the next axis's row, which
// has entries or ip + 1 would be past the last pair -- and rope_mend puts the right one there.
__device__ __forceinline__ void rope_two(const float2* tab, const RopeGeom& rg, const RopeRow& r, int ip, float2 cs[2]) {
    const int b = ip < rg.hd[0] ? r.b[0] : ip < rg.hd[0] + rg.hd[1] ? r.b[1] : r.b[2];
    const f32x4_a8 e = *reinterpret_cast<const f32x4_a8*>(tab + (uint32_t)(b + ip));
    cs[0] = make_float2(e[0], e[1]);
    cs[1] = make_float2(e[2], e[3]);
}

// Entries of the pairs that the second and third axis begin with, where those numbers are odd.
__device__ __forceinline__ void rope_edges(const float2* tab, const RopeGeom& rg, const RopeRow& r, float2 edge[2]) {
    const int h0 = rg.hd[0], h01 = rg.hd[0] + rg.hd[1];
    edge[0] = edge[1] = make_float2(1.f, 0.f);
    if (h0 & 1) edge[0] = tab[(uint32_t)((h0 < h01 ? r.b[1] : r.b[2]) + h0)];
    if (h01 & 1) edge[1] = tab[(uint32_t)(r.b[2] + h01)];
}

__device__ __forceinline__ void rope_mend(const RopeGeom& rg, const float2 edge[2], int ip, float2 cs[2]) {
    if (ip + 1 == rg.hd[0]) cs[1] = edge[0];
    if (ip + 1 == rg.hd[0] + rg.hd[1]) cs[1] = edge[1];
}

}  // namespace dit
