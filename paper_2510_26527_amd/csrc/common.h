// Shared device helpers for the gfx950 kernels: bf16 conversion, wavefront (64-lane)
// reductions, MFMA operand types.  Host code includes it only for the typedefs.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace psd {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;   // one MFMA A/B operand (8 k-values)
typedef __attribute__((ext_vector_type(4))) float f32x4;     // 16x16 MFMA accumulator
typedef __attribute__((ext_vector_type(16))) float f32x16;   // 32x32 MFMA accumulator
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;  // a 16-byte load

typedef __attribute__((ext_vector_type(8))) float f32x8;

constexpr int kWave = 64;

// An fp32 activation as a pair of bf16 values hi + lo (hi = RNE(x), lo = RNE(x - hi)): fed to
// two MFMAs it carries ~16 mantissa bits through the bf16 matrix cores.
__device__ __forceinline__ void split_bf16(const f32x8 &x, bf16x8 *hi, bf16x8 *lo) {
    const bf16x8 h = __builtin_convertvector(x, bf16x8);
    *hi = h;
    *lo = __builtin_convertvector(x - __builtin_convertvector(h, f32x8), bf16x8);
}
__device__ __forceinline__ f32x8 load_f32x8(const float *p) {
    const f32x4 a = *reinterpret_cast<const f32x4 *>(p);
    const f32x4 b = *reinterpret_cast<const f32x4 *>(p + 4);
    return f32x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
}

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// round-to-nearest-even fp32 -> bf16 bit pattern (NaN stays NaN)
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
}

// Operand order: the activations of a pass of up to 16 rows as the matrix cores take them, so that a wavefront reads the
// operand of 32 k in whole 1 KB pieces instead of 16 bytes out of every line of every row.  K is cut into steps of 128
// and these into quarters: quarter q of a step holds k = (q >> 1) * 64 + g * 16 + (q & 1) * 8 + e of lane group g, e < 8, the
// order in which the packed weights are stored.  A quarter is two fragments of 64 lanes x 8 bf16, the high parts hi = RNE(x) and
// the remainders lo = RNE(x - hi), lane = 16 g + row; or, folded (up to 8 rows), one fragment whose lanes 16 g + row and
// 16 g + 8 + row hold both.

__device__ __forceinline__ size_t op_at(int m, int k, bool folded) {          // element index of the high part of x[m][k]
    const int quarter = (k >> 7) * 4 + ((k >> 6) & 1) * 2 + ((k >> 3) & 1);
    return (size_t)quarter * (folded ? 512 : 1024) + ((k >> 4) & 3) * 128 + m * 8 + (k & 7);
}
__device__ __forceinline__ int op_lo(bool folded) { return folded ? 64 : 512; }       // from there to the remainder
__device__ __forceinline__ void op_store(uint16_t *op, int m, int k, bool folded, float x) {
    const uint32_t hi = f32_to_bf16_bits(x);
    uint16_t *p = op + op_at(m, k, folded);
    p[0] = (uint16_t)hi;
    p[op_lo(folded)] = (uint16_t)f32_to_bf16_bits(x - bf16_bits_to_f32(hi));
}
// x[m][k .. k + 3], k a multiple of 4
__device__ __forceinline__ void op_store4(uint16_t *op, int m, int k, bool folded, f32x4 x) {
    const uint32_t h01 = pack_bf16x2(x[0], x[1]), h23 = pack_bf16x2(x[2], x[3]);
    uint16_t *p = op + op_at(m, k, folded);
    *reinterpret_cast<uint2 *>(p) = make_uint2(h01, h23);
    *reinterpret_cast<uint2 *>(p + op_lo(folded)) =
        make_uint2(pack_bf16x2(x[0] - __uint_as_float(h01 << 16), x[1] - __uint_as_float(h01 & 0xffff0000u)),
                   pack_bf16x2(x[2] - __uint_as_float(h23 << 16), x[3] - __uint_as_float(h23 & 0xffff0000u)));
}

// round-to-nearest-even fp32 -> fp16 bit pattern
__device__ __forceinline__ uint16_t f32_to_f16_bits(float f) {
    const _Float16 h = (_Float16)f;
    return __builtin_bit_cast(uint16_t, h);
}

// element loads / stores by storage type
__device__ __forceinline__ float load_elem(const float *p, size_t i) { return p[i]; }
__device__ __forceinline__ float load_elem(const uint16_t *p, size_t i) { return bf16_bits_to_f32(p[i]); }
__device__ __forceinline__ void store_elem(float *p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void store_elem(uint16_t *p, size_t i, float v) { p[i] = (uint16_t)f32_to_bf16_bits(v); }

typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

// 8 bf16 (as stored) -> 8 fp16, exact for every value the fp16 grid holds
__device__ __forceinline__ u32x4 bf16x8_to_f16x8(u32x4 w) {
    u32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const auto h = __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w[e] << 16), __uint_as_float(w[e] & 0xffff0000u));
        r[e] = __builtin_bit_cast(uint32_t, h);
    }
    return r;
}
// 8 fp32 -> 8 fp16, round to nearest even
__device__ __forceinline__ u32x4 f32x8_to_f16x8(const f32x8 &x) {
    const f16x8 h = __builtin_convertvector(x, f16x8);
    return __builtin_bit_cast(u32x4, h);
}

template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        T other = __shfl_xor(v, o, kWave);
        v = other > v ? other : v;
    }
    return v;
}
// butterfly sum: every lane ends with the same value, summed in a fixed tree order
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// fp64 wavefront reductions on the vector ALU's own lane moves (about a tenth of the latency of a trip through the LDS
// crossbar per step).  Inclusive prefix over the lanes in a fixed order: rows of 16 first, then across rows; lanes that a
// move does not reach get `none`.
template <int N>
struct Int { static constexpr int value = N; };
template <int CTRL, int ROWS>
__device__ __forceinline__ double lane_move(double v, double none) {
    const uint64_t x = __builtin_bit_cast(uint64_t, v), o = __builtin_bit_cast(uint64_t, none);
    const uint32_t lo = __builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)x, CTRL, ROWS, 0xf, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(o >> 32), (int)(uint32_t)(x >> 32), CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <typename F>
__device__ __forceinline__ double wave_scan_d(double v, double none, F op) {
    v = op(v, lane_move<0x111, 0xf>(v, none));             // row_shr:1, 2, 4, 8
    v = op(v, lane_move<0x112, 0xf>(v, none));
    v = op(v, lane_move<0x114, 0xf>(v, none));
    v = op(v, lane_move<0x118, 0xf>(v, none));
    v = op(v, lane_move<0x142, 0xa>(v, none));             // row_bcast:15 into rows 1 and 3
    v = op(v, lane_move<0x143, 0xc>(v, none));             // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ double lane_value_d(double v, int lane) {        // the same lane for the whole wavefront
    const uint64_t x = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)x, lane), hi = __builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// the largest value of the wavefront (NaN counts for nothing)
__device__ __forceinline__ float wave_top_f(float v) {
    auto step = [&](auto ctrl, auto rows) {
        v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(-INFINITY), __float_as_int(v), decltype(ctrl)::value,
                                                                decltype(rows)::value, 0xf, false)));
    };
    step(Int<0x111>{}, Int<0xf>{});                        // row_shr:1, 2, 4, 8, then row_bcast:15 and :31
    step(Int<0x112>{}, Int<0xf>{});
    step(Int<0x114>{}, Int<0xf>{});
    step(Int<0x118>{}, Int<0xf>{});
    step(Int<0x142>{}, Int<0xa>{});
    step(Int<0x143>{}, Int<0xc>{});
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ double wave_prefix_sum_d(double v) { return wave_scan_d(v, 0.0, [](double a, double b) { return a + b; }); }
__device__ __forceinline__ double wave_total_d(double v) { return lane_value_d(wave_prefix_sum_d(v), 63); }

}  // namespace psd
