// Device-side building blocks shared by the encode and decode kernels (gfx950, wave64).
#ifndef OCTOPUS_DEVICE_HPP_
#define OCTOPUS_DEVICE_HPP_

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <type_traits>

#include "octopus_internal.h"

namespace octopus {

constexpr int kWave = 64;
constexpr float kEps = 1e-20f;  // clamp of both divisors in Alg. 1

constexpr int cx_gcd(int a, int b) { return b == 0 ? a : cx_gcd(b, a % b); }
constexpr int cx_stream_bytes(int n, int b) {
    return (n <= 0 || b <= 0) ? 0 : ((n + 8 / cx_gcd(b, 8) - 1) / (8 / cx_gcd(b, 8))) * ((8 / cx_gcd(b, 8)) * b / 8);
}

// Compile-time image of octopus_plan_t.  BD1 == 0 means a single class.
template <int D_, int BD0_, int BN0_, int BD1_ = 0, int BN1_ = 0>
struct PlanT {
    static constexpr int D = D_;
    static constexpr int NTRI = (D + 2) / 3;
    static constexpr int NCLASS = BD1_ > 0 ? 2 : 1;
    static constexpr int NT0 = NCLASS == 2 ? (NTRI + 1) / 2 : NTRI;
    static constexpr int NT1 = NTRI - NT0;
    static constexpr int BD0 = BD0_, BN0 = BN0_, BD1 = BD1_, BN1 = BN1_;
    static constexpr int DIR0_BYTES = cx_stream_bytes(2 * NT0, BD0);
    static constexpr int DIR1_BYTES = cx_stream_bytes(2 * NT1, BD1);
    static constexpr int NRM0_BYTES = cx_stream_bytes(NT0, BN0);
    static constexpr int NRM1_BYTES = cx_stream_bytes(NT1, BN1);
    // bit offsets of the streams from the start of the record (gamma occupies bits 0..31)
    static constexpr int DIR0_BIT = 32;
    static constexpr int DIR1_BIT = DIR0_BIT + 8 * DIR0_BYTES;
    static constexpr int NRM0_BIT = DIR1_BIT + 8 * DIR1_BYTES;
    static constexpr int NRM1_BIT = NRM0_BIT + 8 * NRM0_BYTES;
    static constexpr int RECORD_BYTES = 4 + DIR0_BYTES + DIR1_BYTES + NRM0_BYTES + NRM1_BYTES;
    static constexpr int GRANULES = (RECORD_BYTES + 15) / 16;
    static constexpr int NWORDS = GRANULES * 4;
    static constexpr int QS = (3 * NTRI + 3) & ~3;  // floats per rotated query row
    static constexpr int LUT0 = 1 << (2 * BD0);     // direction LUT entries per class
    static constexpr int LUT1 = NCLASS == 2 ? 1 << (2 * BD1) : 0;

    // per-triplet constants
    static constexpr int cls(int i) { return i < NT0 ? 0 : 1; }
    static constexpr int bdir(int i) { return cls(i) ? BD1 : BD0; }
    static constexpr int bnrm(int i) { return cls(i) ? BN1 : BN0; }
    static constexpr int dir_bit(int i) { return cls(i) ? DIR1_BIT + (i - NT0) * 2 * BD1 : DIR0_BIT + i * 2 * BD0; }
    static constexpr int nrm_bit(int i) { return cls(i) ? NRM1_BIT + (i - NT0) * BN1 : NRM0_BIT + i * BN0; }

    static bool matches(const octopus_plan_t &p) {
        if (p.head_dim != D || p.n_class != NCLASS) return false;
        if (p.b_dir[0] != BD0 || p.b_nrm[0] != BN0 || p.class_ntri[0] != NT0) return false;
        if (NCLASS == 2 && (p.b_dir[1] != BD1 || p.b_nrm[1] != BN1 || p.class_ntri[1] != NT1)) return false;
        return p.record_bytes == RECORD_BYTES && p.granules == GRANULES;
    }
};

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// NBITS-wide field at compile-time bit position BITPOS of a record held in 32-bit words.
template <int BITPOS, int NBITS, int NW>
__device__ __forceinline__ uint32_t field(const uint32_t (&w)[NW]) {
    constexpr int wi = BITPOS >> 5, sh = BITPOS & 31;
    constexpr uint32_t mask = (1u << NBITS) - 1u;
    if constexpr (sh + NBITS <= 32) {
        return (w[wi] >> sh) & mask;
    } else {
        static_assert(wi + 1 < NW, "field runs past the record");
        return ((w[wi] >> sh) | (w[wi + 1] << (32 - sh))) & mask;
    }
}

// Same for a field whose upper bits may lie past the last word of the record (they read as zero).
template <int BITPOS, int NBITS, int NW>
__device__ __forceinline__ uint32_t field_clamped(const uint32_t (&w)[NW]) {
    constexpr int wi = BITPOS >> 5, sh = BITPOS & 31;
    constexpr uint32_t mask = (1u << NBITS) - 1u;
    if constexpr (sh + NBITS <= 32 || wi + 1 >= NW) {
        return (w[wi] >> sh) & mask;
    } else {
        return ((w[wi] >> sh) | (w[wi + 1] << (32 - sh))) & mask;
    }
}

// Eq. (oct-decode): unit vector of a point of the square, sign(0) = +1.
__device__ __forceinline__ float4 oct_decode(float xi, float eta) {
    const float r = 1.0f - fabsf(xi) - fabsf(eta);
    float a = xi, b = eta;
    if (r < 0.0f) {
        a = (xi >= 0.0f ? 1.0f : -1.0f) * (1.0f - fabsf(eta));
        b = (eta >= 0.0f ? 1.0f : -1.0f) * (1.0f - fabsf(xi));
    }
    const float nn = sqrtf(a * a + b * b + r * r);
    return make_float4(a / nn, b / nn, r / nn, 0.0f);
}

// Direction table of one class: entry jx | (jy << BD) holds Oct^-1(C_xi[jx], C_xi[jy]); the entry
// index is the 2*BD-bit field of the direction stream read as one number.
template <int BD>
__device__ __forceinline__ void build_dir_lut(float4 *lut, const float *c_xi, int tid, int nthreads) {
    constexpr int K = 1 << BD;
    for (int e = tid; e < K * K; e += nthreads) lut[e] = oct_decode(c_xi[e & (K - 1)], c_xi[e >> BD]);
}

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// Wave-wide reductions on the data-parallel-primitive path (no LDS traffic): shifts within rows of 16
// lanes, then row broadcasts; lane 63 ends up with the total, which is returned wave-uniform.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_take(float v) {
    // lanes whose source lane does not exist, or whose row is masked off, keep their own value
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}

__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_take<0x111, 0xf>(v));  // row_shr:1
    v = fmaxf(v, dpp_take<0x112, 0xf>(v));  // row_shr:2
    v = fmaxf(v, dpp_take<0x114, 0xf>(v));  // row_shr:4
    v = fmaxf(v, dpp_take<0x118, 0xf>(v));  // row_shr:8
    v = fmaxf(v, dpp_take<0x142, 0xa>(v));  // row_bcast:15 into rows 1 and 3
    v = fmaxf(v, dpp_take<0x143, 0xc>(v));  // row_bcast:31 into rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// The same for several values at once, one instruction per stage and value: the permute is part of the maximum (lanes whose
// source does not exist or whose row is masked off keep what they have), where the compiler makes a move, a
// canonicalisation and a maximum of it (18 of 24 instructions per value; 16 x 32768 tokens over 3-bit values, four / eight rows 148 ->
// 142.6 / 240 -> 216 us, eight rows of 4-bit keys at d = 64 53.4 -> 51).  A permute reads a register two wait states after
// it was written at the earliest, and the compiler puts no waits around inline assembly: all stages are ONE statement, so that
// nothing (a copy, a reload) can come between them.  Four values are each other's distance, fewer take waits; the waits at
// the ends are for what comes before and for the lane reads after (tests/test_wave_max_waits.py reads them in the built library).
#define OCTOPUS_MAX_OF(I, CTRL) "v_max_f32_dpp %" #I ", %" #I ", %" #I " " CTRL "\n"
#define OCTOPUS_MAX_OF_1(CTRL) OCTOPUS_MAX_OF(0, CTRL) "s_nop 1\n"
#define OCTOPUS_MAX_OF_2(CTRL) OCTOPUS_MAX_OF(0, CTRL) OCTOPUS_MAX_OF(1, CTRL) "s_nop 0\n"
#define OCTOPUS_MAX_OF_4(CTRL) OCTOPUS_MAX_OF(0, CTRL) OCTOPUS_MAX_OF(1, CTRL) OCTOPUS_MAX_OF(2, CTRL) OCTOPUS_MAX_OF(3, CTRL)
#define OCTOPUS_MAX_OF_8(CTRL) OCTOPUS_MAX_OF_4(CTRL) OCTOPUS_MAX_OF(4, CTRL) OCTOPUS_MAX_OF(5, CTRL) OCTOPUS_MAX_OF(6, CTRL) OCTOPUS_MAX_OF(7, CTRL)
#define OCTOPUS_MAX_STAGES(STAGE)                                                                                \
    "s_nop 1\n" STAGE("row_shr:1 row_mask:0xf bank_mask:0xf") STAGE("row_shr:2 row_mask:0xf bank_mask:0xf")      \
    STAGE("row_shr:4 row_mask:0xf bank_mask:0xf") STAGE("row_shr:8 row_mask:0xf bank_mask:0xf")                  \
    STAGE("row_bcast:15 row_mask:0xa bank_mask:0xf") STAGE("row_bcast:31 row_mask:0xc bank_mask:0xf") "s_nop 1"
template <int N>
__device__ __forceinline__ void wave_max_of(float (&x)[N]) {
    static_assert(N == 1 || N == 2 || N == 4 || N == 8, "values at once");
    if constexpr (N == 1) asm volatile(OCTOPUS_MAX_STAGES(OCTOPUS_MAX_OF_1) : "+v"(x[0]));
    else if constexpr (N == 2) asm volatile(OCTOPUS_MAX_STAGES(OCTOPUS_MAX_OF_2) : "+v"(x[0]), "+v"(x[1]));
    else if constexpr (N == 4) asm volatile(OCTOPUS_MAX_STAGES(OCTOPUS_MAX_OF_4) : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
    else asm volatile(OCTOPUS_MAX_STAGES(OCTOPUS_MAX_OF_8) : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]));
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[i]), 63));
}
#undef OCTOPUS_MAX_OF
#undef OCTOPUS_MAX_OF_1
#undef OCTOPUS_MAX_OF_2
#undef OCTOPUS_MAX_OF_4
#undef OCTOPUS_MAX_OF_8
#undef OCTOPUS_MAX_STAGES

__device__ __forceinline__ float wave_sum(float v) {
    auto take = [](float x, auto ctrl, auto rows) __attribute__((always_inline)) {   // 0 where no lane is read
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, decltype(rows)::value,
                                                          0xf, false));
    };
    using std::integral_constant;
    v += take(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});   // row_shr:1, 2, 4, 8
    v += take(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
    v += take(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
    v += take(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    v += take(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});   // row_bcast:15 into rows 1 and 3
    v += take(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});   // row_bcast:31 into rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Rows of 16 lanes exchanged between two registers: swap16 trades the odd rows of a for the even rows of b
// (rows 1 and 3 of a, rows 0 and 2 of b), swap32 the upper two rows of a for the lower two of b.
__device__ __forceinline__ void swap16(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap32(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

// The value of lane (l ^ M), without LDS traffic (a shuffle through LDS takes over a hundred cycles, these about ten).
template <int M>
__device__ __forceinline__ float lane_xor(float x, int lane) {
    static_assert(M == 1 || M == 2 || M == 4 || M == 8 || M == 16 || M == 32, "one bit of the lane index");
    if constexpr (M == 1) return dpp_take<0xB1, 0xf>(x);        // quad permute [1, 0, 3, 2]
    else if constexpr (M == 2) return dpp_take<0x4E, 0xf>(x);   // quad permute [2, 3, 0, 1]
    else if constexpr (M == 4) {
        // lanes 0-3 and 8-11 of each row from four lanes above, the others from four lanes below
        const int v = __float_as_int(x);
        const int up = __builtin_amdgcn_update_dpp(v, v, 0x104, 0xf, 0x5, false);
        return __int_as_float(__builtin_amdgcn_update_dpp(up, v, 0x114, 0xf, 0xa, false));
    } else if constexpr (M == 8) return dpp_take<0x128, 0xf>(x);   // row rotate by 8
    else {
        float a = x, b = x;
        if constexpr (M == 16) swap16(a, b); else swap32(a, b);   // a: the lower of each pair of rows twice, b: the upper
        return (lane & M) ? a : b;
    }
}

}  // namespace octopus

#endif
