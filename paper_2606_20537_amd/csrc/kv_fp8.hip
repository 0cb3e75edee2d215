// FP8 KV region on gfx950: BF16 <-> OCP E4M3 conversion of KV rows.
//
// Paper §3 "Definition": the KV region may be held in FP8, which roughly
// halves the capsule; the BF16 working stage of the attention is not part of
// the capsule and, after a restore, is rebuilt lazily on the next read (§3
// cost model: restore copies bytes and rebinds, the stage follows on demand).
// Quantize writes appended rows into the FP8 region; dequantize rebuilds the
// BF16 stage for a range of rows.
//
// Format (OCP 8-bit floating point, E4M3): sign, 4 exponent bits with bias 7,
// 3 mantissa bits; subnormals m/8 * 2^-6; largest finite 448 (S.1111.110);
// S.1111.111 is NaN; there are no infinities.  Encoding rounds to nearest,
// ties to even, and saturates: |x| >= 448 and +-inf give +-448; NaN keeps its
// sign (the product's, x times 1 / scale).  Each conversion is one fp32 product
// and one correctly rounded conversion instruction, so the codes and the BF16
// results are bit-identical to any implementation of the same definition.
//
// Streaming, HBM-bound: a unit is 8 elements, 16 bytes of BF16 and 8 of FP8, so
// that the lanes of a wave read and write contiguous bytes on both sides
// (nontemporal); a thread has its two units' loads in flight before it
// converts the first (four: 190 and 207 us at the size below, one: 222 and 218).
// One grid covers up to 64 segments (one per KV buffer), each block a run of
// 4096 elements of one segment found by a binary search over the launch table.
// The conversions are the hardware's (OCP on gfx950:
// v_cvt_pk_fp8_f32, v_cvt_pk_f32_fp8, v_cvt_pk_bf16_f32; round to nearest even),
// with saturation in front of the encoder, which by itself would turn an
// overflow into NaN.  In integer arithmetic they took about 20 instructions an
// element and bound the kernel (24 buffers x 16.8 M elements: quantize 264 us,
// dequantize 247 us; now 183 and 193 us in a kernel trace, 6.6 and 6.3 TB/s).
#include <hip/hip_runtime.h>

#include "internal.h"

namespace cap {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ inline float bits_f32(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ inline uint32_t sign_bit(float x) { return __builtin_bit_cast(uint32_t, x) & 0x80000000u; }

// +-448 for anything larger, infinities included; NaN stays.
__device__ inline float saturate(float x) {
    return __builtin_fabsf(x) > 448.0f ? __builtin_copysignf(448.0f, x) : x;
}

// Two bf16 elements (one word) to two codes in bytes 0 and 1 (hi: 2 and 3) of w.
template <bool HI>
__device__ inline uint32_t encode2(uint32_t v, float mul, uint32_t w) {
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(saturate(bits_f32(v << 16) * mul),
                                                     saturate(bits_f32(v & 0xFFFF0000u) * mul), (int)w, HI);
}

// Codes in bytes 0 and 1 (hi: 2 and 3) of w to two bf16 elements.
template <bool HI>
__device__ inline uint32_t decode2(uint32_t w, float mul) {
    const f32x2 x = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, HI);
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){x[0] * mul, x[1] * mul}, bf16x2));
}

// The conversions give NaN the sign bit whatever sign it had.  Whether any
// byte of w is zero, and (rare, after that) 0x80 in exactly the zero bytes.
__device__ inline bool any_zero(uint32_t w) { return ((w - 0x01010101u) & ~w & 0x80808080u) != 0; }
__device__ inline uint32_t zero_bytes(uint32_t w) { return ~(((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w | 0x7F7F7F7Fu); }

__device__ inline uint32_t segment_of(const Fp8Params& p, uint32_t b) {
    uint32_t lo = 0, hi = p.n_seg - 1;  // last s with first_block[s] <= b
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (p.first_block[mid] <= b) lo = mid; else hi = mid - 1;
    }
    return lo;
}

template <bool QUANT>
__global__ __launch_bounds__(256) void fp8_kernel(const Fp8Params p) {
    const uint32_t block = blockIdx.y * kFp8GridX + blockIdx.x;
    const uint32_t s = __builtin_amdgcn_readfirstlane(segment_of(p, block));
    const uint64_t n = 2 * p.n_groups[s];  // units
    constexpr int kU = 2 * kFp8GroupsPerBlock / 256;
    const uint64_t u0 = (uint64_t)(block - p.first_block[s]) * (256 * kU) + threadIdx.x;
    const float mul = p.mul[s];
    if (QUANT) {
        const u32x4* src = reinterpret_cast<const u32x4*>(p.src[s]);
        u32x2* dst = reinterpret_cast<u32x2*>(p.dst[s]);
        u32x4 in[kU];
        #pragma unroll
        for (int u = 0; u < kU; ++u)
            if (u0 + u * 256 < n) in[u] = __builtin_nontemporal_load(src + u0 + u * 256);
        #pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (u0 + u * 256 < n) {
                u32x2 out;
                #pragma unroll
                for (int w = 0; w < 2; ++w)
                    out[w] = encode2<true>(in[u][2 * w + 1], mul, encode2<false>(in[u][2 * w], mul, 0u));
                // NaN codes take the signs of the products (zero times the
                // infinite reciprocal of a tiny scale is a NaN of its own sign)
                if (any_zero(~out[0]) || any_zero(~out[1])) {
                    #pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        const uint32_t a = in[u][2 * w], b = in[u][2 * w + 1], nan = zero_bytes(~out[w]);
                        const uint32_t sign = sign_bit(bits_f32(a << 16) * mul) >> 24 | sign_bit(bits_f32(a & 0xFFFF0000u) * mul) >> 16 |
                                              sign_bit(bits_f32(b << 16) * mul) >> 8 | sign_bit(bits_f32(b & 0xFFFF0000u) * mul);
                        out[w] = (out[w] & ~nan) | (sign & nan);
                    }
                }
                __builtin_nontemporal_store(out, dst + u0 + u * 256);
            }
        }
    } else {
        const u32x2* src = reinterpret_cast<const u32x2*>(p.src[s]);
        u32x4* dst = reinterpret_cast<u32x4*>(p.dst[s]);
        u32x2 in[kU];
        #pragma unroll
        for (int u = 0; u < kU; ++u)
            if (u0 + u * 256 < n) in[u] = __builtin_nontemporal_load(src + u0 + u * 256);
        #pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (u0 + u * 256 < n) {
                u32x4 out;
                #pragma unroll
                for (int w = 0; w < 2; ++w) {
                    out[2 * w] = decode2<false>(in[u][w], mul);
                    out[2 * w + 1] = decode2<true>(in[u][w], mul);
                }
                if (any_zero(in[u][0] ^ 0x7F7F7F7Fu) || any_zero(in[u][1] ^ 0x7F7F7F7Fu)) {  // positive NaN
                    #pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        const uint32_t nan = zero_bytes(in[u][w] ^ 0x7F7F7F7Fu);
                        out[2 * w] ^= (nan & 0x80u) << 8 | (nan & 0x8000u) << 16;
                        out[2 * w + 1] ^= (nan & 0x800000u) >> 8 | (nan & 0x80000000u);
                    }
                }
                __builtin_nontemporal_store(out, dst + u0 + u * 256);
            }
        }
    }
}

}  // namespace

hipError_t launch_fp8(const Fp8Params& p, hipStream_t stream) {
    const uint32_t blocks = p.first_block[p.n_seg];
    if (blocks == 0) return hipSuccess;
    const void* fn = p.quantize ? reinterpret_cast<const void*>(&fp8_kernel<true>)
                                : reinterpret_cast<const void*>(&fp8_kernel<false>);
    return launch_kernel(fn, dim3(fp8_grid_x(blocks), fp8_grid_y(blocks)), dim3(256), p, stream);
}

}  // namespace cap
