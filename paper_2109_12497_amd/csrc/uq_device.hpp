// Device-side building blocks of libuq (gfx950, wave64).
//
// Everything here follows the arithmetic contract in include/uq.h: IEEE
// binary32 products with no contraction (the library is compiled with
// -ffp-contract=off), correctly rounded tables formed in binary64, and the
// Philox4x32-10 counter-based generator of Salmon, Moraes, Dror and Shaw
// ("Parallel random numbers: as easy as 1, 2, 3", SC'11).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace uq {

constexpr int kBlock = 256;          // threads per block: four wave64s
constexpr int kMaxScales = 16;
constexpr float kFloatMax = 3.40282346638528859812e+38f;

// Native clang vectors (HIP's float4 is a wrapper struct, which the
// nontemporal builtins do not accept).
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Single-use streams: loads and stores marked nontemporal so they do not
// displace reused lines from the caches.
__device__ __forceinline__ f32x4 load_nt(const float* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
}
__device__ __forceinline__ i32x4 load_nt(const int32_t* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const i32x4*>(p));
}
__device__ __forceinline__ u32x4 load_nt(const uint32_t* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ uint32_t load_nt_u32(const void* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(p));
}
__device__ __forceinline__ void store_nt(float* p, f32x4 v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(p));
}

// Stores that write through the caches (cache policy sc0 sc1: every level
// passes the line on at once, in the order of the stores) instead of leaving
// dirty lines in the XCD's L2 to be evicted later, out of order; NT adds the
// nontemporal hint.  Work-free passes on MI355X with 256-thread blocks and
// nontemporal, plain or write-through stores: 4 bytes in and 1 out at 2^27
// coordinates 99.6, 94.7 and 89.7 us; the accumulating pass (8.5 in, 4 out)
// at 25.6 M 45.9, 44 and 38.5 us.  Beyond the 256 MB Infinity Cache the
// accumulating pass, whose next call reads the sums back, is faster with
// both (2.03 against 2.15 ms at 2^30).  `base` is wave-uniform.
template <bool NT, typename V>
__device__ __forceinline__ void store_through(void* base, uint32_t byte_off, V v)
{
    constexpr int kSc0 = 1, kNt = 2, kSc1 = 16;
    constexpr int policy = kSc0 | kSc1 | (NT ? kNt : 0);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00027000);
    if constexpr (sizeof(V) == 16)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, byte_off, 0, policy);
    else if constexpr (sizeof(V) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, byte_off, 0, policy);
    else if constexpr (sizeof(V) == 2)
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, v), r, byte_off, 0, policy);
    else
        __builtin_amdgcn_raw_buffer_store_b8(__builtin_bit_cast(uint8_t, v), r, byte_off, 0, policy);
}

// Scale set passed by value in the kernel arguments.
struct ScaleSet {
    float s[kMaxScales];
    int32_t K;
    float s_last;  // s[K - 1]
};

// Philox4x32-10 block function: ten rounds, each multiplying counter words 0
// and 2 by the Philox multipliers (32x32 -> 64 bit), xoring the high halves
// into the other two words together with the round key, and permuting; the
// key advances by the Weyl increments after every round.  The three-way xors
// are single v_bitop3_b32 instructions (truth table 0x96 = a ^ b ^ c).
__device__ __forceinline__ uint4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t pa = static_cast<uint64_t>(0xD2511F53u) * c0;
        const uint64_t pb = static_cast<uint64_t>(0xCD9E8D57u) * c2;
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pb >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pa >> 32), c3, k1, 0x96);
        c1 = static_cast<uint32_t>(pb);
        c3 = static_cast<uint32_t>(pa);
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return make_uint4(c0, c1, c2, c3);
}

// RN32(a / b) for binary32 a, b: the binary64 quotient rounded once more to
// binary32 is the correctly rounded binary32 quotient (53 >= 2*24 + 2).
__device__ __forceinline__ float div_rn32(float a, float b)
{
    return static_cast<float>(static_cast<double>(a) / static_cast<double>(b));
}

// The zero path: W not a positive finite binary32, or s_0 / W overflowing.
__device__ __forceinline__ bool zero_path(float W, float inv0)
{
    return !(W > 0.0f) || !(W <= kFloatMax) || !(inv0 <= kFloatMax);
}

// v_cmp_class masks: finite nonzero values (+-normal, +-denormal); NaN and
// infinities.
constexpr int kFiniteNonzero = (1 << 3) | (1 << 4) | (1 << 7) | (1 << 8);
constexpr int kNonFinite = (1 << 0) | (1 << 1) | (1 << 2) | (1 << 9);

// sign(v) * mag for an integer magnitude (v's sign bit; 0 stays 0).
__device__ __forceinline__ int32_t apply_sign(uint32_t mag, float v)
{
    const int32_t s = __float_as_int(v) >> 31;
    return (static_cast<int32_t>(mag) ^ s) - s;
}

// x = min(|v| * inv, s0), 0 for zero / NaN / inf v.  inv is 0 on the zero
// path, so every code is then 0.
__device__ __forceinline__ float scaled_magnitude(float v, float inv, float s0)
{
    const bool ok = __builtin_amdgcn_classf(v, kFiniteNonzero);
    const float x = fabsf(v) * inv;
    return fminf(ok ? x : 0.0f, s0);
}

// Stochastic level choice for one coordinate from the high 16 bits of its
// uniform word:
//   l = floor(x), t = floor((x - l) * 2^32), code = sign(v) * (l + [r < t])
// As 0 <= x <= 127, T = floor(x * 2^16) is exact and equals
// l * 2^16 + (t >> 16): one conversion yields the level and the high half of
// the threshold.  With only r's high half known, [r < t] is decided unless
// the halves tie (hi16 == t >> 16), reported in *tie; the caller finishes a
// tie from x (*x_out) and r's low half with quantise_tie.
__device__ __forceinline__ int32_t quantise_hi(float v, float inv, float s0, uint32_t hi16, bool* tie,
                                               float* x_out)
{
    const float x = scaled_magnitude(v, inv, s0);
    const uint32_t T = static_cast<uint32_t>(x * 65536.0f);
    const uint32_t th = T & 0xFFFFu;
    *tie = hi16 == th;
    *x_out = x;
    return apply_sign((T >> 16) + (hi16 < th ? 1u : 0u), v);
}

// The Philox blocks of one lane for several rows of a tile.  A tile's lanes
// share the counter's high word and each row's worker id, so the products of
// the first two rounds split into a part that depends on the row alone
// (RowKey: scalar arithmetic) and one that depends on the lane alone
// (LaneKey: once for all rows); a row then costs 16 products instead of 19.
struct RowKey {
    uint32_t n0, n1;      // counter words 0 and 1 after round 1
    uint32_t p_hi, p_lo;  // round 2's product of word 0
};
struct LaneKey {
    uint32_t n3;          // counter word 3 after round 1
    uint32_t p_hi, p_lo;  // round 2's product of word 2
};

__device__ __forceinline__ RowKey row_key(uint32_t c1, uint32_t worker, uint32_t key0)
{
    const uint64_t pb = static_cast<uint64_t>(0xCD9E8D57u) * worker;
    RowKey r;
    r.n0 = static_cast<uint32_t>(pb >> 32) ^ c1 ^ key0;
    r.n1 = static_cast<uint32_t>(pb);
    const uint64_t pa = static_cast<uint64_t>(0xD2511F53u) * r.n0;
    r.p_hi = static_cast<uint32_t>(pa >> 32);
    r.p_lo = static_cast<uint32_t>(pa);
    return r;
}

__device__ __forceinline__ LaneKey lane_key(uint32_t c0, uint32_t c3, uint32_t key1)
{
    const uint64_t pa = static_cast<uint64_t>(0xD2511F53u) * c0;
    LaneKey l;
    l.n3 = static_cast<uint32_t>(pa);
    const uint64_t pb = static_cast<uint64_t>(0xCD9E8D57u) * (static_cast<uint32_t>(pa >> 32) ^ c3 ^ key1);
    l.p_hi = static_cast<uint32_t>(pb >> 32);
    l.p_lo = static_cast<uint32_t>(pb);
    return l;
}

// The complement of philox4x32_10(c0, c1, worker, c3, key) from its row and
// lane parts (words 0 and 2 are complemented by the last round's
// three-operand xors: truth table 0x69).
__device__ __forceinline__ uint4 philox_tail_not(const RowKey& r, const LaneKey& l, uint32_t key0, uint32_t key1)
{
    uint32_t k0 = key0 + 0x9E3779B9u, k1 = key1 + 0xBB67AE85u;
    uint32_t c0 = __builtin_amdgcn_bitop3_b32(l.p_hi, r.n1, k0, 0x96);
    uint32_t c1 = l.p_lo;
    uint32_t c2 = __builtin_amdgcn_bitop3_b32(r.p_hi, l.n3, k1, 0x96);
    uint32_t c3 = r.p_lo;
#pragma unroll
    for (int round = 2; round < 10; ++round) {
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
        const uint64_t pa = static_cast<uint64_t>(0xD2511F53u) * c0;
        const uint64_t pb = static_cast<uint64_t>(0xCD9E8D57u) * c2;
        if (round < 9) {
            c0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pb >> 32), c1, k0, 0x96);
            c2 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pa >> 32), c3, k1, 0x96);
            c1 = static_cast<uint32_t>(pb);
            c3 = static_cast<uint32_t>(pa);
        } else {
            c0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pb >> 32), c1, k0, 0x69);
            c2 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pa >> 32), c3, k1, 0x69);
            c1 = ~static_cast<uint32_t>(pb);
            c3 = ~static_cast<uint32_t>(pa);
        }
    }
    return make_uint4(c0, c1, c2, c3);
}

// v_cvt_u32_f32: truncates, with 0 for NaN and for negative values and
// 0xFFFFFFFF for values of 2^32 and above (a C++ conversion leaves those
// undefined).
__device__ __forceinline__ uint32_t cvt_u32_sat(float x)
{
    uint32_t r;
    __asm__("v_cvt_u32_f32_e32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// The largest of the low 16 bits of a, b and c, in the low 16 bits (the high
// half of the result is not defined).
__device__ __forceinline__ uint32_t max3_lo16(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t r;
    __asm__("v_max3_u16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Adds half `half` (0: low, 1: high) of `halves` to t.
template <int HALF>
__device__ __forceinline__ uint32_t add_half(uint32_t t, uint32_t halves)
{
    return t + (HALF ? halves >> 16 : halves & 0xFFFFu);
}

// Signs of two coordinates as 16-bit lanes: 1 or -1 (by the sign bits).
__device__ __forceinline__ u16x2 pair_signs(float v0, float v1)
{
    // 0xFFFF in the lane of a negative v (replicated sign bits of the top bytes)
    const uint32_t neg = __builtin_amdgcn_perm(__float_as_uint(v1), __float_as_uint(v0), 0x0B0B0909u);
    return __builtin_bit_cast(u16x2, neg | 0x00010001u);
}

// |code| of one coordinate from its whole uniform word (hi16, lo16):
// l + [r < t], 0 for a NaN or infinite v.  inv and s0x carry a factor of
// 2^16 when pre (the products are then finite for finite v, up to overflow
// to infinity, which the minimum takes to s0); else inv may be infinite and
// the factor is applied after the minimum.
__device__ __forceinline__ uint32_t exact_magnitude(float v, float inv, float s0x, bool pre, uint32_t hi16,
                                                    uint32_t lo16)
{
    float xs;
    if (pre)
        xs = __builtin_amdgcn_classf(v, kNonFinite) ? 0.0f : fminf(fabsf(v) * inv, s0x);
    else
        xs = scaled_magnitude(v, inv, s0x) * 65536.0f;
    const uint32_t T = static_cast<uint32_t>(xs);
    const uint32_t th = T & 0xFFFFu;
    const uint32_t t_lo = static_cast<uint32_t>((xs - floorf(xs)) * 65536.0f);
    return (T >> 16) + ((hi16 < th || (hi16 == th && lo16 < t_lo)) ? 1u : 0u);
}

// The tied case: [r < t] decided by the low halves of r and t.
__device__ __forceinline__ int32_t quantise_tie(float v, float x, uint32_t lo16)
{
    const float lf = floorf(x);
    const uint32_t t = static_cast<uint32_t>((x - lf) * 4294967296.0f);
    return apply_sign(static_cast<uint32_t>(lf) + (lo16 < (t & 0xFFFFu) ? 1u : 0u), v);
}

// Deterministic wave64 sum of a double (fixed butterfly order).
__device__ __forceinline__ double wave_sum(double x)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        x += __shfl_xor(x, off, 64);
    return x;
}

}  // namespace uq
