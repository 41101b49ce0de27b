// Small device helpers shared by the bf16 kernels: MFMA operand types,
// 16-byte register packs, and unaligned 8-element row reads built from
// aligned 16-byte loads.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace dc {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

// v_mfma_f32_32x32x16_bf16 written out so that the register class of the A
// operand is chosen here: AG = true reads it from AGPRs (the 512-entry
// register file of a wave holds a weight operand larger than the 256 VGPRs
// that way), ZERO = true starts a new accumulation (C = 0).  The accumulator
// lives in AGPRs.  The hardware interlocks back-to-back MFMAs that accumulate
// into the same registers; any other reader of the accumulator must come after
// mfma_drain(), and an A/B operand must not be written by a VALU instruction
// in the two instructions before the MFMA (A/B here come from loads).  The
// statements are volatile: memory operations keep their source order around
// them, which fixes how far loads run ahead and where stores interleave.
template <bool AG, bool ZERO>
__device__ __forceinline__ void mfma32x32x16(floatx16& acc, const bf16x8& a, const bf16x8& b) {
    if constexpr (ZERO) {
        if constexpr (AG)
            asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&a"(acc) : "a"(a), "v"(b));
        else
            asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&a"(acc) : "v"(a), "v"(b));
    } else {
        if constexpr (AG)
            asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "a"(a), "v"(b));
        else
            asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
    }
}

// Wait states between the last MFMA writing `acc` and any non-MFMA reader of
// it (32 >= passes + 4 for every 32x32 shape).
__device__ __forceinline__ void mfma_drain(floatx16& acc) {
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7" : "+a"(acc));
}

// Compile-time loop: f(std::integral_constant<int, I>) for I in [B, E).
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

union Pack8 {
    uint4 v;
    uint32_t d[4];
    uint16_t h[8];
    bf16x8 b;
};

// Elements [sh, sh+8) of the 16-element window d[0..7] (two aligned 16-byte chunks).
template <int SH>
__device__ __forceinline__ uint4 window8(const uint32_t (&d)[8]) {
    uint4 r;
    uint32_t* o = reinterpret_cast<uint32_t*>(&r);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if ((SH & 1) == 0)
            o[i] = d[SH / 2 + i];
        else
            o[i] = __builtin_amdgcn_alignbyte(d[SH / 2 + i + 1], d[SH / 2 + i], 2);
    }
    return r;
}

__device__ __forceinline__ uint4 window8_rt(const uint32_t (&d)[8], int sh) {
    switch (sh) {
        case 0: return window8<0>(d);
        case 1: return window8<1>(d);
        case 2: return window8<2>(d);
        case 3: return window8<3>(d);
        case 4: return window8<4>(d);
        case 5: return window8<5>(d);
        case 6: return window8<6>(d);
        default: return window8<7>(d);
    }
}

// The same window for a shift known only at run time (0..7, equal on every
// lane), without branches: selects pick the whole dwords, a byte-align the
// odd element.  Straight-line code lets the scheduler interleave it with
// matrix instructions.
__device__ __forceinline__ uint4 window8_sel(const uint32_t (&d)[8], int sh) {
    const int k = sh >> 1;
    const uint32_t bs = uint32_t(sh & 1) * 2u;
    uint32_t w[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        const uint32_t a = k & 1 ? d[j + 1] : d[j];
        const uint32_t b = k & 1 ? d[j + 3] : d[j + 2];
        w[j] = k & 2 ? b : a;
    }
    uint4 r;
    r.x = __builtin_amdgcn_alignbyte(w[1], w[0], bs);
    r.y = __builtin_amdgcn_alignbyte(w[2], w[1], bs);
    r.z = __builtin_amdgcn_alignbyte(w[3], w[2], bs);
    r.w = __builtin_amdgcn_alignbyte(w[4], w[3], bs);
    return r;
}

// 8 consecutive bf16 of a row starting at column g0 + sh, where g0 is a
// multiple of 8 and sh (0..7) is the same for the whole wave; columns outside
// [0, ncols) read as zero.  `row` is 16-byte aligned with `pitch` (a multiple
// of 8, >= ncols) readable elements.  Loads are unconditional 16-byte loads
// from clamped, always-valid addresses; out-of-range data is masked after.
__device__ __forceinline__ uint4 load_row8(const uint16_t* row, int g0, int sh, int ncols,
                                           int pitch, bool row_ok) {
    const int g = g0 + sh;
    const bool ok0 = row_ok && g < ncols;
    uint4 v = *reinterpret_cast<const uint4*>(row + (ok0 ? g0 : 0));
    if (sh != 0) {
        const bool ok1 = ok0 && g0 + 8 < pitch;
        uint4 v1 = *reinterpret_cast<const uint4*>(row + (ok1 ? g0 + 8 : 0));
        if (!ok1) v1 = make_uint4(0, 0, 0, 0);
        const uint32_t d[8] = {v.x, v.y, v.z, v.w, v1.x, v1.y, v1.z, v1.w};
        v = window8_rt(d, sh);
    }
    const int nv = ok0 ? ncols - g : 0;   // valid elements of this group of 8
    uint32_t* w = reinterpret_cast<uint32_t*>(&v);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t m = (2 * i < nv ? 0x0000ffffu : 0u) | (2 * i + 1 < nv ? 0xffff0000u : 0u);
        w[i] &= m;
    }
    return v;
}

// Keep the first nv (clamped to 0..8) elements of a group of 8, zero the rest.
__device__ __forceinline__ uint4 mask8(uint4 v, int nv) {
    uint32_t* w = reinterpret_cast<uint32_t*>(&v);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t m = (2 * i < nv ? 0x0000ffffu : 0u) | (2 * i + 1 < nv ? 0xffff0000u : 0u);
        w[i] &= m;
    }
    return v;
}

// e / d for e, d < 2^16 by the host's m = 2^32 / d + 1 (0 for d = 1)
__device__ __forceinline__ int div16(int e, uint32_t m) { return m ? int(__umulhi(uint32_t(e), m)) : e; }

// The smallest of the staged values, without the sign and minus one (so that
// zero is the largest).  Nonzero values below 2^-110 do not fit three bf16
// parts: a value's last bit lies 23 binades below its first, bf16's last
// subnormal is 2^-133.  (The leading part would not tell: below 2^-134 it
// rounds to zero.)  Too large values need no such watch: parts and part
// products that overflow, like infinities and NaN, leave infinities or NaN in
// every sum that they reach.
struct PartRange {
    static constexpr uint32_t kLeast = 0x08800000u << 1;   // 2^-110
    uint32_t lo = 0xffffffffu;
    __device__ static __forceinline__ uint32_t key(uint32_t u) { return (u << 1) - 1; }
    __device__ static __forceinline__ bool tiny(uint32_t u) { return key(u) < kLeast - 1; }
    __device__ __forceinline__ bool outside() const { return lo < kLeast - 1; }
};

// 8 fp32 values -> three records of bf16 parts (round to nearest, remainder,
// again): each part holds 8 bits and a sign, so three hold all 24 of a value
// that is not tiny
__device__ __forceinline__ void split8(const float (&f)[8], uint4 (&p)[3], PartRange& range) {
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    uint32_t w[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = f[2 * i], b = f[2 * i + 1];
        range.lo = min(range.lo, min(PartRange::key(__builtin_bit_cast(uint32_t, a)), PartRange::key(__builtin_bit_cast(uint32_t, b))));
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const uint32_t u = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{a, b}), bf2));
            if (s < 2) {
                a -= __builtin_bit_cast(float, u << 16);
                b -= __builtin_bit_cast(float, u & 0xffff0000u);
            }
            w[s][i] = u;
        }
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) p[s] = uint4{w[s][0], w[s][1], w[s][2], w[s][3]};
}

}  // namespace dc
