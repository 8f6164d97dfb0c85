// Device-side helpers shared by the kernels (not part of the ABI): vector types, the MFMA
// wrapper, the 16-bit storage conversions and the padding bias.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fk {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
// the same 16 bytes at any element's address
typedef uint32_t uintx4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef float floatx4_any __attribute__((ext_vector_type(4), aligned(4)));

// Score bias of centroid rows beyond K: it must survive having its low mantissa bits
// overwritten by the packed argmax (-inf would turn into a NaN pattern) and still lose against
// every real score.
constexpr float kPadBias = -3.0e38f;

__device__ __forceinline__ float lp_to_float(uint16_t v, bool bf) {
    return bf ? __uint_as_float((uint32_t)v << 16) : (float)__builtin_bit_cast(_Float16, v);
}

// round-to-nearest-even from fp32 (finite input)
__device__ __forceinline__ uint16_t float_to_lp(float f, bool bf) {
    if (bf) {
        uint32_t u = __float_as_uint(f);
        u += 0x7FFFu + ((u >> 16) & 1u);
        return (uint16_t)(u >> 16);
    }
    return __builtin_bit_cast(uint16_t, (_Float16)f);
}

// D = A (32 x 16) * B (16 x 32) + C with fp32 accumulation; lane (r = lane % 32, h = lane / 32)
// supplies A[r][8h .. 8h+7] and B[8h .. 8h+7][r] and receives D[8*(i/4) + 4h + i%4][r], i < 16.
template <bool BF>
__device__ __forceinline__ floatx16 mfma32(uintx4 a, uintx4 b, floatx16 c) {
    if constexpr (BF)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a),
                                                      __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

// Rows as the caller stores them: `len` elements, no padding, at any element's address.  The kernels
// work on widths d = len rounded up to a multiple of 8 and read a row in pieces of 16 bytes that
// start at j, a multiple of 8 (fp32: of 4) below d.  Nothing outside the row is ever read (len >= 8):
// raw_* reads the piece that would cross the row's end so that it ends there, settle* then moves
// its elements down to where they belong and fills up with zeros.  The two are apart so that a
// kernel can issue all its loads first and settle them under one test of len, which keeps rows
// that need none of it on straight-line code.  RAGGED = false: len is a multiple of 8 and the rows
// are 16-byte aligned; the plain load, whose offset goes into the instruction (assign_f32_split_kernel,
// 217895 points, d = 128, K = 18: 92 us with it, 108 with the test at every load).
template <bool RAGGED = true>
__device__ __forceinline__ uintx4 raw_piece16(const uint16_t* __restrict__ row, int j, int len) {
    if constexpr (!RAGGED) return *(const uintx4*)(row + j);
    return *(const uintx4_any*)(row + min(j, len - 8));
}

__device__ __forceinline__ uintx4 settle16(uintx4 v, int j, int len) {
    const int s = (8 - (len & 7)) * 16;                     // wave-uniform; 16 .. 112 where it matters
    const uint64_t lo = (uint64_t)v[0] | ((uint64_t)v[1] << 32), hi = (uint64_t)v[2] | ((uint64_t)v[3] << 32);
    const uint64_t a = s >= 64 ? hi >> ((s - 64) & 63) : (lo >> s) | (hi << ((64 - s) & 63)), c = s >= 64 ? 0 : hi >> s;
    return j + 8 > len ? uintx4{(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)c, (uint32_t)(c >> 32)} : v;
}

template <bool RAGGED = true>
__device__ __forceinline__ uintx4 row_piece16(const uint16_t* __restrict__ row, int j, int len) {
    uintx4 v = raw_piece16<RAGGED>(row, j, len);
    if (RAGGED && (len & 7)) v = settle16(v, j, len);
    return v;
}

template <bool RAGGED = true>
__device__ __forceinline__ floatx4 raw_piece32(const float* __restrict__ row, int j, int len) {
    if constexpr (!RAGGED) return *(const floatx4*)(row + j);
    return *(const floatx4_any*)(row + min(j, len - 4));
}

__device__ __forceinline__ floatx4 settle32(floatx4 v, int j, int len) {
    const int past = j + 4 - len;                           // elements of the piece past the end
    return past <= 0 ? v
         : past == 1 ? floatx4{v[1], v[2], v[3], 0.f}
         : past == 2 ? floatx4{v[2], v[3], 0.f, 0.f}
         : past == 3 ? floatx4{v[3], 0.f, 0.f, 0.f} : floatx4{0.f, 0.f, 0.f, 0.f};
}

template <bool RAGGED = true>
__device__ __forceinline__ floatx4 row_piece32(const float* __restrict__ row, int j, int len) {
    floatx4 v = raw_piece32<RAGGED>(row, j, len);
    if (RAGGED && (len & 7)) v = settle32(v, j, len);
    return v;
}

// A whole ragged row in registers, zeros past its end: the pieces inside the row by plain loads at any
// element's address, the one that crosses its end from len - 4 and moved into place.  A test of len at
// every load instead is slower for DMAX = 32 and 128 (500000 points, d = 29, K = 9 58 us against 22; 10^6, d =
// 100, K = 12 296 against 219), and the faster form for 64 (300000 points, d = 43, K = 20 34.4 against 37.4;
// d = 60 the same).
template <int DMAX>
__device__ __forceinline__ void load_row32(float (&x)[DMAX], const float* __restrict__ row, int len, bool live) {
    floatx4 last = {0.f, 0.f, 0.f, 0.f};
    if (DMAX != 64 && (len & 3) && live) last = *(const floatx4_any*)(row + len - 4);
#pragma unroll
    for (int j = 0; j < DMAX; j += 4) {
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
        if constexpr (DMAX == 64) {
            if (live && j < len) v = raw_piece32(row, j, len);
        } else {
            if (live && j + 4 <= len) v = *(const floatx4_any*)(row + j);
        }
        x[j] = v[0]; x[j + 1] = v[1]; x[j + 2] = v[2]; x[j + 3] = v[3];
    }
    if (len & 3) {
#pragma unroll
        for (int j = 4; j < DMAX; j += 4)
            if (j == (len & ~3)) {
                const floatx4 v = settle32(DMAX == 64 ? floatx4{x[j], x[j + 1], x[j + 2], x[j + 3]} : last, j, len);
                x[j] = v[0]; x[j + 1] = v[1]; x[j + 2] = v[2]; x[j + 3] = v[3];
            }
    }
}

// Of the filtered fp32 assignment (fk_f32_filter.hip): score bias that every real score loses to / that beats every real score, both
// bf16 values; and the relative error of a score in units of |x'|^2 + |c'|^2 (derived there).
constexpr uint16_t kNever = 0xFF62, kAlways = 0x7F62;      // -/+ 3.0e38

__host__ __device__ constexpr float filter_kappa(int width) {
    return 7.62939453125e-06f + (0.53f * (float)width + 24.f) * 1.1920929e-07f;
}

// The bias piece of a centroid with squared norm n2 after the shift: -n2 / 2 + kappa n2 as three bf16 values (24 bits), and the norm
// that goes with it, from above.  A row whose norm overflows always wins with an infinite norm, so that no point is ever certain of
// it; one that is not finite (or beyond K: `never`) never does.
__device__ __forceinline__ uintx4 split_bias(double n2, int width, bool never, float* norm) {
    const bool fine = !never && n2 < 1e38;                   // false for NaN too
    uint16_t p[3] = {kNever, 0, 0};
    if (fine) {
        double left = (-0.5 + (double)filter_kappa(width)) * n2;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            p[q] = float_to_lp((float)left, true);
            left -= (double)lp_to_float(p[q], true);
        }
    } else if (!never) {
        p[0] = kAlways;
    }
    *norm = fine ? (float)(n2 * 1.000001) : never ? 0.f : INFINITY;
    return uintx4{(uint32_t)p[0] | ((uint32_t)p[1] << 16), p[2], 0u, 0u};
}

// 32-bit LDS address of a pointer into shared memory (for hand-issued LDS instructions)
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)((__attribute__((address_space(3))) const void*)p);
}

}  // namespace fk
