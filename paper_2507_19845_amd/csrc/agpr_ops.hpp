// Accessors for hand-placed accumulators in AGPRs: register numbers must appear literally
// in the instruction text, so there is one specialisation per group of four registers.
// Mechanical: one macro line per accumulator block.
#pragma once
#include "common.hpp"

namespace gpts {

typedef int i32x4_t __attribute__((ext_vector_type(4)));

// a[R:R+3] += X (16 x 32) * Y (32 x 16), R a multiple of 4.  The operands are eight 16-bit
// values per lane: bf16 (F16 = false) or fp16 (F16 = true: the same registers hold fp16 bits
// and the f16 form of the instruction is used).
template <int R, bool F16 = false> __device__ __forceinline__ void mfma16_at(const bf16x8& x, const bf16x8& y);
// value of AGPR R (after the matrix pipeline has drained)
template <int R> __device__ __forceinline__ float agpr_read();
// a[R:R+3] = 0 (and makes the register allocation of the kernel include them)
template <int R> __device__ __forceinline__ void agpr_zero4();

#define GPTS_AGPR_READ(R)                                                  \
  template <> __device__ __forceinline__ float agpr_read<R>() {            \
    float v;                                                               \
    asm volatile("v_accvgpr_read_b32 %0, a" #R : "=v"(v));                 \
    return v;                                                              \
  }
#define GPTS_MFMA16_ONE(F16, MNEMONIC, R0, R1, R2, R3)                                                     \
  template <> __device__ __forceinline__ void mfma16_at<R0, F16>(const bf16x8& x, const bf16x8& y) {       \
    asm volatile(MNEMONIC " a[" #R0 ":" #R3 "], %0, %1, a[" #R0 ":" #R3 "]" ::"v"(__builtin_bit_cast(i32x4_t, x)), \
                 "v"(__builtin_bit_cast(i32x4_t, y))                                                        \
                 : "a" #R0, "a" #R1, "a" #R2, "a" #R3);                                                     \
  }
#define GPTS_AGPR_ZERO4(R0, R1, R2, R3)                                                                   \
  template <> __device__ __forceinline__ void agpr_zero4<R0>() {                                          \
    asm volatile("v_accvgpr_write_b32 a" #R0 ", 0\n\tv_accvgpr_write_b32 a" #R1 ", 0\n\tv_accvgpr_write_b32 a" #R2 \
                 ", 0\n\tv_accvgpr_write_b32 a" #R3 ", 0" ::                                              \
                     : "a" #R0, "a" #R1, "a" #R2, "a" #R3);                                               \
  }
#define GPTS_ACC_BLOCK(R0, R1, R2, R3)                                   \
  GPTS_AGPR_ZERO4(R0, R1, R2, R3)                                        \
  GPTS_MFMA16_ONE(false, "v_mfma_f32_16x16x32_bf16", R0, R1, R2, R3)     \
  GPTS_MFMA16_ONE(true, "v_mfma_f32_16x16x32_f16", R0, R1, R2, R3)       \
  GPTS_AGPR_READ(R0) GPTS_AGPR_READ(R1) GPTS_AGPR_READ(R2) GPTS_AGPR_READ(R3)

GPTS_ACC_BLOCK(0, 1, 2, 3)
GPTS_ACC_BLOCK(4, 5, 6, 7)
GPTS_ACC_BLOCK(8, 9, 10, 11)
GPTS_ACC_BLOCK(12, 13, 14, 15)
GPTS_ACC_BLOCK(16, 17, 18, 19)
GPTS_ACC_BLOCK(20, 21, 22, 23)
GPTS_ACC_BLOCK(24, 25, 26, 27)
GPTS_ACC_BLOCK(28, 29, 30, 31)
GPTS_ACC_BLOCK(32, 33, 34, 35)
GPTS_ACC_BLOCK(36, 37, 38, 39)
GPTS_ACC_BLOCK(40, 41, 42, 43)
GPTS_ACC_BLOCK(44, 45, 46, 47)
GPTS_ACC_BLOCK(48, 49, 50, 51)
GPTS_ACC_BLOCK(52, 53, 54, 55)
GPTS_ACC_BLOCK(56, 57, 58, 59)
GPTS_ACC_BLOCK(60, 61, 62, 63)
GPTS_ACC_BLOCK(64, 65, 66, 67)
GPTS_ACC_BLOCK(68, 69, 70, 71)
GPTS_ACC_BLOCK(72, 73, 74, 75)
GPTS_ACC_BLOCK(76, 77, 78, 79)
GPTS_ACC_BLOCK(80, 81, 82, 83)
GPTS_ACC_BLOCK(84, 85, 86, 87)
GPTS_ACC_BLOCK(88, 89, 90, 91)
GPTS_ACC_BLOCK(92, 93, 94, 95)
GPTS_ACC_BLOCK(96, 97, 98, 99)
GPTS_ACC_BLOCK(100, 101, 102, 103)
GPTS_ACC_BLOCK(104, 105, 106, 107)
GPTS_ACC_BLOCK(108, 109, 110, 111)
GPTS_ACC_BLOCK(112, 113, 114, 115)
GPTS_ACC_BLOCK(116, 117, 118, 119)
GPTS_ACC_BLOCK(120, 121, 122, 123)
GPTS_ACC_BLOCK(124, 125, 126, 127)
GPTS_ACC_BLOCK(128, 129, 130, 131)
GPTS_ACC_BLOCK(132, 133, 134, 135)
GPTS_ACC_BLOCK(136, 137, 138, 139)
GPTS_ACC_BLOCK(140, 141, 142, 143)
GPTS_ACC_BLOCK(144, 145, 146, 147)
GPTS_ACC_BLOCK(148, 149, 150, 151)
GPTS_ACC_BLOCK(152, 153, 154, 155)
GPTS_ACC_BLOCK(156, 157, 158, 159)
GPTS_ACC_BLOCK(160, 161, 162, 163)
GPTS_ACC_BLOCK(164, 165, 166, 167)
GPTS_ACC_BLOCK(168, 169, 170, 171)
GPTS_ACC_BLOCK(172, 173, 174, 175)
GPTS_ACC_BLOCK(176, 177, 178, 179)
GPTS_ACC_BLOCK(180, 181, 182, 183)
GPTS_ACC_BLOCK(184, 185, 186, 187)
GPTS_ACC_BLOCK(188, 189, 190, 191)
GPTS_ACC_BLOCK(192, 193, 194, 195)
GPTS_ACC_BLOCK(196, 197, 198, 199)
GPTS_ACC_BLOCK(200, 201, 202, 203)
GPTS_ACC_BLOCK(204, 205, 206, 207)
GPTS_ACC_BLOCK(208, 209, 210, 211)
GPTS_ACC_BLOCK(212, 213, 214, 215)
GPTS_ACC_BLOCK(216, 217, 218, 219)
GPTS_ACC_BLOCK(220, 221, 222, 223)
GPTS_ACC_BLOCK(224, 225, 226, 227)
GPTS_ACC_BLOCK(228, 229, 230, 231)
GPTS_ACC_BLOCK(232, 233, 234, 235)
GPTS_ACC_BLOCK(236, 237, 238, 239)
GPTS_ACC_BLOCK(240, 241, 242, 243)
GPTS_ACC_BLOCK(244, 245, 246, 247)
GPTS_ACC_BLOCK(248, 249, 250, 251)
GPTS_ACC_BLOCK(252, 253, 254, 255)
#undef GPTS_ACC_BLOCK
#undef GPTS_AGPR_ZERO4
#undef GPTS_MFMA16_ONE
#undef GPTS_AGPR_READ

}  // namespace gpts
