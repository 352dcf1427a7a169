// tilemix_device.h -- shared gfx950 device helpers for the TileMix kernels.
//
// Matrix-core shapes used (CDNA4 / gfx950, wave64):
//   v_mfma_f32_32x32x16_f16 : A 32x16, B 16x32 FP16 -> D 32x32 FP32
//   v_mfma_i32_32x32x32_i8  : A 32x32, B 32x32 INT8 -> D 32x32 INT32 (exact)
// Operand lane layout (both shapes): lane l holds row/column (l % 32) and the
// contraction slice [kw*(l/32), kw*(l/32)+kw) with kw = 8 (f16) or 16 (i8).
// Accumulator layout: register r of lane l is D[8*(r/4) + 4*(l/32) + r%4][l%32].
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tilemix {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr int kQuantBlockQ = 128;  // query rows per INT8 scale block (Appendix C)
constexpr int kQuantBlockK = 64;   // key rows per INT8 scale block (Appendix C)
constexpr int kBlockN = 64;        // keys per compute tile (= key scale block)
constexpr int kMaxKeyTiles = 4096; // key tiles per row whose scales the kernel holds in LDS
                                   // (L_k <= 262144); also bounds the routing words per row
                                   // to 64, which one register pair per wave holds

__device__ __forceinline__ float half_bits_to_float(uint16_t h) {
  _Float16 v;
  __builtin_memcpy(&v, &h, 2);
  return (float)v;
}

// The blockwise INT8 rule of Appendix C: scale d32 = absmax / 127 (IEEE FP32 division), code =
// round-half-even(x / d32).  x * rcp refined by one residual step (rcp = RN(1 / d32)) is the
// correctly rounded x / d32 for every FP16 x and FP16 block absmax (checked exhaustively), at 3
// instead of about 10 instructions.
__device__ __forceinline__ float quotient(float x, float d32, float rcp) {
  const float q0 = fmaf(x, rcp, 0.0f);   // x * rcp (an FMA takes x in FP16 directly)
  return fmaf(fmaf(-q0, d32, x), rcp, q0);
}

// The code of x as the low byte of the returned word: adding 1.5 * 2^23 rounds the quotient half
// to even into the low mantissa bits.  |x| <= absmax keeps it within 127 * (1 + 2^-23), so the
// clamp to [-127, 127] of the rule never acts.
__device__ __forceinline__ uint32_t code_word(float x, float d32, float rcp) {
  return __builtin_bit_cast(uint32_t, quotient(x, d32, rcp) + 12582912.0f);
}

// Low bytes of four code words, packed little-endian.
__device__ __forceinline__ uint32_t pack4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3) {
  const uint32_t lo = __builtin_amdgcn_perm(w1, w0, 0x0c0c0400u);
  const uint32_t hi = __builtin_amdgcn_perm(w3, w2, 0x0c0c0400u);
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// Lanes l and l^32 of a 32x32 accumulator column hold the same query row.  After
// v_permlane32_swap with both operands equal to x, the two results of every lane are
// {x[l], x[l ^ 32]} (in lane-dependent order), so their max / sum is the pair value.
__device__ __forceinline__ float pair_max(float x) {
  const int v = __builtin_bit_cast(int, x);
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return fmaxf(__builtin_bit_cast(float, (int)r[0]), __builtin_bit_cast(float, (int)r[1]));
}

__device__ __forceinline__ float pair_sum(float x) {
  const int v = __builtin_bit_cast(int, x);
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return __builtin_bit_cast(float, (int)r[0]) + __builtin_bit_cast(float, (int)r[1]);
}

// Cross-lane moves by DPP and lane swaps stay in the vector unit; a shuffle through LDS takes some
// 100 cycles per step.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ int dpp(int old, int x) {
  return __builtin_amdgcn_update_dpp(old, x, CTRL, ROW_MASK, 0xf, false);
}

// Maximum over the wave, in every lane.
__device__ __forceinline__ float wave_max(float x) {
  auto step = [](float a, int b) { return fmaxf(a, __builtin_bit_cast(float, b)); };
  auto bits = [](float a) { return __builtin_bit_cast(int, a); };
  x = step(x, dpp<0xB1>(bits(x), bits(x)));    // lane ^ 1
  x = step(x, dpp<0x4E>(bits(x), bits(x)));    // lane ^ 2
  x = step(x, dpp<0x141>(bits(x), bits(x)));   // the other half of 8 lanes, mirrored
  x = step(x, dpp<0x140>(bits(x), bits(x)));   // the other half of 16 lanes, mirrored
  const auto r = __builtin_amdgcn_permlane16_swap(bits(x), bits(x), false, false);
  x = fmaxf(__builtin_bit_cast(float, (int)r[0]), __builtin_bit_cast(float, (int)r[1]));
  return pair_max(x);
}

// Inclusive prefix sum over the wave.
__device__ __forceinline__ int wave_scan(int x) {
  x += dpp<0x111>(0, x);        // one lane up within 16
  x += dpp<0x112>(0, x);        // two
  x += dpp<0x114>(0, x);        // four
  x += dpp<0x118>(0, x);        // eight
  x += dpp<0x142, 0xa>(0, x);   // lane 15 of rows 0 and 2 into rows 1 and 3
  x += dpp<0x143, 0xc>(0, x);   // lane 31 into the upper half
  return x;
}

// Direct global -> LDS copy of 16 bytes per lane: lane l reads base + voff and writes LDS byte
// lds_addr + 16*l (base and lds_addr wave-uniform).  Completion is tracked by vmcnt like any
// vector load; it is issued as inline assembly so that the only waits on it are the explicit
// vmcnt waits of the caller (the compiler would otherwise wait for every copy in flight
// before any LDS read, whichever LDS bytes the copies write).
// base and lds_addr pass through readfirstlane (a no-op on values the compiler already holds in
// scalar registers), so that the scalar operands stay scalar where its uniformity analysis
// loses track of them.
// m0 is a register the compiler reserves (it warns that the clobber names one); the code it
// generates for these kernels never reads m0, so setting it here disturbs nothing else.
__device__ __forceinline__ void dma_16(const void* base, uint32_t voff, uint32_t lds_addr) {
  const uint64_t b = (uint64_t)(uintptr_t)base;
  const uint64_t bs = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32) |
                      (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint32_t ls = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_addr);
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(voff), "s"((const void*)(uintptr_t)bs), "s"(ls)
               : "m0");
}

// 32-bit LDS address of a __shared__ object.
template <typename T>
__device__ __forceinline__ uint32_t lds_addr_of(T* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)(p);
}

// Wait for every outstanding memory operation of the wave (vector, scalar, LDS).  Emitted with
// the builtin, so the compiler knows its own earlier loads are complete as well.
__device__ __forceinline__ void wait_all_memory() { __builtin_amdgcn_s_waitcnt(0); }

__device__ __forceinline__ uint4 ld_global_16(const void* p) {
  return *reinterpret_cast<const uint4*>(p);
}

__device__ __forceinline__ void st_lds_16(char* lds, int off, uint4 v) {
  *reinterpret_cast<uint4*>(lds + off) = v;
}

__device__ __forceinline__ uint4 ld_lds_16(const char* lds, int off) {
  return *reinterpret_cast<const uint4*>(lds + off);
}

__device__ __forceinline__ half8 as_half8(uint4 v) { return __builtin_bit_cast(half8, v); }
__device__ __forceinline__ i32x4 as_i32x4(uint4 v) { return __builtin_bit_cast(i32x4, v); }

__device__ __forceinline__ f32x16 mfma_f16(half8 a, half8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ i32x16 mfma_i8(i32x4 a, i32x4 b, i32x16 c) {
  return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}

// Scale of a block and what its quotients need.  An infinite scale divides every finite value to
// 0: the residual step is then taken with divisor 0, so that it adds nothing.
struct BlockScale {
  float div, rcp;
  uint16_t bits;   // the FP16-stored scale
  bool nonzero;
  __device__ __forceinline__ explicit BlockScale(float amax) {
    const float d32 = amax / 127.0f;   // IEEE FP32 division (compiled without fast-math)
    const bool inf = d32 == __builtin_huge_valf();
    nonzero = amax > 0.0f;
    rcp = nonzero ? 1.0f / d32 : 0.0f;
    div = inf ? 0.0f : d32;
    const _Float16 s = nonzero ? (_Float16)d32 : (_Float16)0.0f;   // RNE
    bits = __builtin_bit_cast(uint16_t, s);
  }
  // Code word of an FP16 value (low byte = code).  The clamp acts only on a NaN quotient (code
  // -127), which only a NaN or an infinity in the block produces.
  __device__ __forceinline__ uint32_t word(float x) const {
    const float q = __builtin_amdgcn_fmed3f(quotient(x, div, rcp), -127.0f, 127.0f);
    return nonzero ? __builtin_bit_cast(uint32_t, q + 12582912.0f) : 0u;
  }
  __device__ __forceinline__ void words(uint4 v, uint32_t (&w)[8]) const {
    const half8 h = as_half8(v);
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = word((float)h[e]);
  }
};

// Key (row of the 32x32 accumulator block) held by register r of lane l.
__device__ __forceinline__ int acc_row(int r, int lane) {
  return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
}

}  // namespace tilemix
