// Exchanges between the lanes of a wave, sums of a few products, and the candidates of an argmax.  Shared by the decode
// kernels and by the wide passes, which reproduce their sums bit for bit.
#ifndef LS_LANES_H_
#define LS_LANES_H_

#include <hip/hip_runtime.h>

// Cross-lane exchanges on the vector ALU: DPP controls within a row of 16 lanes and the lane swaps
// across rows, a few cycles each, where __shfl_xor goes through the LDS crossbar (an LDS round trip
// per step).  All 64 lanes must be active.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_xor1(float v) { return dpp_f<0xB1>(v); }    // quad_perm [1,0,3,2]
__device__ __forceinline__ float lane_xor2(float v) { return dpp_f<0x4E>(v); }    // quad_perm [2,3,0,1]
__device__ __forceinline__ float lane_xor8(float v) { return dpp_f<0x128>(v); }   // row_ror:8
// value of the lane 7 - i of the same group of 8: equals lane i ^ 4 when the four lanes of every quad agree
__device__ __forceinline__ float lane_half_mirror(float v) { return dpp_f<0x141>(v); }
// Combines the two rows of a row pair / the two halves of the wave; both partners get op(even, odd).
// The swap instruction exchanges halves of two registers; it is written as inline assembly (with the
// two wait states it needs after a vector write of its operands) because the builtin, given the
// same value twice, came back with one register for both results.
template <typename Op>
__device__ __forceinline__ float rows_combine16(float v, Op op) {
  float a = v, b = v;
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
  return op(a, b);
}
template <typename Op>
__device__ __forceinline__ float rows_combine32(float v, Op op) {
  float a = v, b = v;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
  return op(a, b);
}
// All-reduce over the wave of a value that is already the same in the four lanes of every quad.
template <typename Op>
__device__ __forceinline__ float wave_combine_quads(float v, Op op) {
  v = op(v, lane_half_mirror(v));
  v = op(v, lane_xor8(v));
  v = rows_combine16(v, op);
  return rows_combine32(v, op);
}
// Sum over the wave on the vector ALU; every lane gets the total.  All 64 lanes must be active.
__device__ __forceinline__ float wave_sum(float v) {
  v += lane_xor1(v);
  v += lane_xor2(v);
  return wave_combine_quads(v, [](float a, float b) { return a + b; });
}

// Sums of products that the wide passes share with the decode kernels, with the fused steps written out: in a * x + b * y
// either product may be the one that is rounded, and what a compiler picks may change with the code around it.
__device__ __forceinline__ float sum2(float a, float x, float b, float y) { return __builtin_fmaf(a, x, b * y); }
__device__ __forceinline__ float sum_of_squares(float x, float y, float z, float w) {
  return __builtin_fmaf(w, w, __builtin_fmaf(z, z, sum2(x, x, y, y)));
}
// (a, b) turned by the angle with cosine c and sine s.
__device__ __forceinline__ void rotate_pair(float a, float b, float c, float s, float& lo, float& hi) {
  lo = sum2(a, c, -b, s);
  hi = sum2(a, s, b, c);
}

// Candidate of a row's argmax: highest value, its index (the lowest on ties), and the runner-up's value.
struct Best { float v1; int i1; float v2; };
__device__ __forceinline__ Best best_merge(const Best& a, const Best& b) {
  const bool aw = (a.v1 > b.v1) || (a.v1 == b.v1 && a.i1 < b.i1);
  Best r;
  r.v1 = aw ? a.v1 : b.v1;
  r.i1 = aw ? a.i1 : b.i1;
  r.v2 = fmaxf(aw ? a.v2 : b.v2, aw ? b.v1 : a.v1);
  return r;
}
__device__ __forceinline__ Best best_shfl_xor(const Best& a, int mask) {
  Best b;
  b.v1 = __shfl_xor(a.v1, mask);
  b.i1 = __shfl_xor(a.i1, mask);
  b.v2 = __shfl_xor(a.v2, mask);
  return b;
}

#endif
