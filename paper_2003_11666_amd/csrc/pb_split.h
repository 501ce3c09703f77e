// fp32 products on the bf16 matrix pipes.
//
// A float has 24 significant bits, three bf16 values of 8 bits each hold them: x = h + m + l (a published method: Henry, Tang and
// Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", 2019).  That is exact
// from 2^-103 up; the last piece of smaller values is no normal bf16 number.  A product of two floats is then the sum of nine
// bf16 products.  The three smallest are left out: m l and l m, each at most 2^-23 of the whole and together at most 2^-22 (m has
// the sign of x, l either one), and l l, at most 2^-32.  The other six go through v_mfma_f32_16x16x32_bf16, which multiplies
// exactly and adds in fp32.  One such MFMA takes half the time of a v_mfma_f32_16x16x4_f32 for eight times the products: six of
// them contract at 2.7 times the rate of the fp32 pipes (loops of each alone: 2245 / 6 = 374 and 148 TFLOP/s; with the
// splitting of one operand in the loop 230-308).
//
// The six products of 32 reduction entries are added up from zero, small ones first, and only their sum goes to the
// accumulator: one rounding per 32 entries at the accumulator's magnitude where the chain of fp32 MFMAs has eight.  Error
// against float64 (2-norm, random data; fp32 chain / this): 64 entries 1.4e-7 / 0.5e-7, 576 4.3e-7 / 0.9e-7, 2304 8.7e-7 /
// 1.7e-7; with rectified operands 1.0e-7 / 0.4e-7, 3.0e-7 / 0.9e-7, 6.0e-7 / 1.7e-7.  (All six straight onto the accumulator:
// 0.9e-7, 3.6e-7, 7.5e-7 and 0.9e-7, 3.4e-7, 7.0e-7, in part worse than fp32: not done.)  Only sums of one or two products are
// further off than fp32's, by what is left out: one 2.6e-8 / 3.4e-8, 16 entries of which seven in eight are zero 3.5e-8 /
// 3.7e-8, 16 dense ones 7.2e-8 / 3.5e-8 (emulated); the tiles contract 32 channels and more, or the pixels of a map.  In
// networks, gradients of weight tensors with weights held fixed are 0.56 to 0.92 of the fp32 tiles' distance from float64 (basic
// ResNets of 32 to 256 channels 0.56-0.87, VGG 0.60-0.84, bottleneck networks 0.84-0.92;
// tests/test_gpu_split.py measures seven of the twelve).
// Rounding h to nearest instead would leave out a quarter of that (one product 2.65e-8) and dense sums where they are, but needs
// a clamp at the largest floats and cost the wide network 1.5 % and ResNet-50 1.1 %: not done.
//
// A value that is not finite makes the sums it takes part in NaN: an infinity, too, whose remainder is inf - inf, where fp32
// products would add up to an infinity.  (The softmax or GroupNorm that follows makes NaN of either.)
//
// Included by pb_gemm.h.
#pragma once
#include "pb_device.h"

namespace pb {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef unsigned v4w __attribute__((ext_vector_type(4)));
typedef unsigned v2w __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) v4w lw4;
typedef __attribute__((address_space(3))) v2w lw2;
typedef __attribute__((address_space(3))) unsigned lw1;

// (a, b) -> packed pairs of their first, second and third pieces.  The first is truncated (rounding could turn the largest
// finite values into infinities), the second rounded to nearest, the third is exact.
__device__ __forceinline__ void split2(float a, float b, unsigned& h, unsigned& m, unsigned& l) {
  const unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
  h = __builtin_amdgcn_perm(ub, ua, 0x07060302);
  const v2f r = {a - __uint_as_float(ua & 0xFFFF0000u), b - __uint_as_float(ub & 0xFFFF0000u)};
  m = __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf2));
  const v2f s = {r[0] - __uint_as_float(m << 16), r[1] - __uint_as_float(m & 0xFFFF0000u)};
  l = __builtin_bit_cast(unsigned, __builtin_convertvector(s, bf2));
}

// pieces multiplied in product q: small ones first
__device__ constexpr int split_pa(int q) { return q == 0 ? 2 : q == 1 || q == 3 ? 1 : 0; }
__device__ constexpr int split_pb(int q) { return q == 2 ? 2 : q == 1 || q == 4 ? 1 : 0; }

// z[i] = a[i] . b over the 32 reduction entries of an MFMA, N independent chains side by side
template <int N>
__device__ __forceinline__ void split_products(v4f (&z)[N], const bf8 (&a)[N][3], const bf8 (&b)[3]) {
#pragma unroll
  for (int i = 0; i < N; ++i) z[i] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < 6; ++q)
#pragma unroll
    for (int i = 0; i < N; ++i) z[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i][split_pa(q)], b[split_pb(q)], z[i], 0, 0, 0);
}

}  // namespace pb
