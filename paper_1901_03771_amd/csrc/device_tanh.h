// A device math function in a text of its own, which only kernels that call it contain; shared with the interpreter like those of
// device_math.h, whose conventions it follows.
//
// gr_tanhf(x): hyperbolic tangent in binary32, within 2 ulp of the exact value (largest 1.48 ulp, relative error in the 2-norm
// 2.52e-8 for normally distributed arguments; the device library's tanhf 1.41 and 2.65e-8).  Two pieces, both evaluated, one selected:
//   |x| <  0.75: tanh(x) = x + x z W(z), z = x^2, W of degree 5 (starts at -1/3; the same kind of fit as erf's)
//   |x| >= 0.75: tanh(x) = sign(x) (1 - 2 / (1 + e)), e = exp(2 a), a = min(|x|, 10): the hardware's power of two of p = round(2 a log2(e))
//                times 1 + f, f = what the rounding left times ln(2); the hardware's reciprocal after one Newton step whose residual
//                does not depend on the rounding of 1 + e.  From |x| = 9.02 on the result is 1.
// NaN compares false and takes the first piece.  No branch: the device library's tanhf has two, and an epilogue over 64 accumulators
// of a lane waits for each chain in turn (first product of a dense layer of 4936 x 27 x 1131 29.8 -> 26.4 us, 3024 x 47 x 1458 31.4 -> 28.4).
GR_DEVICE_MATH_SOURCE(
static __device__ __forceinline__ float gr_tanhf(float x) {
  const float a = __builtin_fabsf(x);
  const float z = x * x;
  float w = 0x1.c753bcp-10f;
  w = __builtin_fmaf(w, z, -0x1.f5d368p-8f);
  w = __builtin_fmaf(w, z, 0x1.5f785ap-6f);
  w = __builtin_fmaf(w, z, -0x1.b97d3cp-5f);
  w = __builtin_fmaf(w, z, 0x1.110db8p-3f);
  w = __builtin_fmaf(w, z, -0x1.55554ap-2f);
  const float small = __builtin_fmaf(a * z, w, a);
  const float ac = __builtin_fminf(a, 10.0f);
  const float p = ac * 0x1.715476p+1f;
  const float f = __builtin_fmaf(ac, 0x1.4ae0cp-25f, __builtin_fmaf(ac, 0x1.715476p+1f, -p)) * 0x1.62e43p-1f;
  const float e0 = __builtin_amdgcn_exp2f(p);
  const float e = __builtin_fmaf(e0, f, e0);
  const float r = __builtin_amdgcn_rcpf(e + 1.0f);
  const float large = __builtin_fmaf(-2.0f, __builtin_fmaf(__builtin_fmaf(-e, r, 1.0f - r), r, r), 1.0f);
  return __builtin_copysignf(a >= 0.75f ? large : small, x);
}
)
