// A device math function in a text of its own, which only kernels that call it contain; shared with the interpreter like those of
// device_math.h, whose conventions it follows.
//
// gr_tanhf(x): hyperbolic tangent in binary32, within 1 ulp of the exact value.  Two pieces, both evaluated, one selected:
//   |x| <  0.625: tanh(x) = x + x z W(z), z = x^2, W of degree 5 (starts at -1/3)
//   |x| >= 0.625: tanh(x) = sign(x) (1 + 1 / d), d = -(1 + e) / 2, e = exp(2 a), a = min(|x|, 10).  e = 2^n + 2^n f Q(f): n = round(2 a log2(e)), f what the
//                rounding left, Q of degree 5 fitted to (2^f - 1) / f, so that the error of e is one of 0.42 of it at most.  What the sum d loses goes into
//                the residual of its hardware reciprocal r, and the result is put together from 1 + r, what that sum loses, and the
//                residual's share.  From |x| = 9.02 on the result is 1.
// Coefficients: weighted minimax fits (Lawson iteration) of the relative errors of tanh and of 2^f over |f| <= 1/2, rounded
// to binary32 one by one from the lowest power on, the others fitted again after each.  NaN compares false and takes the first piece.
// Errors over all floats of a range, largest in ulp and root mean square in units of 2^-24 (from a result of 0.5 on correct rounding is 1 / sqrt(12) = 0.289), this / the
// device library's tanhf: 0.25 to 0.5 0.63, 0.144 / 0.68, 0.145; 0.5 to 0.625 0.71, 0.245 / 0.78, 0.247; 0.625 to 0.75 0.59, 0.289 / 1.41, 0.450; 0.75 to 1
// 0.64, 0.291 / 1.17, 0.399; 1 to 1.5 0.59, 0.289 / 0.99, 0.321; 1.5 to 3 0.54, 0.289 / 0.66, 0.291.  With the hardware's power of two for e (from 0.75 on) 0.75 to 1
// had 1.47, 0.420, and the throughput of tanh alone was 1294 instead of 1236 per ns (a dense step of 4936 x 27 x 1131 62.6 us, 63.3 so).
// No branch: the device library's tanhf has two, and an epilogue over 64 accumulators of a lane waits for each chain in turn (that dense step: 3.4 us more).
GR_DEVICE_MATH_SOURCE(
static __device__ __forceinline__ float gr_tanhf(float x) {
  const float a = __builtin_fabsf(x);
  const float z = x * x;
  float w = 0x1.1a27fep-9f;
  w = __builtin_fmaf(w, z, -0x1.0c5ecep-7f);
  w = __builtin_fmaf(w, z, 0x1.63a55p-6f);
  w = __builtin_fmaf(w, z, -0x1.b9f188p-5f);
  w = __builtin_fmaf(w, z, 0x1.11107ap-3f);
  w = __builtin_fmaf(w, z, -0x1.555554p-2f);
  const float small = __builtin_fmaf(a * z, w, a);
  const float ac = __builtin_fminf(a, 10.0f);
  const float t = __builtin_fmaf(ac, 0x1.715476p+1f, 0x1.8p+23f);
  const float n = t - 0x1.8p+23f;
  const float f = __builtin_fmaf(ac, 0x1.4ae0cp-25f, __builtin_fmaf(ac, 0x1.715476p+1f, -n));
  float q = 0x1.416b5cp-13f;
  q = __builtin_fmaf(q, f, 0x1.5f083p-10f);
  q = __builtin_fmaf(q, f, 0x1.3b2dep-7f);
  q = __builtin_fmaf(q, f, 0x1.c6af7cp-5f);
  q = __builtin_fmaf(q, f, 0x1.ebfbdcp-3f);
  q = __builtin_fmaf(q, f, 0x1.62e43p-1f);
  const float s = __uint_as_float((__float_as_uint(t) << 23) + 0xbf000000u);
  const float sf = s * f;
  const float s1 = s - 0.5f;
  const float d = __builtin_fmaf(sf, q, s1);
  const float r = __builtin_amdgcn_rcpf(d);
  const float rest = __builtin_fmaf(-__builtin_fmaf(sf, q, s1 - d), r, __builtin_fmaf(-d, r, 1.0f));
  const float h = r + 1.0f;
  const float large = h + __builtin_fmaf(r, rest, (1.0f - h) + r);
  return __builtin_copysignf(a >= 0.625f ? large : small, x);
}
)
