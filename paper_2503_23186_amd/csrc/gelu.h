// GELU and its derivative as the epilogues of the dense products compute them, in fp32.
#pragma once

// gelu(u) = u/2 (1 + erf(u / sqrt 2)) with erf(t) = t P(t^2) on |t| <= 3, P of degree 8 fitted to erf(t) / t
// (least squares on Chebyshev nodes, weighted so that the absolute error of erf is what is minimised;
// evaluated in fp32: 2.1e-5), and t clamped to that range beyond it (1 - erf(3) = 2.2e-5).  Fourteen
// full-rate instructions and no reciprocal or exponential: the epilogue runs on the vector ALU with
// nothing to overlap it, and the ~25 instructions per element of an erfc-based form were a tenth of the
// launch.  Absolute error of gelu below 4.4e-5 for every u, a hundredth of what the bf16 store rounds off.
__device__ __forceinline__ float gelu_f(float u) {
  const float t = fminf(fmaxf(u * 0.70710678118654752f, -3.0f), 3.0f);
  const float s = t * t;
  float p = 3.912539981e-08f;
  p = fmaf(p, s, -1.883036475e-06f);
  p = fmaf(p, s, 4.008835822e-05f);
  p = fmaf(p, s, -5.029218737e-04f);
  p = fmaf(p, s, 4.196857568e-03f);
  p = fmaf(p, s, -2.499890141e-02f);
  p = fmaf(p, s, 1.109308004e-01f);
  p = fmaf(p, s, -3.752196431e-01f);
  p = fmaf(p, s, 1.128250599e+00f);
  const float hu = 0.5f * u;
  return fmaf(hu, t * p, hu);
}

// gelu'(u) = Phi(u) + u phi(u).  With a = |u|, E = exp(-a^2 / 2) and R the scaled complementary error function,
// R(x) = exp(x^2) erfc(x):  Phi(-a) = E R(a / sqrt 2) / 2, so gelu'(a) = 1 + E W, gelu'(-a) = -E W with
// W = a S - 1/2 and S = 1 / sqrt(2 pi) + (1 - R(a / sqrt 2)) / (2 a), which is smooth and between 0.4 and 0.8: a
// polynomial of degree 6 in 1 / (1 + 0.26 a), least squares weighted towards a minimax fit of E W (7e-10).  What is
// near 1/2 or 1 is thus rounded once.  Over all bf16 u, on the device: largest error 9.4e-8, rms 6.5e-9 (with erff
// and the terms added one by one 1.27e-7 and 8.7e-9).
__device__ __forceinline__ float gelu_grad_f(float u) {
  const float a = fabsf(u);
  const float e = __builtin_amdgcn_exp2f((u * -0.72134752044448170f) * u);
  const float t = __builtin_amdgcn_rcpf(fmaf(a, 0.26f, 1.0f));
  float s = -4.526899010e-02f;
  s = fmaf(s, t, 1.763568223e-01f);
  s = fmaf(s, t, -1.134966835e-01f);
  s = fmaf(s, t, 1.786069125e-01f);
  s = fmaf(s, t, 6.623491645e-02f);
  s = fmaf(s, t, 1.370640099e-01f);
  s = fmaf(s, t, 3.983875811e-01f);
  const float w = fmaf(a, s, -0.5f);
  return fmaf(e, u < 0.f ? -w : w, u < 0.f ? 0.f : 1.0f);
}
