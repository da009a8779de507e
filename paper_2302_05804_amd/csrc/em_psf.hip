// em_psf.hip -- super-resolved PSFs of Eq. (4) (arXiv:2302.05804, Sec. 2) by
// projected Adam, every frame's fit in one workgroup.
//
// For a frame-grid PSF f (Kf x Kf) the fit seeks h >= 0 (Kh x Kh, fine grid)
// minimising |D(h * g) - f|^2 + lambda |grad h|^2.  g is an isotropic Gaussian,
// so D(h * g) on f's stamp factors as A h A^T with A a Kf x Kh matrix:
//     A[I][a] = sum_{p = D I}^{D I + D - 1} g1(p - anchor - (a - ch)),
// g1 the 1-D Gaussian (unit sum over |d| <= ceil(4 sigma)), anchor = D (Kf-1)/2
// the fine pixel that carries h's centre ch.  Rows of h*g that fall outside
// the D Kf fine stamp belong to no block I and drop out, as in the definition.
// One Adam step is then four small products that stay in LDS:
//     T = h A^T,  rho = A T - f,  U = rho A,  grad = 2 A^T U + 2 lambda L h,
// L the 5-point Laplacian of h extended by zeros (the derivative of the sum
// of squared forward differences), followed by Adam's moment update
// (Kingma & Ba, 2015, Algorithm 1), the step lr max(f) decay^((k-1)/(S-1))
// and the projection max(h, 0).
//
// Layout: one workgroup per frame; A, A^T, f, rho, T^T, U^T and two buffers of
// h (read one, write the other) in LDS, each padded with zeros to KP x KP
// (KP the multiple of 16 at or above Kf and Kh).  The products run on the
// matrix cores in binary32 (v_mfma_f32_16x16x4f32), one 16 x 16 output block
// per wave, so a workgroup has (KP/16)^2 waves; each lane reads 16-byte runs of
// its row of the left operand and of the transposed right operand, and the
// products that feed another one store their result transposed (T^T, U^T) so
// that the next product reads it the same way.  A lane keeps the Adam moments
// of the four pixels of its accumulator for the whole run.  One barrier
// follows each product.  Arithmetic is binary32 except the schedule scalars
// and the final objective (binary64).
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "em_device.h"
#include "em_internal.h"

namespace em {
namespace {

typedef __attribute__((ext_vector_type(4))) float psf_f32x4;

// Every matrix is held padded to KP x KP (KP = 16, 32, 48 or 64, the multiple of
// 16 at or above Kf and Kh) with zeros outside its Kf / Kh extent, rows PP
// floats apart.  One wave per 16 x 16 output block.
template <int KP>
struct PsfShape {
  static constexpr int NB = KP / 16;          // output blocks per side
  static constexpr int NW = NB * NB;          // waves (one block each)
  static constexpr int NT = 64 * NW;
  static constexpr int KS = KP / 4;           // k values per lane group
  static constexpr int PP = KP + 4;           // row pitch (floats)
  static constexpr int MAT = KP * PP;         // floats per matrix
  static constexpr int NMAT = 8;              // A, At, F, R, Tt, Ut, H0, H1
};

// A lane's share of one row of an operand: the k values of its lane group.
template <int KP>
struct PsfRow {
  float4 v[PsfShape<KP>::KS / 4];
  // row 16 blk + lane%16 of a matrix
  __device__ void load(const float* M, int blk) {
    using S = PsfShape<KP>;
    const int lane = threadIdx.x & 63;
    const float* p = M + (16 * blk + (lane & 15)) * S::PP + (lane >> 4) * S::KS;
#pragma unroll
    for (int c = 0; c < S::KS / 4; ++c) v[c] = *reinterpret_cast<const float4*>(p + 4 * c);
  }
};

// C block of L * R with R given transposed (Rt[n][k]): lane i supplies L[i%16][k] and
// Rt[i%16][k] of the block's rows for the k values of its lane group g = i/16, k
// in [g KS, g KS + KS).  The matrix instruction sums its four lane groups, so every
// k is taken once.  Returns C[4 g + j][i%16] of the block in element j.
template <int KP>
__device__ inline psf_f32x4 psf_block(const PsfRow<KP>& L, const PsfRow<KP>& Rt) {
  // four independent accumulators, so that consecutive matrix instructions do
  // not wait for each other's results
  psf_f32x4 acc[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[e] = psf_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < PsfShape<KP>::KS / 4; ++c) {
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(L.v[c].x, Rt.v[c].x, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(L.v[c].y, Rt.v[c].y, acc[1], 0, 0, 0);
    acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(L.v[c].z, Rt.v[c].z, acc[2], 0, 0, 0);
    acc[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(L.v[c].w, Rt.v[c].w, acc[3], 0, 0, 0);
  }
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// The rows of A and A^T that a wave multiplies by in every step (its block's row
// bm and column bn).  Up to 48 x 48 they stay in registers for the whole run, which
// leaves one operand of each product to LDS (16 x 43^2, 2000 steps: 8.24 -> 7.80 ms with
// the neighbours of h read early and the shared divisors); at
// 64 x 64, with 16 waves of 128 registers, they would spill and are read each time.
template <int KP>
struct PsfFixed {
  static constexpr bool HELD = KP <= 48;
  PsfRow<KP> rows[HELD ? 4 : 1];   // A bm, A bn, A^T bm, A^T bn
  const float *A, *At;
  int bm, bn;
  psf_f32x4 f;                     // f at the lane's four residual pixels
  __device__ PsfFixed(const float* A_, const float* At_, const float* F, int bm_, int bn_)
      : A(A_), At(At_), bm(bm_), bn(bn_) {
    using S = PsfShape<KP>;
    if constexpr (HELD) {
      rows[0].load(A, bm);
      rows[1].load(A, bn);
      rows[2].load(At, bm);
      rows[3].load(At, bn);
    }
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < 4; ++j) f[j] = F[(16 * bm + 4 * (lane >> 4) + j) * S::PP + 16 * bn + (lane & 15)];
  }
  template <int WHICH>
  __device__ PsfRow<KP> row() const {
    if constexpr (HELD) {
      return rows[WHICH];
    } else {
      PsfRow<KP> v;
      v.load(WHICH < 2 ? A : At, WHICH % 2 == 0 ? bm : bn);
      return v;
    }
  }
};

// Tt = (h A^T)^T, then R = A T - F (pads stay 0: A and F are 0 there).
template <int KP>
__device__ inline void psf_residual(const PsfFixed<KP>& X, const float* H, float* Tt, float* R,
                                    int bm, int bn) {
  using S = PsfShape<KP>;
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  PsfRow<KP> v;
  v.load(H, bm);
  const psf_f32x4 t = psf_block<KP>(v, X.template row<1>());                 // T[a][J], a = 16bm+4g+j
  *reinterpret_cast<psf_f32x4*>(Tt + (16 * bn + r) * S::PP + 16 * bm + 4 * g) = t;
  __syncthreads();
  v.load(Tt, bn);
  const psf_f32x4 m = psf_block<KP>(X.template row<0>(), v);                 // M[I][J], I = 16bm+4g+j
#pragma unroll
  for (int j = 0; j < 4; ++j) R[(16 * bm + 4 * g + j) * S::PP + 16 * bn + r] = m[j] - X.f[j];
  __syncthreads();
}

// Correctly rounded v / c for a divisor shared by many quotients, from its correctly
// rounded reciprocal rc and two fused steps (Markstein, 1990); a divisor whose
// significand is all ones, where those need not round correctly, divides.
struct PsfDivisor {
  float c, rc;
  bool plain;
  __device__ explicit PsfDivisor(float c_)
      : c(c_), rc(1.f / c_), plain((__float_as_uint(c_) & 0x7fffffu) == 0x7fffffu) {}
  __device__ float divide(float v) const {
    // c is in [2^-24, 1]: inside these bounds quotient and remainder are normal and
    // finite; outside, and for infinities and NaN, divide
    const float a = fabsf(v);
    if (plain || !(a > 1e-30f && a < 1e30f)) return v / c;
    const float q = v * rc;
    return fmaf(fmaf(-q, c, v), rc, q);
  }
};

template <int KP>
__global__ __launch_bounds__(PsfShape<KP>::NT) void psf_fit_kernel(PsfParams P,
                                                                  const float* __restrict__ f,
                                                                  const float* __restrict__ h0,
                                                                  float* __restrict__ hout,
                                                                  double* __restrict__ objective) {
  using S = PsfShape<KP>;
  extern __shared__ float4 psf_smem4[];
  float* sm = reinterpret_cast<float*>(psf_smem4);
  float* A = sm;
  float* At = A + S::MAT;
  float* F = At + S::MAT;
  float* R = F + S::MAT;
  float* Tt = R + S::MAT;
  float* Ut = Tt + S::MAT;
  float* Hc = Ut + S::MAT;
  float* Hn = Hc + S::MAT;
  double* red = reinterpret_cast<double*>(Hn + S::MAT);
  const int kf = P.kf, kh = P.kh, D = P.D;
  const int t = blockIdx.x, tid = threadIdx.x;
  const int w = tid >> 6, lane = tid & 63, g = lane >> 4, r = lane & 15;
  const int bm = w / S::NB, bn = w % S::NB;
  for (int i = tid; i < S::NMAT * S::MAT; i += S::NT) sm[i] = 0.f;
  __syncthreads();

  // A[I][a] = sum over the D fine rows of coarse row I of g1(p - anchor - (a - ch)),
  // g1 the unit-sum 1-D Gaussian (binary64, rounded once); A^T beside it
  const int ch = (kh - 1) / 2, anchor = D * ((kf - 1) / 2);
  const double sg = (double)P.sigma;
  const int rg = sg > 0.0 ? (int)ceil(4.0 * sg) : 0;
  double Z = 0.0;
  for (int d = -rg; d <= rg; ++d) Z += sg > 0.0 ? exp(-(double)(d * d) / (2.0 * sg * sg)) : 1.0;
  for (int q = tid; q < kf * kh; q += S::NT) {
    const int I = q / kh, a = q % kh;
    double v = 0.0;
    for (int p = D * I; p < D * I + D; ++p) {
      const int d = p - anchor - (a - ch);
      if (d >= -rg && d <= rg) v += sg > 0.0 ? exp(-(double)(d * d) / (2.0 * sg * sg)) : 1.0;
    }
    A[I * S::PP + a] = (float)(v / Z);
    At[a * S::PP + I] = (float)(v / Z);
  }
  // f, its maximum, and the start h
  const float* ft = f + (size_t)t * kf * kf;
  float fmax = 0.f;
  for (int q = tid; q < kf * kf; q += S::NT) {
    const float v = ft[q];
    F[(q / kf) * S::PP + q % kf] = v;
    fmax = fmaxf(fmax, v);
  }
  for (int q = tid; q < kh * kh; q += S::NT) {
    const int a = q / kh, b = q % kh;
    float v;
    if (h0) {
      v = h0[(size_t)t * kh * kh + q];
    } else {
      const int p = a - ch + anchor, c2 = b - ch + anchor;
      v = 0.f;
      if (p >= 0 && p < D * kf && c2 >= 0 && c2 < D * kf)
        v = fmaxf(ft[(p / D) * kf + c2 / D] / (float)(D * D), 0.f);
    }
    Hc[a * S::PP + b] = v;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) fmax = fmaxf(fmax, __shfl_xor(fmax, off, 64));
  if (lane == 0) red[w] = (double)fmax;
  __syncthreads();
  for (int i = 0; i < S::NW; ++i) fmax = fmaxf(fmax, (float)red[i]);
  __syncthreads();

  // Adam state of the lane's four pixels (a = 16 bm + 4 g + j, b = 16 bn + r)
  float m1[4] = {0.f, 0.f, 0.f, 0.f}, m2[4] = {0.f, 0.f, 0.f, 0.f};
  // step k uses lr max(f) decay^((k-1)/(S-1)): a running product in binary64
  double lrk_d = (double)P.lr * (double)fmax;
  const double rdec = P.S > 1 ? exp(log((double)P.decay) / (double)(P.S - 1)) : 1.0;
  const float b1 = P.b1, b2 = P.b2, eps = P.eps, lam2 = 2.f * P.lam;
  const int b = 16 * bn + r, a0 = 16 * bm + 4 * g;
  double b1k = 1.0, b2k = 1.0;
  const PsfFixed<KP> X(A, At, F, bm, bn);
  float hv[4];   // h at the lane's four pixels
#pragma unroll
  for (int j = 0; j < 4; ++j) hv[j] = Hc[(a0 + j) * S::PP + b];
  for (int k = 1; k <= P.S; ++k) {
    // h around the lane's pixels (h is 0 in the pads)
    const float up = a0 > 0 ? Hc[(a0 - 1) * S::PP + b] : 0.f;
    const float down = a0 + 4 < KP ? Hc[(a0 + 4) * S::PP + b] : 0.f;
    float left[4], right[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      left[j] = b > 0 ? Hc[(a0 + j) * S::PP + b - 1] : 0.f;
      right[j] = Hc[(a0 + j) * S::PP + b + 1];
    }
    b1k *= (double)b1;
    b2k *= (double)b2;
    const float lrk = (float)lrk_d;
    lrk_d *= rdec;
    const PsfDivisor c1((float)(1.0 - b1k)), c2((float)(1.0 - b2k));
    psf_residual<KP>(X, Hc, Tt, R, bm, bn);
    // U = rho A, stored transposed (Ut[b][I])
    PsfRow<KP> v;
    v.load(R, bm);
    const psf_f32x4 u = psf_block<KP>(v, X.template row<3>());
    *reinterpret_cast<psf_f32x4*>(Ut + (16 * bn + r) * S::PP + 16 * bm + 4 * g) = u;
    __syncthreads();
    // gradient 2 A^T U + 2 lambda L h, Adam, projection
    v.load(Ut, bn);
    const psf_f32x4 gd = psf_block<KP>(X.template row<2>(), v);
    const float old[4] = {hv[0], hv[1], hv[2], hv[3]};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int a = a0 + j;
      float hn = 0.f;
      if (a < kh && b < kh) {
        const float nb = (j > 0 ? old[j > 0 ? j - 1 : 0] : up) + (j < 3 ? old[j < 3 ? j + 1 : 3] : down) +
                         left[j] + right[j];
        const float gr = 2.f * gd[j] + lam2 * (4.f * old[j] - nb);
        m1[j] = b1 * m1[j] + (1.f - b1) * gr;
        m2[j] = b2 * m2[j] + (1.f - b2) * gr * gr;
        const float step = lrk * c1.divide(m1[j]) / (sqrtf(c2.divide(m2[j])) + eps);
        hn = fmaxf(old[j] - step, 0.f);
      }
      hv[j] = hn;
      Hn[a * S::PP + b] = hn;
    }
    __syncthreads();
    float* tmp = Hc;
    Hc = Hn;
    Hn = tmp;
  }

  float* ht = hout + (size_t)t * kh * kh;
  for (int q = tid; q < kh * kh; q += S::NT) ht[q] = Hc[(q / kh) * S::PP + q % kh];
  if (objective) {
    psf_residual<KP>(X, Hc, Tt, R, bm, bn);
    double part = 0.0;
    for (int q = tid; q < kf * kf; q += S::NT) {
      const double rr = (double)R[(q / kf) * S::PP + q % kf];
      part += rr * rr;
    }
    double pen = 0.0;
    auto hat = [&](int i, int j) -> double {
      return (i >= 0 && i < kh && j >= 0 && j < kh) ? (double)Hc[i * S::PP + j] : 0.0;
    };
    for (int q = tid; q < (kh + 1) * kh; q += S::NT) {
      // pair (i, i+1) in column j, and pair (i, i+1) along row j
      const int i = q / kh - 1, j = q % kh;
      const double dv = hat(i + 1, j) - hat(i, j);
      const double dh = hat(j, i + 1) - hat(j, i);
      pen += dv * dv + dh * dh;
    }
    const double tot = block_sum<S::NT>(part + (double)P.lam * pen, red);
    if (tid == 0) objective[t] = tot;
  }
}

inline int psf_kp(int kf, int kh) { return 16 * ((std::max(kf, kh) + 15) / 16); }

template <int KP>
hipError_t launch_kp(const PsfParams& P, const float* f, const float* h0, float* h,
                     double* objective, hipStream_t s) {
  using S = PsfShape<KP>;
  const size_t lds = (size_t)S::NMAT * S::MAT * sizeof(float) + S::NW * sizeof(double);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&psf_fit_kernel<KP>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(psf_fit_kernel<KP>, dim3(P.n), dim3(S::NT), lds, s, P, f, h0, h, objective);
  return hipGetLastError();
}

}  // namespace

size_t psf_lds_bytes(int kf, int kh) {
  const int kp = psf_kp(kf, kh);
  return (size_t)8 * kp * (kp + 4) * sizeof(float) + (size_t)(kp / 16) * (kp / 16) * sizeof(double);
}

hipError_t launch_psf_fit(const PsfParams& P, const float* f, const float* h0, float* h,
                          double* objective, hipStream_t s) {
  switch (psf_kp(P.kf, P.kh)) {
    case 16: return launch_kp<16>(P, f, h0, h, objective, s);
    case 32: return launch_kp<32>(P, f, h0, h, objective, s);
    case 48: return launch_kp<48>(P, f, h0, h, objective, s);
    case 64: return launch_kp<64>(P, f, h0, h, objective, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace em
