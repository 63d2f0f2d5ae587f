// Field product (FP64), eqs. sc2-sc5 in factorised form, on the FP64 matrix cores:
//   F_p = X_p mu_vv - mu_oo X_p + sqrt2 mu_ov c0_p      (p = 0, 1: the real and imaginary planes)
// plus per-block partial sums g_p = sqrt2 <mu_ov, X_p>, <X, F> and |X|^2.
// One block of 256 threads per (RHS, 16 x 16 tile of (i, a), plane): each of its four waves takes a quarter
// of the contraction index (b for X mu_vv, j for mu_oo X) with v_mfma_f64_16x16x4, operands read straight
// from memory, the next four K steps' while four are multiplied (from clamped places, out-of-range ones
// replaced by zero afterwards: a condition on a load would make it wait for the one before it); the
// quarters are added in a fixed order through LDS.  Bound by the chain of these loads, not by their bytes
// or the matrix cores, so a launch that reads the same X and leaves the chip partly idle carries these
// blocks beside its own (the first Coulomb product, the small problems' partial sums).
// f64 16x16x4 operand layout: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; the result
// element t of lane l is D[4 t + l / 16][l % 16].
#pragma once
#include "common.h"

namespace rttda {

typedef double d4v __attribute__((ext_vector_type(4)));

// acc += sgn sum_{k in [k0, k1)} A[k] B[k] over K steps of 4; la(k), lb(k): this lane's operands
template <typename LA, typename LB>
__device__ __forceinline__ void field_part(d4v &acc, int k0, int k1, int g, LA la, LB lb) {
  if (k0 >= k1) return;
  double x[2][4], y[2][4];
  auto load = [&](int b, int k) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int kk = min(k + 4 * u + g, k1 - 1);
      x[b][u] = la(kk);
      y[b][u] = lb(kk);
    }
  };
  auto mul = [&](int b, int k) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool ok = k + 4 * u + g < k1;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ok ? x[b][u] : 0.0, ok ? y[b][u] : 0.0, acc, 0, 0, 0);
    }
  };
  load(0, k0);
  for (int k = k0; k < k1; k += 32) {
    if (k + 16 < k1) load(1, k + 16);
    mul(0, k);
    if (k + 16 >= k1) break;
    if (k + 32 < k1) load(0, k + 32);
    mul(1, k + 16);
  }
}

__device__ __forceinline__ void field_block(const FieldArgs &f, int block) {
  __shared__ double red[4][4][64];
  if (block == 0 && threadIdx.x == 0 && f.st->pend) {
    f.st->step += 1;  // the step the last RK4 epilogue closed (nothing else in this launch reads it)
    f.st->pend = 0;
  }
  const int o = f.o, v = f.v;
  const int fa = field_blocks_a(v), nbf = field_blocks(o, v);
  const int r = block / nbf, p = block % nbf & 1, tile = block % nbf >> 1;
  const int i0 = tile / fa * FT_I, a0 = tile % fa * FT_A;
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int m = lane & 15, g = lane >> 4;
  const size_t ov = (size_t)o * v;
  const double *Xp = f.X + ((size_t)r * 2 + p) * ov;
  const double *moo_r = f.moo + (size_t)r * o * o;
  const double *mov_r = f.mov + (size_t)r * ov;
  const double *mvv_r = f.mvv + (size_t)r * v * v;
  const int i = min(i0 + m, o - 1), a = min(a0 + m, v - 1);  // this lane's operand row (A) and column (B)
  const bool iok = i0 + m < o, aok = a0 + m < v;
  d4v acc = {0.0, 0.0, 0.0, 0.0};
  {  // X_p mu_vv over b in this wave's quarter
    const int kq = (((v + 3) / 4) + 3) / 4 * 4, k0 = q * kq;
    field_part(acc, k0, min(v, k0 + kq), g,
               [&](int b) { const double t = Xp[(size_t)i * v + b]; return iok ? t : 0.0; },
               [&](int b) { const double t = mvv_r[(size_t)b * v + a]; return aok ? t : 0.0; });
  }
  {  // - mu_oo X_p over j in this wave's quarter
    const int kq = (((o + 3) / 4) + 3) / 4 * 4, k0 = q * kq;
    field_part(acc, k0, min(o, k0 + kq), g,
               [&](int j) { const double t = moo_r[(size_t)i * o + j]; return iok ? -t : 0.0; },
               [&](int j) { const double t = Xp[(size_t)j * v + a]; return aok ? t : 0.0; });
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) red[q][t][lane] = acc[t];
  __syncthreads();
  // wave 0: add the quarters, + sqrt2 mu_ov c0_p, outputs, partial sums
  if (q != 0) return;
  const double c0p = f.X0[2 * r + p];
  double pg = 0.0, ptr = 0.0, pnr = 0.0;
  double *Fp = f.F + ((size_t)r * 2 + p) * ov;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int ii = i0 + 4 * t + g, aa = a0 + m;
    if (ii < o && aa < v) {
      const size_t ia = (size_t)ii * v + aa;
      const double mo = mov_r[ia], x = Xp[ia];
      const double s = ((red[0][t][lane] + red[1][t][lane]) + (red[2][t][lane] + red[3][t][lane])) + SQRT2 * mo * c0p;
      Fp[ia] = s;
      pg += SQRT2 * mo * x;
      ptr += x * s;
      pnr += x * x;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    pg += __shfl_xor(pg, off, 64);
    ptr += __shfl_xor(ptr, off, 64);
    pnr += __shfl_xor(pnr, off, 64);
  }
  if (lane == 0) {
    double *out = f.part + (size_t)block * PART_STRIDE;
    out[0] = p == 0 ? pg : 0.0;
    out[1] = p == 1 ? pg : 0.0;
    out[2] = ptr;
    out[3] = pnr;
  }
}

}  // namespace rttda
