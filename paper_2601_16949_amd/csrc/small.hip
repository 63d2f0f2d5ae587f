// Small problems, where a step is bound by chains of latencies and by the gaps between dependent launches
// rather than by any bandwidth (o v up to 2048, at most 64 right-hand sides): each RK4 stage is two launches,
// this one and the stage update.
//  * k_small_2e: the Coulomb and exchange parts of sigma for one slice and a range of Q in one
//    workgroup.  Every Q term of J = 2 sum_Q B^Q <B^Q, X> needs only its own d_Q, so no grid-wide
//    step separates the two Coulomb products here; the exchange term B_oo^Q X B_vv^Q goes through
//    the workgroup's LDS (FP32 FMA: at these sizes the matrix cores would idle on latency anyway).
//    Each workgroup writes one partial slab J - c_x K, the FP32 sum of those of its m ranges of Q; a call with
//    few of the context's right-hand sides takes a workgroup per range, and the stage update adds the ranges
//    so, with the same bits.  Further workgroups of the launch form the field product.
#include <type_traits>

#include "common.h"
#include "field.h"

namespace rttda {
namespace {

__device__ __forceinline__ float bload(const float *p, size_t i) { return p[i]; }
__device__ __forceinline__ float bload(const __hip_bfloat16 *p, size_t i) { return __bfloat162float(p[i]); }

__device__ __forceinline__ float wsum(float x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

constexpr int EPT2 = SMALL_OV_MAX / 256;  // elements per thread of k_small_2e

// sum_k x[k sx] y[k sy] for k < n as four interleaved partial sums (four independent LDS reads and
// FMAs in flight instead of one dependent chain), added in a fixed order
__device__ __forceinline__ float dot4(const float *x, int sx, const float *y, int sy, int n) {
  float a0 = 0, a1 = 0, a2 = 0, a3 = 0;
  int k = 0;
#pragma unroll 4
  for (; k + 4 <= n; k += 4) {
    a0 += x[k * sx] * y[k * sy];
    a1 += x[(k + 1) * sx] * y[(k + 1) * sy];
    a2 += x[(k + 2) * sx] * y[(k + 2) * sy];
    a3 += x[(k + 3) * sx] * y[(k + 3) * sy];
  }
  for (; k < n; ++k) a0 += x[k * sx] * y[k * sy];
  return (a0 + a1) + (a2 + a3);
}

// The first field.blocks workgroups form the field product, the others are (split, slice); 256 threads;
// dynamic LDS: X slice, W, B_vv^Q and B_oo^Q (floats).  All of a Q's factors are loaded together (from
// clamped places), and the next Q's while this one is multiplied: a loop of loads and LDS writes waits for
// each load in turn.
template <typename TB, bool RNG>
__global__ __launch_bounds__(256) void k_small_2e(const TB *__restrict__ Bov, const TB *__restrict__ Boo,
                                                  const TB *__restrict__ Bvv, const float *__restrict__ X, int o,
                                                  int v, int nq, int ns, int nsplit, int m, float cx,
                                                  float *__restrict__ P, FieldArgs f) {
  if ((int)blockIdx.x < f.blocks) {
    field_block(f, blockIdx.x);
    return;
  }
  constexpr int UV = 8, UO = 2;  // values of B_vv^Q and B_oo^Q per thread held ahead; the rest is read in place
  extern __shared__ float sm2[];
  __shared__ float red[4];
  const int lb = (int)blockIdx.x - f.blocks;
  const int sp = lb % nsplit, s = lb / nsplit, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ov = o * v, vv = v * v, oo = o * o;
  float *Xs = sm2, *W = sm2 + ov, *Vs = W + ov, *Os = Vs + vv;
  const float *Xg = X + (size_t)s * ov;
  const int qa = (int)((long long)sp * nq / nsplit), qb = (int)((long long)(sp + 1) * nq / nsplit);
  // RNG: range k of the m in each split begins at Q = floor(k nq / nrg), k = sp m, ...; qf is where the next one
  // begins, and part the numerator's rest there
  const int nrg = RNG ? nsplit * m : 1, step = nq / nrg, rest = nq % nrg;
  int qf = qa, part = RNG ? (int)((long long)sp * m * nq % nrg) : 0;
  auto next = [&]() {
    part += rest;
    qf += step + (part >= nrg ? 1 : 0);
    part -= part >= nrg ? nrg : 0;
  };
  if (RNG) next();
  float tv[UV], to[UO], bq[EPT2];
  auto load_q = [&](int q) {
    const TB *Bq = Bov + (size_t)q * ov, *Vq = Bvv + (size_t)q * vv, *Oq = Boo + (size_t)q * oo;
#pragma unroll
    for (int u = 0; u < UV; ++u) tv[u] = bload(Vq, min(tid + 256 * u, vv - 1));
#pragma unroll
    for (int u = 0; u < UO; ++u) to[u] = bload(Oq, min(tid + 256 * u, oo - 1));
#pragma unroll
    for (int u = 0; u < EPT2; ++u) bq[u] = bload(Bq, min(tid + 256 * u, ov - 1));
  };
  {
    float xs[EPT2];
#pragma unroll
    for (int u = 0; u < EPT2; ++u) xs[u] = Xg[min(tid + 256 * u, ov - 1)];
    if (qa < qb) load_q(qa);
#pragma unroll
    for (int u = 0; u < EPT2; ++u)
      if (tid + 256 * u < ov) Xs[tid + 256 * u] = xs[u];
  }
  float J[EPT2], K[EPT2], T[EPT2];  // a range's sums, and the ranges before it
#pragma unroll
  for (int k = 0; k < EPT2; ++k) J[k] = K[k] = T[k] = 0.f;
  bool first = true;
  for (int q = qa; q < qb; ++q) {
    float bk[EPT2];
#pragma unroll
    for (int u = 0; u < UV; ++u)
      if (tid + 256 * u < vv) Vs[tid + 256 * u] = tv[u];
#pragma unroll
    for (int u = 0; u < UO; ++u)
      if (tid + 256 * u < oo) Os[tid + 256 * u] = to[u];
    for (int e = tid + 256 * UV; e < vv; e += 256) Vs[e] = bload(Bvv + (size_t)q * vv, e);
    for (int e = tid + 256 * UO; e < oo; e += 256) Os[e] = bload(Boo + (size_t)q * oo, e);
    float pd = 0.f;
#pragma unroll
    for (int k = 0; k < EPT2; ++k) {
      const int e = tid + 256 * k;
      bk[k] = bq[k];
      if (e < ov) pd += bk[k] * Xs[e];  // (this thread's own value of X)
    }
    if (q + 1 < qb) load_q(q + 1);
    pd = wsum(pd);
    if (lane == 0) red[wave] = pd;
    __syncthreads();
    const float d = (red[0] + red[1]) + (red[2] + red[3]);
#pragma unroll
    for (int k = 0; k < EPT2; ++k) {
      const int e = tid + 256 * k;
      if (e < ov) {
        J[k] += 2.f * d * bk[k];
        const int i = e / v, a = e - i * v;
        W[e] = dot4(Xs + i * v, 1, Vs + a, v, v);
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < EPT2; ++k) {
      const int e = tid + 256 * k;
      if (e < ov) {
        const int i = e / v, a = e - i * v;
        K[k] += dot4(Os + i * o, 1, W + a, v, o);
      }
    }
    __syncthreads();  // W, red and the staged factors are rewritten by the next Q
    if (RNG && q + 1 == qf && q + 1 < qb) {
#pragma unroll
      for (int k = 0; k < EPT2; ++k) {
        const float x = J[k] - cx * K[k];
        T[k] = first ? x : T[k] + x;
        J[k] = K[k] = 0.f;
      }
      first = false;
      next();
    }
  }
  float *Pp = P + ((size_t)sp * ns + s) * ov;
#pragma unroll
  for (int k = 0; k < EPT2; ++k) {
    const int e = tid + 256 * k;
    const float x = J[k] - cx * K[k];
    if (e < ov) Pp[e] = RNG && !first ? T[k] + x : x;
  }
}

}  // namespace

hipError_t prepare_small() {
  const int bytes = SMALL_LDS_FLOATS * (int)sizeof(float);
  const void *fn[] = {reinterpret_cast<const void *>(&k_small_2e<float, false>),
                      reinterpret_cast<const void *>(&k_small_2e<float, true>),
                      reinterpret_cast<const void *>(&k_small_2e<__hip_bfloat16, false>),
                      reinterpret_cast<const void *>(&k_small_2e<__hip_bfloat16, true>)};
  for (const void *f : fn) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_small_2e(hipStream_t s, int b_dtype, const void *Bov, const void *Boo, const void *Bvv,
                           const float *X, int o, int v, int nq, int ns, int nsplit, int m, float cx, float *P,
                           const FieldArgs &f) {
  const int ov = o * v;
  if (ov > SMALL_OV_MAX || nsplit < 1 || m < 1 || (long long)nsplit * m > nq) return hipErrorInvalidValue;
  const dim3 grid(f.blocks + nsplit * ns);
  const size_t lds = ((size_t)2 * ov + (size_t)v * v + (size_t)o * o) * sizeof(float);
  auto go = [&](auto b, auto rng) {
    using TB = decltype(b);
    hipLaunchKernelGGL((k_small_2e<TB, decltype(rng)::value>), grid, dim3(256), lds, s, static_cast<const TB *>(Bov),
                       static_cast<const TB *>(Boo), static_cast<const TB *>(Bvv), X, o, v, nq, ns, nsplit, m, cx, P,
                       f);
  };
  auto pick = [&](auto b) {
    if (m > 1) go(b, std::true_type{});
    else go(b, std::false_type{});
  };
  if (b_dtype == RTTDA_BF16) pick(__hip_bfloat16{});
  else pick(0.f);
  return hipGetLastError();
}

}  // namespace rttda
