// Bandwidth- and latency-bound kernels of the RT-TDA step on gfx950:
// dipole blocks, Coulomb GEMV pair, FP64 field/trace, stage scalars, RK4 epilogue, kick.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "field.h"

namespace rttda {

namespace {

__device__ __forceinline__ float load_b(const float *p, size_t i) { return p[i]; }
__device__ __forceinline__ float load_b(const __hip_bfloat16 *p, size_t i) { return __bfloat162float(p[i]); }

template <typename T>
__device__ __forceinline__ T wave_sum(T x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// ------------------------------------------------------------------------------------------------
// mu_d = sum_k d_k mu_k, split into the oo, ov and vv blocks, one copy per right-hand side.
// ------------------------------------------------------------------------------------------------
__global__ void k_mu_blocks(const double *__restrict__ mu, const DevPulse *__restrict__ pulses, int o, int v,
                            int R, double *__restrict__ moo, double *__restrict__ mov, double *__restrict__ mvv) {
  const long long n = o + v, nn = n * n, total = (long long)R * nn;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int r = (int)(e / nn);
    const long long pq = e - r * nn;
    const int p = (int)(pq / n), q = (int)(pq - p * n);
    const double *d = pulses[r].dir;
    const double m = d[0] * mu[pq] + d[1] * mu[nn + pq] + d[2] * mu[2 * nn + pq];
    if (p < o && q < o)
      moo[(size_t)r * o * o + (size_t)p * o + q] = m;
    else if (p < o)
      mov[(size_t)r * o * v + (size_t)p * v + (q - o)] = m;
    else if (q >= o)
      mvv[(size_t)r * v * v + (size_t)(p - o) * v + (q - o)] = m;
  }
}

// D_ia = e_a - e_i (diagonal of A, eq. A_matrix_element2).
__global__ void k_gaps(const double *__restrict__ e_occ, const double *__restrict__ e_virt, int o, int v,
                       double *__restrict__ D) {
  const long long total = (long long)o * v;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int i = (int)(e / v), a = (int)(e - (long long)i * v);
    D[e] = e_virt[a] - e_occ[i];
  }
}

__global__ void k_to_f32(const double *__restrict__ c, long long n, float *__restrict__ x) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
    x[e] = (float)c[e];
}

__device__ __forceinline__ void split_bf16(double x, __hip_bfloat16 &hi, __hip_bfloat16 &lo) {
  hi = __float2bfloat16((float)x);
  lo = __float2bfloat16((float)(x - (double)__bfloat162float(hi)));
}

__global__ void k_to_bf16x2(const double *__restrict__ c, long long n, float *__restrict__ x,
                            __hip_bfloat16 *__restrict__ hi, __hip_bfloat16 *__restrict__ lo) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
    x[e] = (float)c[e];
    split_bf16(c[e], hi[e], lo[e]);
  }
}

// ------------------------------------------------------------------------------------------------
// Coulomb, first product: d[Q][s] = sum_ia B_ov[Q][ia] X[s][ia]   (B streamed once from HBM)
// Block = QT rows of B x ST slices x one ia chunk; the chunk partials dpart[chunk][Q][s] are summed
// in a fixed order by the second product.  Each lane takes EPL consecutive ia per load (16 bytes of B
// where ov is a multiple of those values, so that every row starts aligned); rows of other lengths are
// read one value per lane and load, four loads per row in flight (o27 v203 N_Q541 FP32, 3 RHS: 7.7 us;
// with one in flight 30.5 us).
// ------------------------------------------------------------------------------------------------
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u4u __attribute__((ext_vector_type(4), aligned(2)));

// Sum 64 per-lane values over the wave with 63 exchanges: at each halving step a lane keeps the
// half of its values selected by its lane bit and adds the partner's copy of that half.  On exit
// lane l holds the wave total of value l.
template <int K>
__device__ __forceinline__ void transpose_sum_step(float (&v)[64], int lane) {
  const bool up = (lane & K) != 0;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const float send = up ? v[j] : v[j + K];
    const float keep = up ? v[j + K] : v[j];
    v[j] = keep + __shfl_xor(send, K, 64);
  }
  if constexpr (K > 1) transpose_sum_step<K / 2>(v, lane);
}

__device__ __forceinline__ float wave_transpose_sum64(float (&v)[64], int lane) {
  transpose_sum_step<32>(v, lane);
  return v[0];
}

// One 16-byte load of a B row: EPL values widened to FP32
template <int EPL>
__device__ __forceinline__ void load_row(const float *p, size_t i, float (&x)[EPL]) {
  static_assert(EPL == 4, "FP32 rows: four values per 16-byte load");
  const f4u t = *reinterpret_cast<const f4u *>(p + i);
  x[0] = t[0], x[1] = t[1], x[2] = t[2], x[3] = t[3];
}
template <int EPL>
__device__ __forceinline__ void load_row(const __hip_bfloat16 *p, size_t i, float (&x)[EPL]) {
  static_assert(EPL == 4 || EPL == 8, "BF16 rows: four or eight values per load");
  typedef unsigned u2u __attribute__((ext_vector_type(2), aligned(2)));
  unsigned w[EPL / 2];  // element 2k in the low half of word k
  if constexpr (EPL == 8) {
    const u4u u = *reinterpret_cast<const u4u *>(p + i);
    w[0] = u[0], w[1] = u[1], w[2] = u[2], w[3] = u[3];
  } else {
    const u2u u = *reinterpret_cast<const u2u *>(p + i);
    w[0] = u[0], w[1] = u[1];
  }
#pragma unroll
  for (int k = 0; k < EPL / 2; ++k) {
    x[2 * k] = __uint_as_float(w[k] << 16);
    x[2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
  }
}
template <typename TB>
constexpr int row_epl() {
  return 16 / (int)sizeof(TB);
}

template <typename TB, int QT, int ST, int EPL>
__global__ __launch_bounds__(256) void k_gemv1(const TB *__restrict__ B, const float *__restrict__ X, int nq, int ov,
                                               int ns, int echunk, float *__restrict__ dpart, FieldArgs f) {
  static_assert(QT * ST <= 64, "one reduced value per lane");
  if ((int)blockIdx.x < f.blocks) {
    field_block(f, blockIdx.x);
    return;
  }
  const int nqb = (nq + QT - 1) / QT, nsb = (ns + ST - 1) / ST, lb = (int)blockIdx.x - f.blocks;
  const int q0 = lb % nqb * QT, s0 = lb / nqb % nsb * ST, ez = lb / (nqb * nsb);
  const int e0 = ez * echunk, e1 = min(ov, e0 + echunk);
  const int nqv = min(QT, nq - q0), nsv = min(ST, ns - s0);
  float acc[QT][ST];
#pragma unroll
  for (int a = 0; a < QT; ++a)
#pragma unroll
    for (int b = 0; b < ST; ++b) acc[a][b] = 0.f;
  // (rows past nq read row q0, slices past ns slice s0: their sums are not stored)
  if constexpr (EPL > 1) {
    for (int e = e0 + EPL * (int)threadIdx.x; e < e1; e += 256 * EPL) {
      float xs[ST][EPL];
#pragma unroll
      for (int b = 0; b < ST; ++b)
#pragma unroll
        for (int g = 0; g < EPL / 4; ++g) {
          const f4u t = *reinterpret_cast<const f4u *>(X + (size_t)(s0 + (b < nsv ? b : 0)) * ov + e + 4 * g);
          xs[b][4 * g] = t[0], xs[b][4 * g + 1] = t[1], xs[b][4 * g + 2] = t[2], xs[b][4 * g + 3] = t[3];
        }
      // all QT rows' loads issued before any of their products
      float bq[QT][EPL];
#pragma unroll
      for (int a = 0; a < QT; ++a) load_row<EPL>(B, (size_t)(q0 + (a < nqv ? a : 0)) * ov + e, bq[a]);
#pragma unroll
      for (int a = 0; a < QT; ++a)
#pragma unroll
        for (int b = 0; b < ST; ++b) {
          float t = acc[a][b];
#pragma unroll
          for (int k = 0; k < EPL; ++k) t = fmaf(bq[a][k], xs[b][k], t);
          acc[a][b] = t;
        }
    }
  } else {
    constexpr int U = 4;  // (values past the chunk read its last one again and are left out)
    for (int e = e0 + (int)threadIdx.x; e < e1; e += 256 * U) {
      float xs[U][ST], bq[U][QT];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int ee = min(e + 256 * u, e1 - 1);
#pragma unroll
        for (int b = 0; b < ST; ++b) xs[u][b] = X[(size_t)(s0 + (b < nsv ? b : 0)) * ov + ee];
#pragma unroll
        for (int a = 0; a < QT; ++a) bq[u][a] = load_b(B, (size_t)(q0 + (a < nqv ? a : 0)) * ov + ee);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int a = 0; a < QT; ++a)
#pragma unroll
          for (int b = 0; b < ST; ++b) {
            const float t = fmaf(bq[u][a], xs[u][b], acc[a][b]);
            acc[a][b] = e + 256 * u < e1 ? t : acc[a][b];
          }
    }
  }
  float vals[64];
#pragma unroll
  for (int k = 0; k < 64; ++k) vals[k] = k < QT * ST ? acc[k / ST][k % ST] : 0.f;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __shared__ float red[4][64];
  red[wave][lane] = wave_transpose_sum64(vals, lane);
  __syncthreads();
  if (threadIdx.x < QT * ST) {
    const int k = threadIdx.x, a = k / ST, b = k % ST;
    if (a < nqv && b < nsv)
      dpart[((size_t)ez * nq + q0 + a) * ns + s0 + b] = (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
  }
}

// ------------------------------------------------------------------------------------------------
// Coulomb, second product: P[split][s][ia] = 2 sum_{Q in split} B_ov[Q][ia] d[Q][s], with d the sum of
// the first product's nes chunk partials (in chunk order), staged in LDS.
// QW = 4 (ov % 4 == 0): each lane holds EPL consecutive ia, 16 bytes of a B row per load (a row's last
// lane takes its last EPL values: it stores some a second time, with the same bits), eight rows in
// flight; a block covers 64 EPL ia and its waves take every fourth Q of the split's range, their
// partials meeting in LDS in wave order.  QW = 1 (other row lengths): one ia per lane, sixteen rows in
// flight, every Q.  Each slice's sum depends only on its own d values, so a batch and a single RHS give
// the same bits.
// Bound by HBM where B_ov is large (o60 v400 N_Q1500, 3 RHS: 22 us in BF16, 25 us in FP32), by the chain of
// its loads where it is small.  o24 v184 N_Q480 BF16, one RHS: 5.6 us (with rows past the last batch of a
// range read one at a time and d's chunks summed in a launch of their own, 9.6 + 1.8 us); rows of any
// length, o27 v203 N_Q541 FP32, 3 RHS: 7.8 us (one row in flight, 9.9 + 4.8 us).
// ------------------------------------------------------------------------------------------------
template <typename TB, int ST, int QW, int EPL>
__global__ __launch_bounds__(256) void k_gemv2(const TB *__restrict__ B, const float *__restrict__ dpart, int nes,
                                               int nq, int ov, int ns, int nsplit, float *__restrict__ P) {
  constexpr int QCH = 256, U = EPL == 1 ? 16 : 8;
  __shared__ float dsh[QCH][ST];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ebase = ((int)blockIdx.x * (QW == 1 ? 4 : 1) + (QW == 1 ? wave : 0)) * (64 * EPL) + EPL * lane;
  const bool live = ebase < ov;
  const int e = min(ebase, ov - EPL);
  const int w = QW == 1 ? 0 : wave;
  const int s0 = blockIdx.y * ST, sp = blockIdx.z;
  const int qa = (int)((long long)sp * nq / nsplit), qb = (int)((long long)(sp + 1) * nq / nsplit);
  float acc[ST][EPL];
#pragma unroll
  for (int b = 0; b < ST; ++b)
#pragma unroll
    for (int k = 0; k < EPL; ++k) acc[b][k] = 0.f;
  for (int qc = qa; qc < qb; qc += QCH) {
    const int nqc = min(QCH, qb - qc);
    __syncthreads();
    // four values of d per thread at a time, four chunks of each in flight
    for (int k0 = threadIdx.x; k0 < nqc * ST; k0 += 4 * 256) {
      float d[4] = {0.f, 0.f, 0.f, 0.f};
      for (int c = 0; c < nes; c += 4) {
        float t[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = min(k0 + 256 * i, nqc * ST - 1), qq = k / ST, b = k % ST;
          const float *src = dpart + (size_t)(qc + qq) * ns + s0 + (s0 + b < ns ? b : 0);
#pragma unroll
          for (int u = 0; u < 4; ++u) t[i][u] = src[(size_t)min(c + u, nes - 1) * nq * ns];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int u = 0; u < 4; ++u) d[i] = c + u < nes ? d[i] + t[i][u] : d[i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (k0 + 256 * i < nqc * ST) dsh[(k0 + 256 * i) / ST][(k0 + 256 * i) % ST] = d[i];
    }
    __syncthreads();
    if (live) {
      for (int qq = w; qq < nqc; qq += QW * U) {
        // (rows past the range read its last one again and are left out of the sums: a condition on the
        // load would make each wait for the one before it)
        float bq[U][EPL];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const size_t at = (size_t)(qc + min(qq + QW * u, nqc - 1)) * ov + e;
          if constexpr (EPL == 1) bq[u][0] = load_b(B, at);
          else load_row<EPL>(B, at, bq[u]);
        }
        auto add = [&](int u) {
#pragma unroll
          for (int b = 0; b < ST; ++b) {
            const float d = dsh[qq + QW * u][b];
#pragma unroll
            for (int k = 0; k < EPL; ++k) acc[b][k] = fmaf(bq[u][k], d, acc[b][k]);
          }
        };
        // (a whole batch has no branch between its rows, which would put each row's LDS reads behind
        // the sums of the one before)
        if (qq + QW * (U - 1) < nqc) {
#pragma unroll
          for (int u = 0; u < U; ++u) add(u);
        } else {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (qq + QW * u < nqc) add(u);
          }
        }
      }
    }
  }
  if constexpr (QW == 1) {
    if (!live) return;
#pragma unroll
    for (int b = 0; b < ST; ++b) {
      if (s0 + b < ns) P[((size_t)sp * ns + s0 + b) * ov + e] = 2.f * acc[b][0];
    }
  } else {
    // wave partials through LDS, four values per lane at a time; wave w stores slices w, w + 4, ...
    __shared__ float4 red[4][ST][64];
#pragma unroll
    for (int g = 0; g < EPL / 4; ++g) {
      __syncthreads();
#pragma unroll
      for (int b = 0; b < ST; ++b)
        red[w][b][lane] = make_float4(acc[b][4 * g], acc[b][4 * g + 1], acc[b][4 * g + 2], acc[b][4 * g + 3]);
      __syncthreads();
      for (int b = wave; b < ST; b += 4) {
        if (!live || s0 + b >= ns) continue;
        const float4 r0 = red[0][b][lane], r1 = red[1][b][lane], r2 = red[2][b][lane], r3 = red[3][b][lane];
        f4u t;
        t[0] = 2.f * ((r0.x + r1.x) + (r2.x + r3.x));
        t[1] = 2.f * ((r0.y + r1.y) + (r2.y + r3.y));
        t[2] = 2.f * ((r0.z + r1.z) + (r2.z + r3.z));
        t[3] = 2.f * ((r0.w + r1.w) + (r2.w + r3.w));
        *reinterpret_cast<f4u *>(P + ((size_t)sp * ns + s0 + b) * ov + e + 4 * g) = t;
      }
    }
  }
}

// The field product as a launch of its own (see field.h)
__global__ __launch_bounds__(256) void k_field(FieldArgs f) { field_block(f, blockIdx.x); }

// ------------------------------------------------------------------------------------------------
// Stage scalars of one right-hand side, by one block of 256 threads: its pulse field E(t_stage), the
// ground-row product g, the trace, norm and energy samples with the norm guard, and the RK4 update of
// c0 (dc0/dt = -i(-E g) = i E g).  The field kernel's per-block partial sums are added one component per
// wave (lanes over blocks, then a fixed shuffle tree).  Several right-hand sides that trip the guard at
// one step write the same value.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ double stage_node(int stage) { return stage == 0 ? 0.0 : (stage == 3 ? 1.0 : 0.5); }

__device__ __forceinline__ void scalar_rhs(int r, int R, int nbf, int stage, int mode, double dt,
                                           const DevPulse *__restrict__ pulses, DevState *__restrict__ st,
                                           const double *__restrict__ part, double *__restrict__ sc,
                                           double *__restrict__ c0, double *__restrict__ acc0, double *__restrict__ xs0,
                                           double *__restrict__ out, double *__restrict__ normref,
                                           double *__restrict__ s0) {
  __shared__ double tot[PART_STRIDE + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long step = st->step, k = step - st->step0;
  {
    double t = 0.0;
    const double *pp = part + (size_t)r * nbf * PART_STRIDE + wave;
    for (int b = lane; b < nbf; b += 64) t += pp[(size_t)b * PART_STRIDE];
    t = wave_sum(t);
    if (lane == 0) tot[wave] = t;
  }
  if ((mode & SM_ENERGY) && st->energy && wave == 0) {  // the epilogue's per-block partial sums
    const long long nbe = st->nbe;
    double e = 0.0;
    for (long long b = lane; b < nbe; b += 64) e += st->epart[(size_t)r * nbe + b];
    e = wave_sum(e);
    if (lane == 0) st->energy[k * R + r] = e;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  const double g0 = tot[0], g1 = tot[1], tr = tot[2], nr = tot[3];
  double E = 0.0;
  if (mode & SM_EFIELD)
    E = pulse_field(pulses[r], ((double)step + stage_node(stage)) * dt);
  else if (mode & SM_KEEP_E)
    E = sc[r * SC_STRIDE + SC_E];
  sc[r * SC_STRIDE + SC_GRE] = g0;
  sc[r * SC_STRIDE + SC_GIM] = g1;
  sc[r * SC_STRIDE + SC_E] = E;
  // X0 of this stage (c0 at stage 0, else the stage value)
  const double x0r = (stage == 0) ? c0[2 * r] : xs0[2 * r];
  const double x0i = (stage == 0) ? c0[2 * r + 1] : xs0[2 * r + 1];
  if (mode & (SM_TRACE | SM_OUT)) {
    const double t = tr + (x0r * g0 + x0i * g1);
    const double n2 = nr + (x0r * x0r + x0i * x0i);
    if (mode & SM_OUT) out[r] = t;
    if (mode & SM_TRACE) {
      if (st->trace) st->trace[k * R + r] = t;
      if (st->norms) st->norms[k * R + r] = n2;
      if (k == 0 && !st->keep_ref) {
        normref[r] = n2;
      } else if (!(n2 <= 2.0 * normref[r]) && st->bad_step < 0) {  // also catches NaN
        st->bad_step = step;
      }
    }
  }
  if (mode & SM_SIGMA0) {
    s0[2 * r] = -E * g0;
    s0[2 * r + 1] = -E * g1;
  }
  if (mode & SM_C0) {
    // k0 = -i * (H X)_0 = -i * (-E g) = i E g
    const double kr = -E * g1, ki = E * g0;
    const double cr = c0[2 * r], ci = c0[2 * r + 1];
    if (stage == 0) {
      acc0[2 * r] = cr + dt / 6.0 * kr;
      acc0[2 * r + 1] = ci + dt / 6.0 * ki;
      xs0[2 * r] = cr + 0.5 * dt * kr;
      xs0[2 * r + 1] = ci + 0.5 * dt * ki;
    } else if (stage == 1) {
      acc0[2 * r] += dt / 3.0 * kr;
      acc0[2 * r + 1] += dt / 3.0 * ki;
      xs0[2 * r] = cr + 0.5 * dt * kr;
      xs0[2 * r + 1] = ci + 0.5 * dt * ki;
    } else if (stage == 2) {
      acc0[2 * r] += dt / 3.0 * kr;
      acc0[2 * r + 1] += dt / 3.0 * ki;
      xs0[2 * r] = cr + dt * kr;
      xs0[2 * r + 1] = ci + dt * ki;
    } else {
      c0[2 * r] = acc0[2 * r] + dt / 6.0 * kr;
      c0[2 * r + 1] = acc0[2 * r + 1] + dt / 6.0 * ki;
    }
  }
}

// The stage scalars as a launch of their own (one block per right-hand side), where no RK4 epilogue
// follows that carries them
__global__ __launch_bounds__(256) void k_scalar(int R, int nbf, int stage, int mode, double dt,
                                                const DevPulse *__restrict__ pulses, DevState *__restrict__ st,
                                                const double *__restrict__ part, double *__restrict__ sc,
                                                double *__restrict__ c0, double *__restrict__ acc0,
                                                double *__restrict__ xs0, double *__restrict__ out,
                                                double *__restrict__ normref, double *__restrict__ s0) {
  scalar_rhs(blockIdx.x, R, nbf, stage, mode, dt, pulses, st, part, sc, c0, acc0, xs0, out, normref, s0);
  if ((mode & SM_INC) && blockIdx.x == 0 && threadIdx.x == 0) st->pend = 1;
}

// Sum of the partial slabs `sb` at element e of a block of 256 threads that holds 64 elements: each wave
// adds a quarter of the sums (eight loads per plane in flight, in memory order), and the quarters meet in
// LDS in wave order.  Every thread of lane l receives the sum of element l.  NP planes, `plane` floats
// apart.  (Slabs past a quarter read its last one again and are left out of the sum: a condition on the
// load would make each wait for the one before it.)  GRP: some sums are of several slabs.
template <int NP, bool GRP>
__device__ __forceinline__ void slab_sum(const float *__restrict__ P, size_t slab, size_t plane, Slabs sb, size_t e,
                                         bool live, double (&out)[NP]) {
  __shared__ double quarter[4][NP][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  auto first = [&](int k) { return !GRP || k < sb.nc ? k : sb.nc + (k - sb.nc) * sb.grp; };  // its place in memory
  const int a = first(wave * sb.n / 4), b = first((wave + 1) * sb.n / 4);
  double t[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) t[p] = 0.0;
  if (live) {
    constexpr int U = 8;
    auto load = [&](int sl, float (&x)[NP][U]) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int p = 0; p < NP; ++p) x[p][u] = P[(size_t)min(sl + u, b - 1) * slab + p * plane + e];
    };
    if constexpr (!GRP) {
      for (int sl = a; sl < b; sl += U) {
        float x[NP][U];
        load(sl, x);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int p = 0; p < NP; ++p) t[p] += sl + u < b ? (double)x[p][u] : 0.0;
      }
    } else {  // f: the sum of the g slabs of a group so far (without a branch between the slabs)
      int g = 0;
      float f[NP] = {};
      for (int sl = a; sl < b; sl += U) {
        float x[NP][U];
        load(sl, x);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool last = g + 1 == sb.grp || sl + u < sb.nc, ok = sl + u < b;
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            f[p] = g == 0 ? x[p][u] : f[p] + x[p][u];
            t[p] += last && ok ? (double)f[p] : 0.0;
          }
          g = last ? 0 : g + 1;
        }
      }
    }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) quarter[wave][p][lane] = t[p];
  __syncthreads();
#pragma unroll
  for (int p = 0; p < NP; ++p)
    out[p] = (quarter[0][p][lane] + quarter[1][p][lane]) + (quarter[2][p][lane] + quarter[3][p][lane]);
  __syncthreads();
}

// ------------------------------------------------------------------------------------------------
// Symplectic split-operator step (Propagation Algorithm subsection: X = q + i p, dq/dt = H p,
// dp/dt = -H q; second order, kick-drift-kick):
//   drift:  q <- q + dt (H p_h)                    at t_n + dt/2
//   kick:   p <- p_h - dt/2 (H q);  p_h <- p - dt/2 (H q)   at t_n + dt   (two half kicks merged)
// with H x = D x + (Coulomb + exchange partials of x) - E F_x on one real plane and ground element
// (H x)_0 = -E g_x.  c holds (q, p) at whole steps; W (the stage buffer) holds the work state
// (q, p_h).  The FP32 (+ BF16 hi/lo) copy of the next plane to multiply goes to x32 [R][o][v].
// A block of 256 threads holds 64 (r, i, a): its waves share the slabs, the first updates; the ground
// element of RHS r by the thread with ia == 0.
// ------------------------------------------------------------------------------------------------
template <int PREC, bool GRP>
__global__ __launch_bounds__(256) void k_sso_update(int R, int o, int v, Slabs slabs, int mode, int use_field, double dt,
                                                    const double *__restrict__ D, const float *__restrict__ P,
                                                    const double *__restrict__ F, const double *__restrict__ sc,
                                                    double *__restrict__ c, double *__restrict__ c0,
                                                    double *__restrict__ W, double *__restrict__ W0,
                                                    float *__restrict__ x32, __hip_bfloat16 *__restrict__ xhi,
                                                    __hip_bfloat16 *__restrict__ xlo) {
  const size_t ov = (size_t)o * v;
  const size_t total = (size_t)R * ov;
  const size_t slab = total;  // one plane per RHS: floats per partial slab
  const int pl = (mode == SSO_DRIFT) ? 1 : 0;  // plane of the multiplied vector
  for (size_t e0 = blockIdx.x * (size_t)64; e0 < total; e0 += (size_t)gridDim.x * 64) {
    const size_t e = e0 + (threadIdx.x & 63);
    double psum[1];
    slab_sum<1, GRP>(P, slab, 0, slabs, e, e < total, psum);
    if (threadIdx.x >= 64 || e >= total) continue;
    const size_t r = e / ov, ia = e - r * ov;
    const size_t iq = r * 2 * ov + ia, ip = iq + ov;
    const double x = (mode == SSO_KICK_FIRST) ? c[iq] : W[pl ? ip : iq];
    const double E = sc[r * SC_STRIDE + SC_E];
    double hx = D[ia] * x + psum[0];
    if (use_field) hx -= E * F[pl ? ip : iq];
    double nxt;
    if (mode == SSO_DRIFT) {
      const double qn = c[iq] + dt * hx;
      c[iq] = qn;
      W[iq] = qn;
      nxt = qn;
    } else if (mode == SSO_KICK) {
      const double pn = W[ip] - 0.5 * dt * hx;
      c[ip] = pn;
      nxt = pn - 0.5 * dt * hx;
      W[ip] = nxt;
    } else {
      W[iq] = x;
      nxt = c[ip] - 0.5 * dt * hx;
      W[ip] = nxt;
    }
    x32[e] = (float)nxt;
    if (PREC == 1) split_bf16(nxt, xhi[e], xlo[e]);
    if (ia == 0) {
      const double h0 = use_field ? -E * sc[r * SC_STRIDE + (pl ? SC_GIM : SC_GRE)] : 0.0;
      if (mode == SSO_DRIFT) {
        const double q0 = c0[2 * r] + dt * h0;
        c0[2 * r] = q0;
        W0[2 * r] = q0;
      } else if (mode == SSO_KICK) {
        const double p0 = W0[2 * r + 1] - 0.5 * dt * h0;
        c0[2 * r + 1] = p0;
        W0[2 * r + 1] = p0 - 0.5 * dt * h0;
      } else {
        W0[2 * r] = c0[2 * r];
        W0[2 * r + 1] = c0[2 * r + 1] - 0.5 * dt * h0;
      }
    }
  }
}

// FP32 (+ BF16 hi/lo) copy of one plane of c into x32 [R][o][v].
template <int PREC>
__global__ void k_plane_copy(int R, size_t ov, int plane, const double *__restrict__ c, float *__restrict__ x32,
                             __hip_bfloat16 *__restrict__ xhi, __hip_bfloat16 *__restrict__ xlo) {
  const size_t total = (size_t)R * ov;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const size_t r = e / ov, ia = e - r * ov;
    const double x = c[(r * 2 + plane) * ov + ia];
    x32[e] = (float)x;
    if (PREC == 1) split_bf16(x, xhi[e], xlo[e]);
  }
}

// ------------------------------------------------------------------------------------------------
// Lanczos iteration on A (stability guard: the RK4 step is stable for rho(A) dt below ~2.8).
// Vectors of length ov in FP64; A v = D v + (Coulomb + exchange partials of v) for one real
// slice.  Block partial sums go to part[blockIdx.x] and are added in a fixed order by the next launch.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ double block_sum(double x, double *sh) {
  x = wave_sum(x);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) sh[wave] = x;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w];
  return t;
}

// start vector: a fixed pseudo-random vector (SplitMix64 of the index), part = |v|^2
__global__ __launch_bounds__(256) void k_lz_init(long long n, double *__restrict__ v, double *__restrict__ part) {
  __shared__ double sh[4];
  double acc = 0.0;
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
    unsigned long long z = (unsigned long long)e + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    const double x = (double)(z >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0;
    v[e] = x;
    acc += x * x;
  }
  const double t = block_sum(acc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// Sum of a launch's nb block partials, by a whole block of 256 threads (threads over blocks, waves by
// shuffles, the waves in order): every block of the next launch forms it for itself, so that no launch and no
// copy to the host stand between the dot products and their use
__device__ __forceinline__ double lz_total(const double *__restrict__ part, int nb) {
  __shared__ double sh[4];
  __shared__ double tot;
  double t = 0.0;
  for (int k = threadIdx.x; k < nb; k += 256) t += part[k];
  t = block_sum(t, sh);
  if (threadIdx.x == 0) tot = t;
  __syncthreads();
  return tot;
}

// w = A v - beta vprev, part = <w, v>; a block of 256 threads holds 64 elements at a time, its waves
// share the slabs
__global__ __launch_bounds__(256) void k_lz_apply(long long n, int nslab, const double *__restrict__ D,
                                                  const float *__restrict__ P, const double *__restrict__ v,
                                                  const double *__restrict__ vprev,
                                                  const double *__restrict__ pbeta, double *__restrict__ w,
                                                  double *__restrict__ part) {
  __shared__ double sh[4];
  const double beta = pbeta ? *pbeta : 0.0;
  double acc = 0.0;
  for (long long e0 = blockIdx.x * 64LL; e0 < n; e0 += (long long)gridDim.x * 64) {
    const long long e = e0 + (threadIdx.x & 63);
    double p[1];
    slab_sum<1, false>(P, (size_t)n, 0, Slabs{nslab, 0, 1}, (size_t)e, e < n, p);
    if (threadIdx.x >= 64 || e >= n) continue;
    const double s = D[e] * v[e] + p[0] - beta * vprev[e];
    w[e] = s;
    acc += s * v[e];
  }
  const double t = block_sum(acc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// w -= alpha v, part = |w|^2
__global__ __launch_bounds__(256) void k_lz_orth(long long n, const double *__restrict__ v,
                                                 const double *__restrict__ dots, double *__restrict__ alpha_out,
                                                 double *__restrict__ w, double *__restrict__ part) {
  __shared__ double sh[4];
  const double alpha = lz_total(dots, gridDim.x);
  if (blockIdx.x == 0 && threadIdx.x == 0) *alpha_out = alpha;
  double acc = 0.0;
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
    const double x = w[e] - alpha * v[e];
    w[e] = x;
    acc += x * x;
  }
  const double t = block_sum(acc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// beta = sqrt(sum dots), vprev = v (shift), v = w / beta; FP32 (+ BF16 hi/lo) copy of v for the next product
template <int PREC>
__global__ __launch_bounds__(256) void k_lz_next(long long n, const double *__restrict__ dots,
                                                 double *__restrict__ beta_out, const double *__restrict__ w,
                                                 double *__restrict__ v, double *__restrict__ vprev,
                                                 float *__restrict__ x32, __hip_bfloat16 *__restrict__ xhi,
                                                 __hip_bfloat16 *__restrict__ xlo, int shift) {
  const double t = lz_total(dots, gridDim.x);
  const double b = sqrt(t < 0.0 ? 0.0 : t), scale = 1.0 / b;  // (a NaN stays one: fmax would make it 0, "the end")
  if (blockIdx.x == 0 && threadIdx.x == 0) *beta_out = b;
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
    if (shift) vprev[e] = v[e];
    const double x = w[e] * scale;
    v[e] = x;
    x32[e] = (float)x;
    if (PREC == 1) split_bf16(x, xhi[e], xlo[e]);
  }
}

// ------------------------------------------------------------------------------------------------
// RK4 epilogue (FP64): sigma = D X + sum of Coulomb/exchange partials - E F;  k = -i sigma;
// stage accumulation into acc, next stage input (FP64 + FP32 or BF16 hi/lo copy), c at stage 4.
// A block of 256 threads holds 64 (i, a) of one RHS: its four waves share the slabs (a chain of load
// latencies where there are many of them and few elements), then two of them update one plane each:
// Re k = Im sigma and Im k = -Re sigma, so plane p's update takes the other plane's sigma.
// Xin is c in stage 0 and xs64 after it, and one wave writes the plane of xs64 that the other has read: the
// barriers of the slab sum stand between the two, and none of the three pointers is __restrict__.
// The last block of each RHS carries its stage scalars (es.mode != 0), which nothing else here reads.
// o24 v184 N_Q480, one RHS: 6.4 us; one thread per (i, a) summing every slab took 10.9 us, and the
// scalars' own launch 4.1 us.
// ------------------------------------------------------------------------------------------------
template <int PREC, bool GRP>
__global__ __launch_bounds__(256) void k_epilogue(int R, int o, int v, Slabs slabs, int stage, int mode, int use_field,
                                                  double dt, const double *__restrict__ D,
                                                  const float *__restrict__ P, const double *__restrict__ F,
                                                  double *__restrict__ sc, const double *Xin, double *c,
                                                  double *__restrict__ acc, double *xs64, float *__restrict__ x32,
                                                  __hip_bfloat16 *__restrict__ xhi, __hip_bfloat16 *__restrict__ xlo,
                                                  double *__restrict__ s_out, double *__restrict__ epart, int nbe,
                                                  StageScalars es) {
  const size_t ov = (size_t)o * v;
  const size_t slab = 2 * (size_t)R * ov;  // floats per partial slab
  const int r = blockIdx.y;                // one RHS per block row
  if ((int)blockIdx.x == nbe) {
    scalar_rhs(r, R, es.nbf, stage, es.mode, dt, es.pulses, es.st, es.part, sc, es.c0, es.acc0, es.xs0, nullptr,
               es.normref, nullptr);
    if ((es.mode & SM_INC) && r == 0 && threadIdx.x == 0) es.st->pend = 1;
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __shared__ double Esh;  // (read behind the slab sum's barriers)
  if (use_field && threadIdx.x == 0)  // with the scalars in this launch the field is this block's own to evaluate
    Esh = es.mode & SM_EFIELD ? pulse_field(es.pulses[r], ((double)es.st->step + stage_node(stage)) * dt)
                              : sc[r * SC_STRIDE + SC_E];
  double en = 0.0;  // this thread's part of <X, A X>
  for (size_t ia0 = blockIdx.x * (size_t)64; ia0 < ov; ia0 += (size_t)nbe * 64) {
    const size_t ia = ia0 + lane;
    // the update's operands are under way while the slabs are summed (from a clamped place and of any
    // plane, where they are not used)
    const int p = wave & 1, q = 1 - p;  // waves 0 and 1: plane p's update takes plane q's sigma
    const size_t im = (size_t)r * 2 * ov + (ia < ov ? ia : ov - 1);
    const size_t ip = im + p * ov, iq = im + q * ov;
    const double x = Xin[iq], d = D[im - (size_t)r * 2 * ov];
    const double f = use_field ? F[iq] : 0.0;
    double y = 0.0, ya = 0.0;
    if (mode == EP_RK4) {
      y = stage == 0 ? Xin[ip] : stage == 3 ? 0.0 : c[ip];
      ya = stage == 0 ? 0.0 : acc[ip];
    }
    double ps[2];
    slab_sum<2, GRP>(P, slab, ov, slabs, im, ia < ov, ps);
    if (wave >= 2 || ia >= ov) continue;
    double sg = d * x + ps[q];
    if (epart) en += x * sg;
    if (mode == EP_ENERGY) continue;
    if (use_field) sg -= Esh * f;
    if (mode == EP_SIGMA) {
      s_out[iq] = sg;
      continue;
    }
    const double k = p == 0 ? sg : -sg;
    double n;
    if (stage == 0) {
      acc[ip] = y + dt / 6.0 * k;
      n = y + 0.5 * dt * k;
    } else if (stage == 3) {
      n = ya + dt / 6.0 * k;
      c[ip] = n;
    } else {
      acc[ip] = ya + dt / 3.0 * k;
      n = y + ((stage == 1) ? 0.5 * dt : dt) * k;
    }
    if (stage != 3) xs64[ip] = n;
    x32[ip] = (float)n;
    if (PREC == 1) split_bf16(n, xhi[ip], xlo[ip]);
  }
  if (epart) {  // block sum in a fixed order: waves, then the wave totals
    __shared__ double ws[4];
    en = wave_sum(en);
    if (lane == 0) ws[wave] = en;
    __syncthreads();
    if (threadIdx.x == 0) epart[(size_t)r * nbe + blockIdx.x] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
  }
}

// First-order delta kick X <- X + i kappa M X for RHS with a delta pulse.
__global__ void k_kick(int R, int ov, const DevPulse *__restrict__ pulses, const double *__restrict__ F,
                       const double *__restrict__ sc, double *__restrict__ c, double *__restrict__ c0) {
  const size_t total = (size_t)R * ov;
  const size_t gid = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  for (size_t e = gid; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const size_t r = e / ov, ia = e - r * ov;
    if (pulses[r].kind != RTTDA_PULSE_DELTA) continue;
    const double kap = pulses[r].e0;
    const size_t i0 = r * 2 * ov + ia, i1 = i0 + ov;
    const double f0 = F[i0], f1 = F[i1];
    c[i0] -= kap * f1;
    c[i1] += kap * f0;
  }
  if (gid < (size_t)R && pulses[gid].kind == RTTDA_PULSE_DELTA) {
    const double kap = pulses[gid].e0;
    const double g0 = sc[gid * SC_STRIDE + SC_GRE], g1 = sc[gid * SC_STRIDE + SC_GIM];
    c0[2 * gid] -= kap * g1;
    c0[2 * gid + 1] += kap * g0;
  }
}

// One Taylor term of the unitary kick exp(i kappa M) X for the RHS with PULSE_DELTA_EXACT:
// given F = (M T)_C and g = (M T)_0 of the previous term T, the next term is (i kappa / j) M T;
// it replaces T and is added to the state (c, c0).
__global__ void k_kick_term(int R, int ov, const DevPulse *__restrict__ pulses, const double *__restrict__ F,
                            const double *__restrict__ sc, double inv_j, double *__restrict__ T,
                            double *__restrict__ T0, double *__restrict__ c, double *__restrict__ c0) {
  const size_t total = (size_t)R * ov;
  const size_t gid = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  for (size_t e = gid; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const size_t r = e / ov, ia = e - r * ov;
    if (pulses[r].kind != RTTDA_PULSE_DELTA_EXACT) continue;
    const double s = pulses[r].e0 * inv_j;
    const size_t i0 = r * 2 * ov + ia, i1 = i0 + ov;
    const double t0 = -s * F[i1], t1 = s * F[i0];
    T[i0] = t0;
    T[i1] = t1;
    c[i0] += t0;
    c[i1] += t1;
  }
  if (gid < (size_t)R && pulses[gid].kind == RTTDA_PULSE_DELTA_EXACT) {
    const double s = pulses[gid].e0 * inv_j;
    const double t0 = -s * sc[gid * SC_STRIDE + SC_GIM], t1 = s * sc[gid * SC_STRIDE + SC_GRE];
    T0[2 * gid] = t0;
    T0[2 * gid + 1] = t1;
    c0[2 * gid] += t0;
    c0[2 * gid + 1] += t1;
  }
}

__global__ void k_set_state(DevState *st, long long step0, double *trace, double *norms, double *corr, double *pops,
                            const double *popU, int popk, double *energy, const double *epart, long long nbe,
                            int resume) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    st->step = step0;
    st->step0 = step0;
    st->pend = 0;
    if (!resume) st->bad_step = -1;
    st->keep_ref = resume;
    st->energy = energy;
    st->epart = epart;
    st->nbe = nbe;
    st->trace = trace;
    st->norms = norms;
    st->corr = corr;
    st->pops = pops;
    st->popU = popU;
    st->popk = popk;
  }
}

// Eigenstate populations (eq. populations) at k = step - step0: pops[k][r][I] = |<U_I, X_r>|^2
// with real unit vectors U_I over the amplitudes c_ia (both planes); one block per (RHS, state),
// blocks past the state count return at once, a fixed-order block reduction.
__global__ __launch_bounds__(256) void k_pop(int R, size_t ov, const double *__restrict__ X,
                                             const DevState *__restrict__ st) {
  __shared__ double sh[2][4];
  double *pops = st->pops;
  const int K = (int)st->popk, r = blockIdx.x, I = blockIdx.y;
  if (pops == nullptr || I >= K) return;
  const double *u = st->popU + (size_t)I * ov, *x = X + (size_t)r * 2 * ov;
  double re = 0.0, im = 0.0;
  for (size_t e = threadIdx.x; e < ov; e += 256) {
    re += u[e] * x[e];
    im += u[e] * x[ov + e];
  }
  re = wave_sum(re);
  im = wave_sum(im);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    sh[0][wave] = re;
    sh[1][wave] = im;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double a = (sh[0][0] + sh[0][1]) + (sh[0][2] + sh[0][3]), b = (sh[1][0] + sh[1][1]) + (sh[1][2] + sh[1][3]);
    const long long k = st->step + st->pend - st->step0;
    pops[(k * R + r) * K + I] = a * a + b * b;
  }
}

// Time-correlation function (eq. time_correlation_function): corr[k][r] = <Xref_r | X_r>
// = conj(x0ref) x0 + sum_ia conj(Xref_ia) X_ia at k = step - step0, one block per RHS (the two
// planes of length ov and the ground amplitude), a fixed-order block reduction.
__global__ __launch_bounds__(256) void k_corr(int R, size_t ov, const double *__restrict__ X,
                                              const double *__restrict__ X0, const double *__restrict__ xref,
                                              const double *__restrict__ xref0, const DevState *__restrict__ st) {
  __shared__ double sh[2][4];
  double *corr = st->corr;
  if (corr == nullptr) return;
  const int r = blockIdx.x;
  const double *x = X + (size_t)r * 2 * ov, *y = xref + (size_t)r * 2 * ov;
  double re = 0.0, im = 0.0;
  for (size_t e = threadIdx.x; e < ov; e += 256) {
    const double a0 = y[e], a1 = y[ov + e], b0 = x[e], b1 = x[ov + e];
    re += a0 * b0 + a1 * b1;
    im += a0 * b1 - a1 * b0;
  }
  re = wave_sum(re);
  im = wave_sum(im);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    sh[0][wave] = re;
    sh[1][wave] = im;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double g0 = xref0[2 * r], g1 = xref0[2 * r + 1], c0 = X0[2 * r], c1 = X0[2 * r + 1];
    const long long k = st->step + st->pend - st->step0;
    corr[(k * R + r) * 2] = (g0 * c0 + g1 * c1) + ((sh[0][0] + sh[0][1]) + (sh[0][2] + sh[0][3]));
    corr[(k * R + r) * 2 + 1] = (g0 * c1 - g1 * c0) + ((sh[1][0] + sh[1][1]) + (sh[1][2] + sh[1][3]));
  }
}

inline int grid_for(long long n, int block = 256, int cap = 8192) {
  long long g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (int)g;
}

}  // namespace

hipError_t launch_mu_blocks(hipStream_t s, const double *mu, const DevPulse *pulses, int o, int v, int R,
                            double *moo, double *mov, double *mvv) {
  const long long n = (long long)(o + v) * (o + v) * R;
  hipLaunchKernelGGL(k_mu_blocks, dim3(grid_for(n)), dim3(256), 0, s, mu, pulses, o, v, R, moo, mov, mvv);
  return hipGetLastError();
}

hipError_t launch_gaps(hipStream_t s, const double *e_occ, const double *e_virt, int o, int v, double *D) {
  hipLaunchKernelGGL(k_gaps, dim3(grid_for((long long)o * v)), dim3(256), 0, s, e_occ, e_virt, o, v, D);
  return hipGetLastError();
}

hipError_t launch_to_f32(hipStream_t s, const double *c, long long n, float *x32) {
  hipLaunchKernelGGL(k_to_f32, dim3(grid_for(n)), dim3(256), 0, s, c, n, x32);
  return hipGetLastError();
}

hipError_t launch_to_bf16x2(hipStream_t s, const double *c, long long n, float *x32, __hip_bfloat16 *hi,
                            __hip_bfloat16 *lo) {
  hipLaunchKernelGGL(k_to_bf16x2, dim3(grid_for(n)), dim3(256), 0, s, c, n, x32, hi, lo);
  return hipGetLastError();
}

int gemv1_chunks(int nq, int ov) {
  // independent of the slice count, so that a batch and a single RHS sum d identically
  if (nq <= 0 || ov <= 0) return 1;
  // as many ia chunks as keep the grid within one round of three workgroups per CU (the occupancy
  // of the six- and eight-slice forms' registers), so that no second, partly filled round follows
  const int blocks = (nq + 7) / 8;
  int es = std::max(1, std::min({768 / blocks, GEMV1_CHUNKS_MAX, ov / 2048}));
  const int echunk = (((ov + es - 1) / es) + 1023) / 1024 * 1024;
  return (ov + echunk - 1) / echunk;
}

template <typename TB>
static void gemv1_st(hipStream_t s, const TB *B, const float *X, int nq, int ov, int ns, int nes, float *dpart,
                     const FieldArgs &f) {
  constexpr int QT = 8;
  const int echunk = nes == 1 ? ov : (((ov + nes - 1) / nes) + 1023) / 1024 * 1024;
  auto go = [&](auto st) {
    constexpr int ST = decltype(st)::value;
    const dim3 grid(f.blocks + (nq + QT - 1) / QT * ((ns + ST - 1) / ST) * nes);
    auto run = [&](auto epl) {
      hipLaunchKernelGGL((k_gemv1<TB, QT, ST, decltype(epl)::value>), grid, dim3(256), 0, s, B, X, nq, ov, ns, echunk,
                         dpart, f);
    };
    if (ov % row_epl<TB>() == 0) run(std::integral_constant<int, row_epl<TB>()>{});
    else if (ov % 4 == 0) run(std::integral_constant<int, 4>{});
    else run(std::integral_constant<int, 1>{});
  };
  if (ns <= 2) go(std::integral_constant<int, 2>{});
  else if (ns <= 4) go(std::integral_constant<int, 4>{});
  else if (ns <= 6) go(std::integral_constant<int, 6>{});
  else go(std::integral_constant<int, 8>{});
}

hipError_t launch_gemv1(hipStream_t s, int b_dtype, const void *B, const float *X, int nq, int ov, int ns, int nes,
                        float *dpart, const FieldArgs &f) {
  if (b_dtype == RTTDA_BF16)
    gemv1_st(s, static_cast<const __hip_bfloat16 *>(B), X, nq, ov, ns, nes, dpart, f);
  else
    gemv1_st(s, static_cast<const float *>(B), X, nq, ov, ns, nes, dpart, f);
  return hipGetLastError();
}

template <typename TB>
static void gemv2_st(hipStream_t s, const TB *B, const float *dpart, int nes, int nq, int ov, int ns, int nsplit,
                     float *P) {
  constexpr int EPL = row_epl<TB>();
  auto go = [&](auto st) {
    constexpr int ST = decltype(st)::value;
    const int sy = (ns + ST - 1) / ST;
    if (ov % 4 == 0 && ov >= EPL)
      hipLaunchKernelGGL((k_gemv2<TB, ST, 4, EPL>), dim3((ov + 64 * EPL - 1) / (64 * EPL), sy, nsplit), dim3(256), 0, s,
                         B, dpart, nes, nq, ov, ns, nsplit, P);
    else
      hipLaunchKernelGGL((k_gemv2<TB, ST, 1, 1>), dim3((ov + 255) / 256, sy, nsplit), dim3(256), 0, s, B, dpart, nes, nq,
                         ov, ns, nsplit, P);
  };
  if (ns <= 2) go(std::integral_constant<int, 2>{});
  else if (ns <= 4) go(std::integral_constant<int, 4>{});
  else if (ns <= 6) go(std::integral_constant<int, 6>{});
  else go(std::integral_constant<int, 8>{});
}

hipError_t launch_gemv2(hipStream_t s, int b_dtype, const void *B, const float *dpart, int nes, int nq, int ov, int ns,
                        int nsplit, float *P) {
  if (b_dtype == RTTDA_BF16)
    gemv2_st(s, static_cast<const __hip_bfloat16 *>(B), dpart, nes, nq, ov, ns, nsplit, P);
  else
    gemv2_st(s, static_cast<const float *>(B), dpart, nes, nq, ov, ns, nsplit, P);
  return hipGetLastError();
}

hipError_t launch_field(hipStream_t s, const FieldArgs &f) {
  if (f.blocks > 0) hipLaunchKernelGGL(k_field, dim3(f.blocks), dim3(256), 0, s, f);
  return hipGetLastError();
}

hipError_t launch_scalar(hipStream_t s, int R, int nbf, int stage, int mode, double dt, const DevPulse *pulses,
                         DevState *st, const double *part, double *sc, double *c0, double *acc0, double *xs0,
                         double *out, double *normref, double *s0) {
  hipLaunchKernelGGL(k_scalar, dim3(R), dim3(256), 0, s, R, nbf, stage, mode, dt, pulses, st, part, sc, c0, acc0,
                     xs0, out, normref, s0);
  return hipGetLastError();
}

// go(PREC, GRP) for a launch's precision and slabs
template <typename F>
static void by_prec_and_groups(int prec, const Slabs &slabs, F go) {
  auto pick = [&](auto pr) {
    if (slabs.grp > 1) go(pr, std::true_type{});
    else go(pr, std::false_type{});
  };
  if (prec == RTTDA_PREC_MIXED_BF16) pick(std::integral_constant<int, 1>{});
  else pick(std::integral_constant<int, 0>{});
}

hipError_t launch_epilogue(hipStream_t s, int prec, int R, int o, int v, Slabs slabs, int stage, int mode,
                           int use_field, double dt, const double *D, const float *P, const double *F, double *sc,
                           const double *Xin, double *c, double *acc, double *xs64, float *x32, __hip_bfloat16 *xhi,
                           __hip_bfloat16 *xlo, double *s_out, double *epart, const StageScalars *scalars) {
  StageScalars es{};
  if (scalars) es = *scalars;
  const int nbe = epilogue_blocks((long long)o * v);
  dim3 grid(nbe + (es.mode ? 1 : 0), R);
  auto go = [&](auto pr, auto grp) {
    hipLaunchKernelGGL((k_epilogue<decltype(pr)::value, decltype(grp)::value>), grid, dim3(256), 0, s, R, o, v, slabs,
                       stage, mode, use_field, dt, D, P, F, sc, Xin, c, acc, xs64, x32, xhi, xlo, s_out, epart, nbe, es);
  };
  by_prec_and_groups(prec, slabs, go);
  return hipGetLastError();
}

int epilogue_blocks(long long ov) { return (int)std::min<long long>((ov + 63) / 64, EP_BX_MAX); }

hipError_t launch_sso_update(hipStream_t s, int prec, int R, int o, int v, Slabs slabs, int mode, int use_field,
                             double dt, const double *D, const float *P, const double *F, const double *sc, double *c,
                             double *c0, double *W, double *W0, float *x32, __hip_bfloat16 *xhi,
                             __hip_bfloat16 *xlo) {
  const long long n = (long long)R * o * v;
  dim3 grid(grid_for(n, 64, 65536));
  auto go = [&](auto pr, auto grp) {
    hipLaunchKernelGGL((k_sso_update<decltype(pr)::value, decltype(grp)::value>), grid, dim3(256), 0, s, R, o, v, slabs,
                       mode, use_field, dt, D, P, F, sc, c, c0, W, W0, x32, xhi, xlo);
  };
  by_prec_and_groups(prec, slabs, go);
  return hipGetLastError();
}

hipError_t launch_plane_copy(hipStream_t s, int prec, int R, size_t ov, int plane, const double *c, float *x32,
                             __hip_bfloat16 *xhi, __hip_bfloat16 *xlo) {
  const long long n = (long long)R * (long long)ov;
  dim3 grid(grid_for(n, 256, 65536));
  if (prec == RTTDA_PREC_MIXED_BF16)
    hipLaunchKernelGGL((k_plane_copy<1>), grid, dim3(256), 0, s, R, ov, plane, c, x32, xhi, xlo);
  else
    hipLaunchKernelGGL((k_plane_copy<0>), grid, dim3(256), 0, s, R, ov, plane, c, x32, xhi, xlo);
  return hipGetLastError();
}

int lz_blocks(long long n) { return (int)std::min<long long>(LZ_BLOCKS_MAX, std::max<long long>(1, (n + 63) / 64)); }

hipError_t launch_lz_init(hipStream_t s, long long n, double *v, double *part) {
  hipLaunchKernelGGL(k_lz_init, dim3(lz_blocks(n)), dim3(256), 0, s, n, v, part);
  return hipGetLastError();
}
hipError_t launch_lz_apply(hipStream_t s, long long n, int nslab, const double *D, const float *P, const double *v,
                           const double *vprev, const double *beta, double *w, double *part) {
  hipLaunchKernelGGL(k_lz_apply, dim3(lz_blocks(n)), dim3(256), 0, s, n, nslab, D, P, v, vprev, beta, w, part);
  return hipGetLastError();
}
hipError_t launch_lz_orth(hipStream_t s, long long n, const double *v, const double *dots, double *alpha, double *w,
                          double *part) {
  hipLaunchKernelGGL(k_lz_orth, dim3(lz_blocks(n)), dim3(256), 0, s, n, v, dots, alpha, w, part);
  return hipGetLastError();
}
hipError_t launch_lz_next(hipStream_t s, int prec, long long n, const double *dots, double *beta, const double *w,
                          double *v, double *vprev, float *x32, __hip_bfloat16 *xhi, __hip_bfloat16 *xlo, int shift) {
  if (prec == RTTDA_PREC_MIXED_BF16)
    hipLaunchKernelGGL((k_lz_next<1>), dim3(lz_blocks(n)), dim3(256), 0, s, n, dots, beta, w, v, vprev, x32, xhi, xlo,
                       shift);
  else
    hipLaunchKernelGGL((k_lz_next<0>), dim3(lz_blocks(n)), dim3(256), 0, s, n, dots, beta, w, v, vprev, x32, xhi, xlo,
                       shift);
  return hipGetLastError();
}

hipError_t launch_kick(hipStream_t s, int R, int ov, const DevPulse *pulses, const double *F, const double *sc,
                       double *c, double *c0) {
  const long long n = (long long)R * ov;
  hipLaunchKernelGGL(k_kick, dim3(grid_for(n)), dim3(256), 0, s, R, ov, pulses, F, sc, c, c0);
  return hipGetLastError();
}

hipError_t launch_kick_term(hipStream_t s, int R, int ov, const DevPulse *pulses, const double *F, const double *sc,
                            double inv_j, double *T, double *T0, double *c, double *c0) {
  const long long n = (long long)R * ov;
  hipLaunchKernelGGL(k_kick_term, dim3(grid_for(n)), dim3(256), 0, s, R, ov, pulses, F, sc, inv_j, T, T0, c, c0);
  return hipGetLastError();
}

hipError_t launch_set_state(hipStream_t s, DevState *st, long long step0, double *trace, double *norms,
                            double *corr, double *pops, const double *popU, int popk, double *energy,
                            const double *epart, long long nbe, int resume) {
  hipLaunchKernelGGL(k_set_state, dim3(1), dim3(64), 0, s, st, step0, trace, norms, corr, pops, popU, popk, energy,
                     epart, nbe, resume);
  return hipGetLastError();
}

// Kick spectra on a frequency grid (eq. fourier_transform, with the half-Hann window that
// equals a full Hann window on the mirrored record): for a dipole trace (kind 0)
//   S_s(w) = w sum_n h_n (mu_n - mu_0) sin(w t_n) dt / kappa,
// for the time-correlation function (kind 1)
//   S_s(w) = w Re sum_n h_n R_n exp(i w t_n) dt,
// with h_n = (1 + cos(pi n / N)) / 2, t_n = n dt, n = 0..N.
//
// Bound by FP64 arithmetic: one block of NT threads per SPW frequencies, its threads over the samples n = t,
// t + NT, ..., so that every frequency has NT sums in flight (one thread per frequency left most of
// the chip idle behind a serial chain of sincos: 24.9 ms for 20001 samples, three signals and 2001
// frequencies, 0.043 ms now).  A thread's phases advance by a rotation through NT w dt (and the
// window's by NT pi / N), set afresh from sincos every SPREF samples, so that the rotation's
// rounding stays near that of the arguments themselves.  Signals are taken SPS at a time; the block
// sum runs in a fixed order.  A record of up to SPEC_SHORT samples takes blocks of one wave: where there are
// many frequencies a thread's first sincos cost more than its few samples (100000 frequencies, one signal: 200
// samples 211 -> 66 us, 1000 samples 236 -> 97 us; 2000 samples of one frequency would take 15 us for 11).  Still
// shorter records of many frequencies take a thread per frequency, which has its samples' sincos and no others
// (100000 frequencies: 1 sample 5 us, 10 samples 10, 64 samples 47, where a wave each takes 48; 2000
// frequencies of 30 samples would take 15 for 7).
// average: out[w] = the mean over the signals (eq. spectrum_average) instead of out[s][w].
constexpr int SPW = 4, SPS = 3, SPREF = 32;
constexpr int SPEC_SHORT = 1024;
inline bool spec_each(int n_t, int n_w) { return n_t <= 128 && n_w >= 1024 * n_t; }

// one thread per frequency
template <int KIND>
__global__ __launch_bounds__(256) void k_spectrum_each(const double *__restrict__ sig, int n_t, int nsig, double dt,
                                                       double kappa, int n_w, double w0, double dw, int average,
                                                       double *__restrict__ out) {
  const int wi = blockIdx.x * 256 + threadIdx.x;
  if (wi >= n_w) return;
  const double w = w0 + dw * wi;
  const int N = n_t - 1;
  double mean = 0.0;
  for (int s0 = 0; s0 < nsig; s0 += SPS) {
    double acc[SPS] = {};
    for (int n = 0; n < n_t; ++n) {
      const double h = N > 0 ? 0.5 * (1.0 + cos(M_PI * (double)n / N)) : 1.0;
      double sn, cs;
      sincos(w * (n * dt), &sn, &cs);
#pragma unroll
      for (int s = 0; s < SPS; ++s) {
        if (s0 + s >= nsig) break;
        const size_t e = (size_t)n * nsig + s0 + s;
        acc[s] += KIND == 0 ? h * (sig[e] - sig[s0 + s]) * sn : h * (sig[2 * e] * cs - sig[2 * e + 1] * sn);
      }
    }
#pragma unroll
    for (int s = 0; s < SPS; ++s) {
      if (s0 + s >= nsig) break;
      const double val = KIND == 0 ? w * acc[s] * dt / kappa : w * acc[s] * dt;
      if (average)
        mean += val;
      else
        out[(size_t)(s0 + s) * n_w + wi] = val;
    }
  }
  if (average) out[wi] = mean / nsig;
}

template <int KIND, int NT>
__global__ __launch_bounds__(NT) void k_spectrum(const double *__restrict__ sig, int n_t, int nsig, double dt,
                                                  double kappa, int n_w, double w0, double dw, int average,
                                                  double *__restrict__ out) {
  __shared__ double red[NT / 64][SPW][SPS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int w_base = blockIdx.x * SPW;
  const int N = n_t - 1;
  double w[SPW], rc[SPW], rs[SPW];  // frequencies and the rotations through NT samples
#pragma unroll
  for (int k = 0; k < SPW; ++k) {
    w[k] = w0 + dw * (w_base + k);
    rs[k] = 0.0, rc[k] = 1.0;
    if (n_t > NT) sincos(w[k] * (NT * dt), &rs[k], &rc[k]);
  }
  double hrs = 0.0, hrc = 1.0;
  if (n_t > NT) sincos(M_PI * (double)NT / N, &hrs, &hrc);
  double mean = 0.0;  // thread k < SPW: frequency w_base + k
  for (int s0 = 0; s0 < nsig; s0 += SPS) {
    const int ns = min(SPS, nsig - s0);
    double base[SPS], acc[SPW][SPS];
#pragma unroll
    for (int s = 0; s < SPS; ++s) {
      base[s] = KIND == 0 && s < ns ? sig[s0 + s] : 0.0;
#pragma unroll
      for (int k = 0; k < SPW; ++k) acc[k][s] = 0.0;
    }
    for (long long n0 = tid; n0 < n_t; n0 += NT * SPREF) {
      double sn[SPW], cs[SPW], hs = 0.0, hc = 1.0;
#pragma unroll
      for (int k = 0; k < SPW; ++k) sincos(w[k] * (n0 * dt), &sn[k], &cs[k]);
      if (N > 0) sincos(M_PI * (double)n0 / N, &hs, &hc);
      const long long n1 = min((long long)n_t, n0 + NT * SPREF);
      for (long long n = n0; n < n1; n += NT) {
        const double h = 0.5 * (1.0 + hc);
        double a[SPS], b[SPS];  // windowed sample: the trace, or the real and imaginary correlation
#pragma unroll
        for (int s = 0; s < SPS; ++s) {
          a[s] = b[s] = 0.0;
          if (s < ns) {
            const size_t e = (size_t)n * nsig + s0 + s;
            if (KIND == 0) {
              a[s] = h * (sig[e] - base[s]);
            } else {
              a[s] = h * sig[2 * e];
              b[s] = h * sig[2 * e + 1];
            }
          }
        }
#pragma unroll
        for (int k = 0; k < SPW; ++k) {
#pragma unroll
          for (int s = 0; s < SPS; ++s) {
            if (KIND == 0)
              acc[k][s] = fma(a[s], sn[k], acc[k][s]);
            else
              acc[k][s] += a[s] * cs[k] - b[s] * sn[k];
          }
          const double t = cs[k] * rc[k] - sn[k] * rs[k];
          sn[k] = sn[k] * rc[k] + cs[k] * rs[k];
          cs[k] = t;
        }
        const double t = hc * hrc - hs * hrs;
        hs = hs * hrc + hc * hrs;
        hc = t;
      }
    }
    __syncthreads();  // red of the previous signals has been read
#pragma unroll
    for (int k = 0; k < SPW; ++k)
#pragma unroll
      for (int s = 0; s < SPS; ++s) {
        const double t = wave_sum(acc[k][s]);
        if (lane == 0) red[wave][k][s] = t;
      }
    __syncthreads();
    if (tid < SPW && w_base + tid < n_w) {
      const double wk = w0 + dw * (w_base + tid);
      for (int s = 0; s < ns; ++s) {
        double sum = red[0][tid][s];
        if constexpr (NT == 256) sum = (sum + red[1][tid][s]) + (red[2][tid][s] + red[3][tid][s]);
        const double val = KIND == 0 ? wk * sum * dt / kappa : wk * sum * dt;
        if (average)
          mean += val;
        else
          out[(size_t)(s0 + s) * n_w + w_base + tid] = val;
      }
    }
  }
  if (average && tid < SPW && w_base + tid < n_w) out[w_base + tid] = mean / nsig;
}

hipError_t launch_spectrum(hipStream_t s, int kind, const double *sig, int n_t, int nsig, double dt, double kappa,
                           int n_w, double w0, double dw, int average, double *out) {
  const dim3 grid((n_w + SPW - 1) / SPW);
  auto go = [&](auto k, auto nt) {
    constexpr int NT = decltype(nt)::value;
    hipLaunchKernelGGL((k_spectrum<decltype(k)::value, NT>), grid, dim3(NT), 0, s, sig, n_t, nsig, dt, kappa, n_w, w0,
                       dw, average, out);
  };
  auto pick = [&](auto k) {
    if (spec_each(n_t, n_w))
      hipLaunchKernelGGL((k_spectrum_each<decltype(k)::value>), dim3((n_w + 255) / 256), dim3(256), 0, s, sig, n_t, nsig,
                         dt, kappa, n_w, w0, dw, average, out);
    else if (n_t <= SPEC_SHORT) go(k, std::integral_constant<int, 64>{});
    else go(k, std::integral_constant<int, 256>{});
  };
  if (kind == 0) pick(std::integral_constant<int, 0>{});
  else pick(std::integral_constant<int, 1>{});
  return hipGetLastError();
}

hipError_t launch_pop(hipStream_t s, int R, size_t ov, const double *X, const DevState *st) {
  hipLaunchKernelGGL(k_pop, dim3(R, POP_MAX), dim3(256), 0, s, R, ov, X, st);
  return hipGetLastError();
}

hipError_t launch_corr(hipStream_t s, int R, size_t ov, const double *X, const double *X0, const double *xref,
                       const double *xref0, const DevState *st) {
  hipLaunchKernelGGL(k_corr, dim3(R), dim3(256), 0, s, R, ov, X, X0, xref, xref0, st);
  return hipGetLastError();
}

}  // namespace rttda
