// Coulomb pair on the FP32 matrix cores for many slices (a batch of 16 or more right-hand sides):
// with 2R slices the two products are skinny GEMMs, d = B_ov X^T (N_Q x 2R) and J = 2 d^T B_ov
// (2R x ov), and the vector-unit GEMVs that serve a few slices spend most of a step's compute on
// them.  v_mfma_f32_16x16x4f32: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; register t
// of the result is D[4 (l / 16) + t][l % 16].  Operands are staged in LDS with coalesced loads
// (BF16 factors are widened to FP32 on the way).  Each output element is a fixed-order sum whose
// order does not depend on the slice count, so a batch and one of its RHS alone give the same d
// and J bitwise.
#include <type_traits>

#include "common.h"
#include "field.h"

namespace rttda {
namespace {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef f4v f4u __attribute__((aligned(4)));
typedef unsigned u2v __attribute__((ext_vector_type(2)));
typedef u2v u2u __attribute__((aligned(2)));

__device__ __forceinline__ float ld(const float *p, size_t i) { return p[i]; }
__device__ __forceinline__ float ld(const __hip_bfloat16 *p, size_t i) { return __bfloat162float(p[i]); }
__device__ __forceinline__ f4v ld4(const float *p, size_t i) { return *reinterpret_cast<const f4u *>(p + i); }
__device__ __forceinline__ f4v ld4(const __hip_bfloat16 *p, size_t i) {
  const u2v w = *reinterpret_cast<const u2u *>(p + i);
  return f4v{__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xffff0000u), __uint_as_float(w[1] << 16),
             __uint_as_float(w[1] & 0xffff0000u)};
}

constexpr int CM_QT = 64;   // Q rows per workgroup of the first product (16 per wave)
constexpr int CM_KT = 32;   // K values staged per LDS round
constexpr int CM_IT = 64;   // ia columns per workgroup of the second product (16 per wave)

// A tile of ROWS x COLS values (a multiple of 1024) on its way to LDS, four neighbours of a row per thread
// and piece.  Rows below nrow, columns below ncol exist; the others are zero.  They are read from a clamped
// place all the same: a condition on a load makes it wait for the one before it.  V4: columns come whole
// in fours (one load), else one by one.
template <int ROWS, int COLS, bool V4>
struct Tile {
  static constexpr int N = ROWS * COLS / 1024;
  static_assert(ROWS * COLS % 1024 == 0, "whole pieces");
  f4v x[N];
  template <typename T>
  __device__ __forceinline__ void load(const T *p, size_t stride, int nrow, int ncol) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int t = (int)threadIdx.x + 256 * i, r = t / (COLS / 4), c = 4 * (t % (COLS / 4));
      const size_t row = (size_t)min(r, nrow - 1) * stride;
      if constexpr (V4) {
        x[i] = ld4(p, row + (c < ncol ? c : 0));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[i][e] = ld(p, row + min(c + e, ncol - 1));
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) x[i][e] = r < nrow && c + e < ncol ? x[i][e] : 0.f;
    }
  }
  template <int LD>
  __device__ __forceinline__ void store(float (&to)[ROWS][LD]) const {
    static_assert(LD % 4 == 0, "16-byte LDS writes");
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int t = (int)threadIdx.x + 256 * i, r = t / (COLS / 4), c = 4 * (t % (COLS / 4));
      *reinterpret_cast<f4v *>(&to[r][c]) = x[i];
    }
  }
};

// dpart[chunk][q][s] = sum over the chunk's ia of B[q][ia] X[s][ia]; workgroups: (Q blocks, slice blocks,
// chunks), one or so per CU, then those of the field product beside them.  NJ blocks of 16 slices per
// workgroup: no more than the batch has, up to 8.  The next round's operands are loaded while this one is
// multiplied; the LDS rows' lengths (36 words) put the 64 lanes' reads in distinct banks.
// o40 v300 N_Q1000, pair and field product: 64 RHS 174 us, 16 RHS 57 us (375 and 241 with a round's loads one
// after the other, eight blocks always and the field product in a launch of its own).
template <typename TB, bool V4, int NJ>
__global__ __launch_bounds__(256) void k_coul1_mfma(const TB *__restrict__ B, const float *__restrict__ X, int nq,
                                                    int ov, int ns, int echunk, float *__restrict__ dpart,
                                                    FieldArgs f) {
  constexpr int CM_ST = 16 * NJ;
  const int lb = blockIdx.x, nmain = (int)gridDim.x - f.blocks;
  if (lb >= nmain) {
    field_block(f, lb - nmain);
    return;
  }
  __shared__ __attribute__((aligned(16))) float As[CM_QT][CM_KT + 4];
  __shared__ __attribute__((aligned(16))) float Bs[CM_ST][CM_KT + 4];
  const int nqb = (nq + CM_QT - 1) / CM_QT, nsb = (ns + CM_ST - 1) / CM_ST;
  const int q0 = lb % nqb * CM_QT, s0 = lb / nqb % nsb * CM_ST, ch = lb / (nqb * nsb);
  const int e0 = ch * echunk, e1 = min(ov, e0 + echunk);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  f4v acc[CM_ST / 16];
#pragma unroll
  for (int j = 0; j < CM_ST / 16; ++j) acc[j] = f4v{0.f, 0.f, 0.f, 0.f};
  Tile<CM_QT, CM_KT, V4> ta;
  Tile<CM_ST, CM_KT, V4> tb;
  auto load = [&](int e) {
    ta.load(B + (size_t)q0 * ov + e, ov, nq - q0, e1 - e);
    tb.load(X + (size_t)s0 * ov + e, ov, ns - s0, e1 - e);
  };
  load(e0);
  for (int e = e0; e < e1; e += CM_KT) {
    __syncthreads();  // the previous round's operands have been read
    ta.store(As);
    tb.store(Bs);
    __syncthreads();
    if (e + CM_KT < e1) load(e + CM_KT);
#pragma unroll
    for (int kk = 0; kk < CM_KT / 4; ++kk) {
      const float a = As[16 * wave + li][4 * kk + lk];
#pragma unroll
      for (int j = 0; j < CM_ST / 16; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, Bs[16 * j + li][4 * kk + lk], acc[j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < CM_ST / 16; ++j)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int q = q0 + 16 * wave + 4 * lk + t, sl = s0 + 16 * j + li;
      if (q < nq && sl < ns) dpart[((size_t)ch * nq + q) * ns + sl] = acc[j][t];
    }
}

// chunk partials of d added into chunk 0's place, in order, eight loads in flight
__global__ void k_dsum_m(float *__restrict__ dpart, int n, int nes) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
    float d = dpart[e];
    for (int k = 1; k < nes; k += 8) {
      float t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = dpart[(size_t)min(k + u, nes - 1) * n + e];
#pragma unroll
      for (int u = 0; u < 8; ++u) d = k + u < nes ? d + t[u] : d;
    }
    dpart[e] = d;
  }
}

// P[split][s][ia] = 2 sum_{Q in split} d[Q][s] B[Q][ia]; grid (ia blocks, slice blocks, splits)
template <typename TB, bool V4, int NJ>
__global__ __launch_bounds__(256) void k_coul2_mfma(const TB *__restrict__ B, const float *__restrict__ d, int nq,
                                                    int ov, int ns, int nsplit, float *__restrict__ P) {
  constexpr int CM_ST = 16 * NJ;
  __shared__ __attribute__((aligned(16))) float Ds[CM_KT][CM_ST + 16];  // [Q][s]
  __shared__ __attribute__((aligned(16))) float Bs[CM_KT][CM_IT + 16];  // [Q][ia]
  const int e0 = blockIdx.x * CM_IT, s0 = blockIdx.y * CM_ST, sp = blockIdx.z;
  const int qa = (int)((long long)sp * nq / nsplit), qb = (int)((long long)(sp + 1) * nq / nsplit);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  f4v acc[CM_ST / 16];
#pragma unroll
  for (int j = 0; j < CM_ST / 16; ++j) acc[j] = f4v{0.f, 0.f, 0.f, 0.f};
  Tile<CM_KT, CM_ST, false> td;
  Tile<CM_KT, CM_IT, V4> tb;
  auto load = [&](int q) {
    td.load(d + (size_t)q * ns + s0, ns, qb - q, ns - s0);
    tb.load(B + (size_t)q * ov + e0, ov, qb - q, ov - e0);
  };
  if (qa < qb) load(qa);
  for (int q = qa; q < qb; q += CM_KT) {
    __syncthreads();
    td.store(Ds);
    tb.store(Bs);
    __syncthreads();
    if (q + CM_KT < qb) load(q + CM_KT);
#pragma unroll
    for (int kk = 0; kk < CM_KT / 4; ++kk) {
      const float b = Bs[4 * kk + lk][16 * wave + li];
#pragma unroll
      for (int j = 0; j < CM_ST / 16; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(Ds[4 * kk + lk][16 * j + li], b, acc[j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < CM_ST / 16; ++j)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int sl = s0 + 16 * j + 4 * lk + t, ia = e0 + 16 * wave + li;
      if (sl < ns && ia < ov) P[((size_t)sp * ns + sl) * ov + ia] = 2.f * acc[j][t];
    }
}

}  // namespace

int coulomb_mfma_chunks(int nq, int ov) {
  // independent of the slice count (a batch and one of its RHS alone sum d the same way): about
  // 256 workgroups for the first product, at most GEMV1_CHUNKS_MAX chunks of at least 128 ia
  const int qblocks = (nq + CM_QT - 1) / CM_QT;
  const int want = (256 + qblocks - 1) / qblocks;
  return std::max(1, std::min({want, GEMV1_CHUNKS_MAX, std::max(1, ov / 128)}));
}

template <typename TB>
static void coulomb_mfma(hipStream_t s, const TB *B, const float *X, int nq, int ov, int ns, int nes, int nsplit,
                         float *dpart, float *P, const FieldArgs &f) {
  const int echunk = ((ov + nes - 1) / nes + CM_KT - 1) / CM_KT * CM_KT;
  const int nch = (ov + echunk - 1) / echunk;
  auto go = [&](auto v4, auto nj) {
    constexpr bool V4 = decltype(v4)::value;
    constexpr int NJ = decltype(nj)::value;
    const int nsb = (ns + 16 * NJ - 1) / (16 * NJ);
    const dim3 g1(f.blocks + (nq + CM_QT - 1) / CM_QT * nsb * nch), g2((ov + CM_IT - 1) / CM_IT, nsb, nsplit);
    hipLaunchKernelGGL((k_coul1_mfma<TB, V4, NJ>), g1, dim3(256), 0, s, B, X, nq, ov, ns, echunk, dpart, f);
    if (nch > 1)
      hipLaunchKernelGGL(k_dsum_m, dim3(std::max(1, std::min(1024, (nq * ns + 255) / 256))), dim3(256), 0, s, dpart,
                         nq * ns, nch);
    hipLaunchKernelGGL((k_coul2_mfma<TB, V4, NJ>), g2, dim3(256), 0, s, B, dpart, nq, ov, ns, nsplit, P);
  };
  auto pick = [&](auto nj) {
    if (ov % 4 == 0) go(std::true_type{}, nj);  // no group of four values crosses the end of a row
    else go(std::false_type{}, nj);
  };
  if (ns <= 32) pick(std::integral_constant<int, 2>{});
  else if (ns <= 64) pick(std::integral_constant<int, 4>{});
  else pick(std::integral_constant<int, 8>{});
}

hipError_t launch_coulomb_mfma(hipStream_t s, int b_dtype, const void *B, const float *X, int nq, int ov, int ns,
                               int nes, int nsplit, float *dpart, float *P, const FieldArgs &f) {
  if (b_dtype == RTTDA_BF16)
    coulomb_mfma(s, static_cast<const __hip_bfloat16 *>(B), X, nq, ov, ns, nes, nsplit, dpart, P, f);
  else
    coulomb_mfma(s, static_cast<const float *>(B), X, nq, ov, ns, nes, nsplit, dpart, P, f);
  return hipGetLastError();
}

}  // namespace rttda
