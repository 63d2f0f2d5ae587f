// Exchange contraction for large o in split BF16 precision, as two batched GEMMs per chunk of Q
// instead of one fused kernel (the fused kernels keep W = X B_vv^Q on chip, which forces a
// workgroup tile of one slice's rows and re-reads all of X for every (Q, column tile); at large o
// that re-read traffic, not the matrix cores, sets the time):
//
//   (A) W^Q = X B_vv^Q for all stacked rows r = (slice, i) of X at once, with X = X_hi + X_lo and
//       FP32 accumulation on v_mfma_f32_32x32x16_bf16; the workgroup tile is 256 columns (of a chunk's Q one
//       after the other) x 256 or 192 rows, and the result is stored transposed, W^T[Q][c][r], as BF16 hi
//       and lo planes.
//   (B) P[ks][s] (+)= scale * sum_{Q in split ks} B_oo^Q W_s^Q with W = W_hi + W_lo: a GEMM whose
//       reduction index runs over (Q, j); the slab of split ks is stored by the first chunk and
//       read-modified-written (same thread, fixed order) by later chunks.
//
// The exchange term is the c_x sum_Q B^Q_ij B^Q_ab part of the DF hybrid A (section "Real-Time
// TDA", the A matrix elements with the exact-exchange fraction c_x).  Both kernels stage operand
// tiles with gfx950 global_load_lds (16 bytes per lane) into three XOR-swizzled LDS buffers; loads
// of chunk c+2 are in flight while chunk c is multiplied; waits count vmcnt explicitly and the
// barrier drains only LDS reads.  Needs v % 8 == 0 (16-byte rows); a slice's o rows are padded to a
// multiple of 8 in W, in the staged X and, where o is none, in a copy of B_oo.
//
// o240 v1800, 3 RHS, per 400 Q: 10.2 -> 7.9 ms.  Of the 10.2: tiles that ended with each Q's columns
// (v = 7 x 256 + 8), 0.6; a chunk's loads issued in one burst, which held up the matrix instructions behind
// it, 0.5; X's 64-byte row pieces, W's 2-byte stores and the pipeline drained around them once per tile,
// 1.0; and in (B) the old slab values read one after the other, 0.2.  (A) alone now runs at 1.2 PFLOP/s, as
// a plain bf16 product of 8192^3 does there; skipping its loads would take 28 % off the time before.
// o96 v720 N_Q1920, one RHS: 1.57 -> 1.22 ms (1.47 with the 192-row tile alone).
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace rttda {
namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;

__device__ __attribute__((aligned(256))) unsigned int g_zero_page_g[64];  // 256 zero bytes

constexpr int KC = 32;  // bf16 per chunk row: 64 bytes = four 16-byte chunks

// XOR swizzle of the four 16-byte chunks of a 64-byte row: the 16-byte reads of 8 consecutive rows
// (one 128-byte bank sweep) and of 16 consecutive rows (one 256-byte sweep) at one logical chunk all
// land in distinct bank groups
__device__ __forceinline__ int swz(int r) { return ((r >> 1) & 3) ^ ((r >> 3) & 1); }

__device__ __forceinline__ void dma16(const void *src, void *lds_base) {
  __builtin_amdgcn_global_load_lds(src, (lds_void *)lds_base, 16, 0, 0);
}

template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xF | (7 << 4) | (0 << 8) | (3 << 14));
  asm volatile("s_barrier" ::: "memory");
}

__device__ __forceinline__ f16v zero16() {
  f16v z;
#pragma unroll
  for (int t = 0; t < 16; ++t) z[t] = 0.f;
  return z;
}

// logical workgroup id: consecutive ids on one XCD (hardware deals workgroups round robin)
__device__ __forceinline__ int xcd_local_id() {
  const int per_xcd = (int)gridDim.x / 8;
  return (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
}

// ---------------------------------------------------------------------------------------------
// X hi/lo in the order kernel (A) stages it: Xt[kc][rt][hi rows | lo rows][32], a slice's rows padded to op
// (a multiple of 8), the four 16-byte groups of a row swizzled as in LDS, padding and columns past v zero.  A load instruction of (A) then reads
// 1 KiB in a row instead of 64 bytes of sixteen rows (half-used lines, and split ones where a row is not
// a multiple of 128 bytes).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_xgemm_x(const __bf16 *__restrict__ Xh, const __bf16 *__restrict__ Xl, int o,
                                                 int op, int v, int M, int tr, int n_rt, int nkc,
                                                 __bf16 *__restrict__ Xt) {
  const size_t total = (size_t)nkc * n_rt * tr * 8;  // 16-byte groups
  for (size_t k = blockIdx.x * (size_t)256 + threadIdx.x; k < total; k += (size_t)gridDim.x * 256) {
    const int g = (int)(k & 3);
    const size_t row = k >> 2;  // ((kc * n_rt + rt) * 2 + plane) * tr + r
    const int r = (int)(row % tr), pl = (int)(row / tr) & 1;
    const size_t tile = row / (2 * tr);
    const int m = (int)(tile % n_rt) * tr + r, a = (int)(tile / n_rt) * KC + 8 * (g ^ swz(r));
    const bool live = m < M && m % op < o && a < v;
    const bf8 x =
        *reinterpret_cast<const bf8 *>((pl ? Xl : Xh) + (live ? ((size_t)(m / op) * o + m % op) * v + a : 0));
    *reinterpret_cast<bf8 *>(Xt + 8 * k) = live ? x : bf8{};
  }
}

// B_oo of a chunk of Q with rows and columns padded to op (a multiple of 8) by zeros, for the 16-byte loads
// of kernel (B): o96 v720 N_Q1920's 35 MB would take about 15 us of 1230
__global__ __launch_bounds__(256) void k_xgemm_o(const __bf16 *__restrict__ Boo, int o, int op, int nqc,
                                                 __bf16 *__restrict__ Ot) {
  const int ng = op / 8;
  const size_t total = (size_t)nqc * op * ng;
  for (size_t k = blockIdx.x * (size_t)256 + threadIdx.x; k < total; k += (size_t)gridDim.x * 256) {
    const int g = (int)(k % ng), i = (int)(k / ng % op);
    const __bf16 *row = Boo + (k / ng / op * o + min(i, o - 1)) * o;
    bf8 x;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const __bf16 t = row[min(8 * g + j, o - 1)];
      x[j] = i < o && 8 * g + j < o ? t : (__bf16)0.f;
    }
    *reinterpret_cast<bf8 *>(Ot + 8 * k) = x;
  }
}

// ---------------------------------------------------------------------------------------------
// (A) W^T[n][r] = sum_b B_vv[n][b] X[r][b] over the flattened columns n = (qq, c) of a chunk of Q
//     (B_vv symmetric: row c = column c), so that no tile but the last is partly empty, whatever v is
// Waves: NWC along n x NWR along r; each wave CB x RB blocks of 32 x 32.  One workgroup per CU takes
// tile after tile without draining its loads: the next tile's first two chunks load during the last two
// of the current one, and a tile's stores (through a block of LDS per wave, 16 bytes per lane) are waited
// for two chunks into the next.
// ---------------------------------------------------------------------------------------------
template <int NWC, int NWR, int CB, int RB>
struct CfgA {
  static constexpr int NW = NWC * NWR, NT = 64 * NW;
  static constexpr int TC = NWC * CB * 32, TR = NWR * RB * 32;
  static constexpr int ROWS = TC + 2 * TR;     // tile rows per buffer: B_vv, X hi, X lo
  static constexpr int NL = ROWS / (16 * NW);  // 16-row load instructions per wave and chunk
  static constexpr int NS = 4 * CB * RB;       // 16-byte store instructions per wave and tile
  static constexpr size_t LDS = ((size_t)3 * ROWS * KC + NW * 1024) * 2;
  static_assert(ROWS % (16 * NW) == 0, "tile rows split into whole load instructions");
  static_assert(NL + NS < 64, "loads and stores in flight within the wait counter");
  static_assert(LDS <= 160 * 1024, "LDS");
};

template <int NWC, int NWR, int CB, int RB>
__global__ __launch_bounds__(64 * NWC * NWR, 1) void k_xgemm_w(const __bf16 *__restrict__ Bvv,
                                                               const __bf16 *__restrict__ Xt, int v, int M, int N,
                                                               int n_ct, int n_rt, __bf16 *__restrict__ Wh,
                                                               __bf16 *__restrict__ Wl) {
  using C = CfgA<NWC, NWR, CB, RB>;
  constexpr int NL = C::NL, TC = C::TC, TR = C::TR, ROWS = C::ROWS;
  extern __shared__ __attribute__((aligned(16))) __bf16 ldsa[];  // [3][B_vv TC | X hi TR | X lo TR][32], [NW][32][32]

  // tile order: the row tiles of one column tile are adjacent and share its rows of B_vv in L2 (row
  // tiles varying slowest, which keeps a tile of X in L2 instead, took 3..11 % longer for 3 RHS)
  const int n_tiles = n_ct * n_rt;
  int tile = xcd_local_id();  // the tile that is multiplied, in steps of the grid
  if (tile >= n_tiles) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, m = lane & 31, lrow = lane >> 2;
  const int wc = wave / NWR, wr = wave % NWR;
  const int nkc = (v + KC - 1) / KC;
  // the zero page's address stays in registers for the whole kernel (re-deriving it inside the
  // loop puts a scalar memory load among the LDS reads, which forces full LDS waits)
  const void *zp = g_zero_page_g;
  asm volatile("" : "+s"(zp));

  // The stream of loads: chunk after chunk of tile after tile, two chunks ahead of the products.  A load
  // takes 16 tile rows, each lane its 16-byte group, swizzled within the row; where they lie is kept in
  // scalar registers (bases of the tile and chunk), the lane's part is the same for every load.  Past the
  // last tile it is loaded again, into buffers that nothing reads.
  const int a_lane = 8 * ((lane & 3) ^ swz(lrow));
  const unsigned row_bytes = 2u * v, va = lrow * row_bytes + 2 * a_lane, vx = 16 * lane;
  unsigned uo[NL];  // a load's first row: bytes from the tile's
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int u = (wave * NL + k) * 16;
    uo[k] = u < TC ? u * row_bytes : (unsigned)(u - TC) * (KC * 2);
  }
  const char *pa = nullptr, *px = nullptr;  // the chunk to load: B_vv rows, X
  int lt = tile, la = 0, lrows = 0, lbuf = 0;  // its tile, first b, the tile's count of B_vv rows, its buffer
  const size_t xstep = (size_t)n_rt * 2 * TR * KC * 2;
  auto load_tile = [&]() {
    const int t = min(lt, n_tiles - 1), c0 = (t / n_rt) * TC;
    pa = reinterpret_cast<const char *>(Bvv) + (size_t)c0 * row_bytes;
    px = reinterpret_cast<const char *>(Xt) + (size_t)(t % n_rt) * 2 * TR * KC * 2;
    lrows = N - c0;
    la = 0;
  };
  auto issue1 = [&](int k) {  // loads 0..NL-1 of a chunk, in order
    const int u = (wave * NL + k) * 16;
    const bool is_a = u < TC;
    const int k_lim = is_a ? v - la : KC, r_lim = is_a ? lrows - u : 16;
    const char *src = (is_a ? pa + 0 : px + 0) + uo[k] + (is_a ? va : vx);
    const bool ok = (a_lane < k_lim) & (lrow < r_lim);
    dma16(ok ? (const void *)src : zp, ldsa + lbuf * (ROWS * KC) + u * KC);
    if (k == NL - 1) {
      lbuf = lbuf == 2 ? 0 : lbuf + 1;
      la += KC;
      pa += 2 * KC;
      px += xstep;
      if (la >= v) {
        lt += gridDim.x;
        load_tile();
      }
    }
  };

  f16v acc[CB][RB];
  struct Frag {
    bf8 a[CB], xh[RB], xl[RB];
  };
  auto read_step = [&](int buf, int u, Frag &F) {
    const __bf16 *As = ldsa + buf * (ROWS * KC), *Xhs = As + TC * KC, *Xls = Xhs + TR * KC;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const int r = (wc * CB + cb) * 32 + m;
      F.a[cb] = *reinterpret_cast<const bf8 *>(&As[r * KC + 8 * ((2 * u + h) ^ swz(r))]);
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int r = (wr * RB + rb) * 32 + m;
      F.xh[rb] = *reinterpret_cast<const bf8 *>(&Xhs[r * KC + 8 * ((2 * u + h) ^ swz(r))]);
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int r = (wr * RB + rb) * 32 + m;
      F.xl[rb] = *reinterpret_cast<const bf8 *>(&Xls[r * KC + 8 * ((2 * u + h) ^ swz(r))]);
    }
  };
  // one half of a K step's products, X_hi (part 0) or X_lo (part 1) against the B_vv fragments, with
  // loads [k0, k1) spread between its column blocks (in one burst they block the matrix instructions
  // behind them while the address unit takes the eight waves' loads)
  auto mfma_part = [&](auto ncb_tag, const Frag &F, int part, int k0, int k1) {
    constexpr int NCB = decltype(ncb_tag)::value;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      if (cb < NCB) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
          acc[cb][rb] =
              __builtin_amdgcn_mfma_f32_32x32x16_bf16(part ? F.xl[rb] : F.xh[rb], F.a[cb], acc[cb][rb], 0, 0, 0);
      }
      if (k0 < k1) {
        __builtin_amdgcn_sched_barrier(0);
        const int ka = k0 + (k1 - k0) * cb / CB, kb = k0 + (k1 - k0) * (cb + 1) / CB;
#pragma unroll
        for (int k = ka; k < kb; ++k) issue1(k);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  // The pipelined loop over one tile's chunks, specialised on this wave's count of valid column blocks
  // (wave-uniform; only the last column tile has fewer than CB).  Choosing the specialisation once,
  // outside the loop, keeps branches out of it.  Waves without valid blocks (NCB = 0) still take part in
  // every load and barrier.  Per chunk, after the barrier that publishes it: read K step 0's fragments
  // (F0), run K step 1 of the chunk before (F1, read before the barrier) while they arrive, then the X_hi
  // half of K step 0, then read K step 1's fragments into F1 while the X_lo half runs.  The loads of the
  // chunk two ahead go into the buffer of the chunk before; past the last tile they load that tile again,
  // which keeps the loop free of branches around the loads.
  int rbuf = 0;
  bool stored = false;  // exactly NS stores of the tile before may be in flight behind the loads
  auto main_loop = [&](auto ncb_tag) {
    Frag F0, F1;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) F1.a[cb] = bf8{};  // "K step 1 of chunk -1": adds zero
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) F1.xh[rb] = F1.xl[rb] = bf8{};
    for (int kc = 0; kc < nkc; ++kc) {
      // this chunk has landed; the next one's loads and, for two chunks, the stores between them and the
      // following loads may be in flight (memory operations of a wave complete in order)
      if (stored && kc < 2)
        wait_vm<NL + C::NS>();
      else
        wait_vm<NL>();
      lds_barrier();  // publishes the chunk; every wave has read the chunk before it
      __builtin_amdgcn_sched_barrier(0);
      read_step(rbuf, 0, F0);
      __builtin_amdgcn_sched_barrier(0);
      // second K step of chunk kc-1 (a full chunk: only the last chunk can end inside a step)
      mfma_part(ncb_tag, F1, 0, 0, NL / 3);
      mfma_part(ncb_tag, F1, 1, NL / 3, 2 * NL / 3);
      __builtin_amdgcn_sched_barrier(0);
      mfma_part(ncb_tag, F0, 0, 2 * NL / 3, NL);  // K step 0 of a chunk always lies inside [0, v)
      __builtin_amdgcn_sched_barrier(0);
      read_step(rbuf, 1, F1);
      __builtin_amdgcn_sched_barrier(0);
      mfma_part(ncb_tag, F0, 1, 0, 0);
      rbuf = rbuf == 2 ? 0 : rbuf + 1;
    }
    if (16 < v - (nkc - 1) * KC) {
      mfma_part(ncb_tag, F1, 0, 0, 0);
      mfma_part(ncb_tag, F1, 1, 0, 0);
    }
  };
  static_assert(CB >= 1 && CB <= 4, "column blocks per wave");

  load_tile();
#pragma unroll
  for (int k = 0; k < 2 * NL; ++k) issue1(k % NL);
  for (; tile < n_tiles; tile += gridDim.x) {
    const int c_base = (tile / n_rt) * TC + wc * CB * 32, r_base = (tile % n_rt) * TR + wr * RB * 32;
    int nvalid = r_base < M ? min(CB, max(0, (N - c_base + 31) / 32)) : 0;
    nvalid = __builtin_amdgcn_readfirstlane(nvalid);
#pragma unroll
    for (int a = 0; a < CB; ++a)
#pragma unroll
      for (int b = 0; b < RB; ++b) acc[a][b] = zero16();
    if (nvalid == CB) {
      main_loop(std::integral_constant<int, CB>{});
    } else if (nvalid == 0) {
      main_loop(std::integral_constant<int, 0>{});
    } else {
      if constexpr (CB >= 4) {
        if (nvalid == 3) main_loop(std::integral_constant<int, 3>{});
      }
      if constexpr (CB >= 3) {
        if (nvalid == 2) main_loop(std::integral_constant<int, 2>{});
      }
      if constexpr (CB >= 2) {
        if (nvalid == 1) main_loop(std::integral_constant<int, 1>{});
      }
    }

    // store W^T as hi/lo planes: register t of lane (32h + m) holds column c = m and row 8(t/4) + 4h + t%4
    // of a block, which goes through this wave's own LDS block (swizzled) so that a column's 32 rows
    // leave as 16 bytes per lane
    const bool full = c_base + CB * 32 <= N && r_base + RB * 32 <= M;
    __bf16 *stage = ldsa + 3 * ROWS * KC + wave * 1024;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          __bf16 *W = p ? Wl : Wh;
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            bf4 x;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const float w = acc[cb][rb][4 * g + t];
              const __bf16 hi = (__bf16)w;
              x[t] = p ? (__bf16)(w - (float)hi) : hi;
            }
            *reinterpret_cast<bf4 *>(&stage[m * 32 + 8 * (g ^ ((m >> 2) & 3)) + 4 * h]) = x;
          }
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int c = 16 * i + lrow, g = lane & 3;
            const bf8 x = *reinterpret_cast<const bf8 *>(&stage[c * 32 + 8 * (g ^ ((c >> 2) & 3))]);
            const int cc = c_base + cb * 32 + c, rr = r_base + rb * 32 + 8 * g;
            __bf16 *dst = W + (size_t)cc * M + rr;
            if (full || (cc < N && rr < M)) *reinterpret_cast<bf8 *>(dst) = x;
          }
        }
    stored = full;
    if (!full) wait_vm<0>();  // (an unknown number of stores)
  }
  wait_vm<0>();  // no LDS write may still be in flight when the workgroup ends
}

// ---------------------------------------------------------------------------------------------
// (B) P[ks][s][i][c] (+)= scale * sum_{qq in split ks} sum_j B_oo^(q0+qq)[i][j] W^T[qq][c][s*op + j]
// over the flattened columns n = (s, c).
// Waves: NWM along i x NWN along n; each wave MB x NB blocks.  Reduction chunks run over (qq, j).
// ---------------------------------------------------------------------------------------------
template <int NWM, int NWN, int MB, int NB>
struct CfgB {
  static constexpr int NW = NWM * NWN, NT = 64 * NW;
  static constexpr int TM = NWM * MB * 32, TN = NWN * NB * 32;
  static constexpr int ROWS = TM + 2 * TN;     // tile rows per buffer: B_oo, W hi, W lo
  static constexpr int NL = ROWS / (16 * NW);  // 16-row load instructions per wave and chunk
  static constexpr size_t LDS = (size_t)3 * ROWS * KC * 2;
  static_assert(ROWS % (16 * NW) == 0, "tile rows split into whole load instructions");
  static_assert(LDS <= 160 * 1024, "LDS");
};

template <int NWM, int NWN, int MB, int NB>
__global__ __launch_bounds__(64 * NWM * NWN, 1) void k_boo_w(const __bf16 *__restrict__ Boo,
                                                             const __bf16 *__restrict__ Wh,
                                                             const __bf16 *__restrict__ Wl, int o, int op, int v,
                                                             int ns, int nqc, int nsplit, int n_ct, int accumulate,
                                                             float scale, float *__restrict__ P) {
  using C = CfgB<NWM, NWN, MB, NB>;
  constexpr int NL = C::NL, TM = C::TM, TN = C::TN, ROWS = C::ROWS;
  extern __shared__ __attribute__((aligned(16))) __bf16 ldsb[];  // [3][B_oo TM | W hi TN | W lo TN][32]

  const int lb = xcd_local_id();
  if (lb >= n_ct * nsplit) return;
  const int ct = lb % n_ct, ks = lb / n_ct;
  const int qa = (int)((long long)ks * nqc / nsplit), qb = (int)((long long)(ks + 1) * nqc / nsplit);
  const int c_base = ct * TN, M = ns * op, N = ns * v;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, m = lane & 31, lrow = lane >> 2;
  const int wm = wave / NWN, wn = wave % NWN;
  const int nkj = (op + KC - 1) / KC;
  const int NC = (qb - qa) * nkj;
  int nvalid = 0;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) nvalid += (c_base + (wn * NB + nb) * 32 < N) ? 1 : 0;
  if (wm * MB * 32 >= o) nvalid = 0;
  // (nvalid is wave-uniform)
  // the zero page's address stays in registers for the whole kernel (re-deriving it inside the
  // loop puts a scalar memory load among the LDS reads, which forces full LDS waits)
  const void *zp = g_zero_page_g;
  asm volatile("" : "+s"(zp));

  // A load takes 16 tile rows, each lane its 16-byte group, swizzled within the row; the bases of the
  // chunk to load are kept in scalar registers.  Rows past op or N read the first one (their sums are not
  // stored); j past op, and chunks past the end, load the zero page.
  const int j_lane = 8 * ((lane & 3) ^ swz(lrow));
  unsigned vo[NL];  // bytes from the base
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int u = (wave * NL + k) * 16, r = u + lrow;
    const int n = c_base + (u < TM + TN ? r - TM : r - TM - TN);
    const unsigned ao = (unsigned)(r < op ? r : 0) * op;
    const unsigned wo = n < N ? (unsigned)(n % v) * M + (unsigned)(n / v) * op : 0u;
    vo[k] = 2 * ((u < TM ? ao : wo) + j_lane);
  }
  const char *po = reinterpret_cast<const char *>(Boo + (size_t)qa * op * op);
  const char *ph = reinterpret_cast<const char *>(Wh + (size_t)qa * v * M);
  const size_t dl = reinterpret_cast<const char *>(Wl) - reinterpret_cast<const char *>(Wh);
  int ji = 0, left = NC, lbuf = 0;  // first j of the chunk to load, chunks left, buffer
  auto issue1 = [&](int k) {        // loads 0..NL-1 of a chunk, in order
    const int u = (wave * NL + k) * 16, j_lim = left > 0 ? op - ji : 0;
    const char *src = (u < TM ? po + 0 : ph + 0) + (u < TM + TN ? 0 : dl) + vo[k];
    dma16(j_lane < j_lim ? (const void *)src : zp, ldsb + lbuf * (ROWS * KC) + u * KC);
    if (k == NL - 1) {
      lbuf = lbuf == 2 ? 0 : lbuf + 1;
      --left;
      const bool wrap = ji + KC >= op;  // on to the next Q
      po += wrap ? ((size_t)op * op - ji) * 2 : (size_t)KC * 2;
      ph += wrap ? ((size_t)v * M - ji) * 2 : (size_t)KC * 2;
      ji = wrap ? 0 : ji + KC;
    }
  };

  f16v acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = zero16();

  // Same pipeline as the first kernel (see there): K step 0's fragments are read right after the
  // barrier while K step 1 of the previous chunk runs; K step 1's are read during the W_lo half of
  // K step 0.  Steps past o read zero rows of the B_oo tile and add nothing.
  struct Frag {
    bf8 a[MB], wh[NB], wl[NB];
  };
  auto read_step = [&](int c, int u, Frag &F) {
    const __bf16 *As = ldsb + (c % 3) * (ROWS * KC);
    const __bf16 *Whs = As + TM * KC;
    const __bf16 *Wls = Whs + TN * KC;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int r = (wm * MB + mb) * 32 + m;
      F.a[mb] = *reinterpret_cast<const bf8 *>(&As[r * KC + 8 * ((2 * u + h) ^ swz(r))]);
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int r = (wn * NB + nb) * 32 + m;
      const int co = r * KC + 8 * ((2 * u + h) ^ swz(r));
      F.wh[nb] = *reinterpret_cast<const bf8 *>(&Whs[co]);
      F.wl[nb] = *reinterpret_cast<const bf8 *>(&Wls[co]);
    }
  };
  auto mfma_part = [&](auto nnb_tag, const Frag &F, int part, int k0, int k1) {
    constexpr int NNB = decltype(nnb_tag)::value;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
      for (int nb = 0; nb < NNB; ++nb)
        acc[mb][nb] =
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(F.a[mb], part ? F.wl[nb] : F.wh[nb], acc[mb][nb], 0, 0, 0);
      if (k0 < k1) {
        __builtin_amdgcn_sched_barrier(0);
        const int ka = k0 + (k1 - k0) * mb / MB, kb = k0 + (k1 - k0) * (mb + 1) / MB;
#pragma unroll
        for (int k = ka; k < kb; ++k) issue1(k);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  auto main_loop = [&](auto nnb_tag) {
    Frag F0, F1;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) F1.a[mb] = bf8{};
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) F1.wh[nb] = F1.wl[nb] = bf8{};
#pragma unroll
    for (int k = 0; k < 2 * NL; ++k) issue1(k % NL);
    for (int c = 0; c < NC; ++c) {
      wait_vm<NL>();  // chunk c has landed (chunk c+1 may be in flight)
      lds_barrier();
      __builtin_amdgcn_sched_barrier(0);
      read_step(c, 0, F0);
      __builtin_amdgcn_sched_barrier(0);
      // K step 1 of chunk c-1 (zero fragments before chunk 0), with the loads of chunk c+2 into its buffer
      mfma_part(nnb_tag, F1, 0, 0, NL / 3);
      mfma_part(nnb_tag, F1, 1, NL / 3, 2 * NL / 3);
      __builtin_amdgcn_sched_barrier(0);
      mfma_part(nnb_tag, F0, 0, 2 * NL / 3, NL);
      __builtin_amdgcn_sched_barrier(0);
      read_step(c, 1, F1);
      __builtin_amdgcn_sched_barrier(0);
      mfma_part(nnb_tag, F0, 1, 0, 0);
    }
    mfma_part(nnb_tag, F1, 0, 0, 0);
    mfma_part(nnb_tag, F1, 1, 0, 0);
    wait_vm<0>();  // no LDS write may still be in flight when the workgroup ends
  };
  static_assert(NB >= 1 && NB <= 4, "column blocks per wave");
  if (nvalid == NB) {
    main_loop(std::integral_constant<int, NB>{});
  } else if (nvalid == 0) {
    main_loop(std::integral_constant<int, 0>{});
  } else {
    if constexpr (NB >= 4) {
      if (nvalid == 3) main_loop(std::integral_constant<int, 3>{});
    }
    if constexpr (NB >= 3) {
      if (nvalid == 2) main_loop(std::integral_constant<int, 2>{});
    }
    if constexpr (NB >= 2) {
      if (nvalid == 1) main_loop(std::integral_constant<int, 1>{});
    }
  }

  // a split with no Q in this chunk still stores its (zero) slab on the first chunk
  // (the old values of a block are read together, from clamped places, not one after the other)
  float *Pp = P + (size_t)ks * ns * o * v;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int n = c_base + (wn * NB + nb) * 32 + m, nn = min(n, N - 1);
    float *Pn = Pp + (size_t)(nn / v) * o * v + nn % v;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      float old[16];
      const int i0 = (wm * MB + mb) * 32 + 4 * h;
#pragma unroll
      for (int t = 0; t < 16; ++t) old[t] = 0.f;
      if (accumulate) {
#pragma unroll
        for (int t = 0; t < 16; ++t) old[t] = Pn[(size_t)min(i0 + 8 * (t / 4) + t % 4, o - 1) * v];
      }
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int i = i0 + 8 * (t / 4) + t % 4;
        const float val = scale * acc[mb][nb][t];
        if (i < o && n < N) Pn[(size_t)i * v] = accumulate ? old[t] + val : val;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Host side: the chunk loop.  W hi/lo for `qc` values of Q take qc * v * M * 4 bytes of scratch.
// ---------------------------------------------------------------------------------------------
template <int NWC, int NWR, int CB, int RB, int NWM, int NWN, int MB, int NB>
hipError_t launch_xgemm(hipStream_t s, const void *Boo, const void *Bvv, const void *X, const void *Xlo, int o,
                        int v, int nq, int ns, int nsplit, float scale, float *P, void *scratch,
                        size_t scratch_bytes) {
  using CA = CfgA<NWC, NWR, CB, RB>;
  using CBf = CfgB<NWM, NWN, MB, NB>;
  const int op = (o + 7) / 8 * 8;
  if (op > CBf::TM || (v & 7) != 0 || nq <= 0 || scratch == nullptr || scratch_bytes % 16 != 0)
    return hipErrorInvalidValue;
  const int M = ns * op, nkc = (v + KC - 1) / KC, n_rt = (M + CA::TR - 1) / CA::TR;
  const size_t per_q = (size_t)v * M * 2 * sizeof(__bf16);
  const size_t xt = (size_t)nkc * KC * n_rt * CA::TR * 2;  // X in staging order, values
  if (xt * sizeof(__bf16) > xgemm_x_bytes(v, M)) return hipErrorInvalidValue;
  const int qc = (int)std::min<size_t>((size_t)nq, scratch_bytes / per_q);
  if (qc < 1) return hipErrorInvalidValue;
  __bf16 *Wh = static_cast<__bf16 *>(scratch);
  __bf16 *Wl = Wh + (size_t)qc * v * M;
  __bf16 *Xt = Wh + scratch_bytes / sizeof(__bf16), *Ot = Xt + xgemm_x_bytes(v, M) / sizeof(__bf16);
  const int n_ctb = (ns * v + CBf::TN - 1) / CBf::TN;
  const __bf16 *vv = static_cast<const __bf16 *>(Bvv), *oo = static_cast<const __bf16 *>(Boo);
  hipLaunchKernelGGL(k_xgemm_x, dim3((unsigned)std::min<size_t>(2048, (xt / 8 + 255) / 256)), dim3(256), 0, s,
                     static_cast<const __bf16 *>(X), static_cast<const __bf16 *>(Xlo), o, op, v, M, CA::TR, n_rt, nkc, Xt);
  for (int q0 = 0; q0 < nq; q0 += qc) {
    const int nqc = std::min(qc, nq - q0);
    const int n_ct = (nqc * v + CA::TC - 1) / CA::TC;
    hipLaunchKernelGGL((k_xgemm_w<NWC, NWR, CB, RB>), dim3(std::min(256, (n_ct * n_rt + 7) / 8 * 8)), dim3(CA::NT),
                       CA::LDS, s, vv + (size_t)q0 * v * v, Xt, v, M, nqc * v, n_ct, n_rt, Wh, Wl);
    if (op != o)
      hipLaunchKernelGGL(k_xgemm_o, dim3((unsigned)std::min<size_t>(4096, ((size_t)nqc * op * (op / 8) + 255) / 256)),
                         dim3(256), 0, s, oo + (size_t)q0 * o * o, o, op, nqc, Ot);
    hipLaunchKernelGGL((k_boo_w<NWM, NWN, MB, NB>), dim3((n_ctb * nsplit + 7) / 8 * 8), dim3(CBf::NT), CBf::LDS, s,
                       op == o ? oo + (size_t)q0 * o * o : Ot, Wh, Wl, o, op, v, ns, nqc, nsplit, n_ctb, q0 > 0 ? 1 : 0, scale, P);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int NWC, int NWR, int CB, int RB, int NWM, int NWN, int MB, int NB>
hipError_t prepare_xgemm() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_xgemm_w<NWC, NWR, CB, RB>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)CfgA<NWC, NWR, CB, RB>::LDS);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void *>(&k_boo_w<NWM, NWN, MB, NB>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)CfgB<NWM, NWN, MB, NB>::LDS);
}

#define XGM(NWC, NWR, CB, RB, NWM, NWN, MB, NB, NAME)                                                   \
  ExchangeVariant {                                                                                          \
    RTTDA_PREC_MIXED_BF16, CfgB<NWM, NWN, MB, NB>::TM, 1, CfgA<NWC, NWR, CB, RB>::TC, NAME,                  \
        &launch_xgemm<NWC, NWR, CB, RB, NWM, NWN, MB, NB>,                                              \
        std::max(CfgA<NWC, NWR, CB, RB>::LDS, CfgB<NWM, NWN, MB, NB>::LDS),                                  \
        &prepare_xgemm<NWC, NWR, CB, RB, NWM, NWN, MB, NB>, 8, 8, 1, XGEMM_O_MIN, true, 0, 1 << 30, nullptr,   \
        nullptr, CfgA<NWC, NWR, CB, RB>::TR, CfgB<NWM, NWN, MB, NB>::TN                                               \
  }

const ExchangeVariant kGemmVariants[] = {
    XGM(2, 4, 4, 2, 2, 4, 2, 2, "bf16x2gemm_a256x256w8_b128x256w8"),
    XGM(4, 2, 2, 3, 2, 4, 2, 2, "bf16x2gemm_a256x192w8_b128x256w8"),
    XGM(2, 4, 4, 2, 4, 2, 2, 2, "bf16x2gemm_a256x256w8_b256x128w8"),
    XGM(4, 2, 2, 3, 4, 2, 2, 2, "bf16x2gemm_a256x192w8_b256x128w8"),
};

}  // namespace

int exchange_gemm_variant_count() { return (int)(sizeof(kGemmVariants) / sizeof(kGemmVariants[0])); }
const ExchangeVariant *exchange_gemm_variant(int k) { return &kGemmVariants[k]; }

}  // namespace rttda
