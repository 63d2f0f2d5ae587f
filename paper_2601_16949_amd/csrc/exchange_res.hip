// Exchange contraction with X resident in LDS (both precisions):
//   P[split][s][i][c] = scale * sum_{Q in split} (B_oo^Q X_s B_vv^Q)[i][c]
//
// Same two products per Q as the other exchange kernels (W = X_s B_vv^Q in matrix-core accumulators,
// then K += B_oo^Q W with the accumulators as the second operand), for shapes where the padded X of
// one or a few slices fits the LDS of a CU.  X is then staged once per workgroup, already in operand
// order, and only the factors move: every wave owns 16-column blocks of the output and a range of
// Q and reads its own rows of the symmetric B_vv^Q straight into registers, `D` K steps ahead.  No
// barrier and no LDS write separates the staging from the last Q, so the waves of a SIMD drift apart
// and one's matrix work covers the other's waits; the kernels that stage both operands through LDS
// stop all waves at every K chunk for that.
//
// Operands travel as 16-byte groups (eight BF16 or four FP32 values).  A K step is four groups: lane
// (g, n) = (lane / 16, lane % 16) holds one group of row n, which for BF16 is one
// v_mfma_f32_16x16x32_bf16 and for FP32 four v_mfma_f32_16x16x4_f32.  Which group of the row a lane
// group g takes is free (X is laid out to match): two K steps (a double step, eight groups, 128 bytes
// of a row) are loaded as pairs of rows, lanes 2a and 2a + 1 taking 32 contiguous bytes of row 2a in
// one load and of row 2a + 1 in the other, and the lanes of a pair exchange halves.  (A load with 16
// bytes per row and lane costs the L1 a lookup per lane: with it the lookups, one a cycle, set the
// time.)  The last group of a row is the row's last eight (four) values; X's copy of it holds zeros
// where the group before it has those values already, and zeros in the groups past it.  So any v works,
// nothing is read outside a row, and no lane is masked (global memory takes rows of any alignment).
// The K product does the same with rows: the accumulators of lane (g, n) are the W rows it must supply,
// and X's rows are laid out so that they are consecutive j (eight per pair of 16-row blocks in BF16,
// four per block in FP32); the last group of j is o's last eight (four) rows with the repeated ones
// zero.  B_oo^Q fragments are then one load per lane too.
//
// What bounds it: in FP32 the matrix cores (busy about 89 % of the time at o60 v400 N_Q1500, 3 RHS: 1660
// us per launch, where the best LDS-staged tile takes 1870).  In split BF16, whose products are eight
// times shorter, the L1's lookups of B_vv and B_oo rows and the waits of two waves per SIMD (matrix
// cores busy about 48 %: 386 us against 536-600); the 64-row and the two-slice 32-row tiles also spill
// (51 and 27 registers, 80 and 48 bytes a lane: K accumulators that are read and written once per Q, in
// order behind the ring's loads).  The Q ranges of a workgroup are long (42 slabs there
// against 220-357), which the stage epilogue feels: 18 us for 38-51.
// Odd sizes run like even ones: o37 v277 N_Q743, 2 RHS, split BF16: 86 us (320 for the register-staged
// tile); o27 v203 N_Q541, 3 RHS, FP32: 124 us (192).
//
// Split BF16 as in exchange_bf16.hip: X = X_hi + X_lo (two planes), W likewise, FP32 accumulators.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace rttda {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef short s4v __attribute__((ext_vector_type(4)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef u4 u4_unaligned __attribute__((aligned(2)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef u2 u2_unaligned __attribute__((aligned(2)));

constexpr int NWAVE = 8;                      // waves per workgroup, two per SIMD
constexpr size_t LDS_MAX = (size_t)160 << 10;  // a CU's LDS

// BF: split BF16 (else FP32); JB 16-row blocks per slice, KS slices per workgroup, at most NCBM column
// blocks per wave
// PK (FP32): two slices of at most 16 JB - 8 rows share 2 JB - 1 row blocks, the first eight rows of each in
// the halves of the middle one, its other rows in the blocks on its side (so that a slice's sums run in one
// order wherever it stands).  Where the matrix cores set the time, that is the work of o up to 24 or 40 rows
// without a half-empty block per slice: o40 v300 N_Q1000, 64 RHS 10.4 -> 8.6 ms per launch (the best paired
// LDS-staged tile: 9.3), o24 v168 N_Q600, 32 RHS 732 -> 610 us, o36 v252 N_Q900, 3 RHS 333 -> 308 us.
template <bool BF, int JB, int KS, int NCBM, bool PK = false>
struct CfgR {
  static_assert(!PK || (!BF && KS == 2), "packed pairs: FP32, two slices");
  static constexpr int RB = PK ? 2 * JB - 1 : JB * KS;  // row blocks of X and W
  static constexpr int KB = JB * KS;                     // row blocks of K
  static constexpr int OMAX = PK ? 16 * JB - 8 : 16 * JB;
  static constexpr int PL = BF ? 2 : 1;           // planes of X
  static constexpr int GV = BF ? 8 : 4;           // values per 16-byte group
  static constexpr int SZ = BF ? 2 : 4;           // bytes per factor value
  static constexpr int STEP_LDS = RB * PL * 1024;  // bytes of X per K step
  static constexpr int VMAX = (int)(LDS_MAX / STEP_LDS) * 4 * GV;
};

// How a workgroup's waves share the columns and its Q range.  Its column tile's blocks go to ncg groups
// of waves, the first `wide` of them one block wider, and each group's Q range to qs waves.  rem: the
// last rem blocks of the tile are left to a second phase, in which all eight waves take an eighth of
// the Q range each.
struct Split {
  int nct, ncg, qs, rem;
};

// first block and width of column group cg in a tile of nb blocks (rem of them left out)
__host__ __device__ inline void group_blocks(int nb, int rem, int ncg, int cg, int &b0, int &w) {
  const int base = (nb - rem) / ncg, wide = (nb - rem) % ncg;
  b0 = cg * base + (cg < wide ? cg : wide);
  w = base + (cg < wide ? 1 : 0);
}
__host__ __device__ inline int tile_block(int nblk, int nct, int ct) { return (int)((long long)ct * nblk / nct); }

// The split with the least matrix work per Q on the fullest SIMD (waves w and w + 4 share one).  A
// wave's X reads are spread over its width, so narrow groups cost more than their matrix work: a
// single block per wave is bound by the LDS at about twice its matrix time, two at about 1.1 times.
// Depends on v alone, so that a batch and a single right-hand side sum alike.
inline Split choose_split(int v, int ncbm) {
  const int nblk = (v + 15) / 16;
  auto cost = [](int w) { return w == 1 ? 2.0 : w == 2 ? 2.2 : (double)w; };
  Split s{0, 0, 0, 0};
  double best = 1e300;
  for (int nct = 1; nct <= nblk; ++nct) {
    const int nb = nblk - tile_block(nblk, nct, nct - 1);  // the last tile is the widest
    for (int ncg = 1; ncg <= NWAVE; ++ncg) {
      const int qs = NWAVE / ncg;
      for (int rem = 0; rem <= (qs == 1 ? std::min(ncbm, nb - 1) : 0); ++rem) {
        if ((nb - rem + ncg - 1) / ncg > ncbm) continue;
        double load[4] = {0, 0, 0, 0};
        for (int w = 0; w < ncg * qs; ++w) {
          int b0, width;
          group_blocks(nb, rem, ncg, w % ncg, b0, width);
          load[w % 4] += width ? cost(width) : 0.0;
        }
        const double c = nct * (std::max(std::max(load[0], load[1]), std::max(load[2], load[3])) / qs +
                                (rem ? 2.0 * cost(rem) / NWAVE + 0.05 : 0.0));
        if (c < best - 1e-12) {
          best = c;
          s = Split{nct, ncg, qs, rem};
        }
      }
    }
    if (s.nct > 0 && nct > s.nct) break;  // more tiles than the first count that fits only if they cost less
  }
  return s;
}

// source row of X row slot rs (0 .. 16 JB - 1), or -1 for a row of zeros
template <bool BF, int JB>
__device__ __forceinline__ int slot_row(int rs, int o) {
  const int blk = rs >> 4, gg = (rs >> 2) & 3, t = rs & 3;
  const bool pair = BF && (blk | 1) < JB;
  const int w = pair ? 8 : 4;
  const int j0 = pair ? 32 * (blk >> 1) + 8 * gg : 16 * blk + 4 * gg, e = pair ? t + 4 * (blk & 1) : t;
  if (j0 + w <= o) return j0 + e;
  const int j = o - w + e;
  return j0 < o && j >= j0 ? j : -1;
}

// RANGES: 0, a workgroup per split of Q.  Else each split is cut into m ranges of Q, whose sums are added in FP32,
// in order: 2 (RNG), a workgroup takes a split and adds them in its slab (FP32) or leaves each (split BF16); 1
// (EACH), one takes a range and leaves its sum.  The stage update adds what is left, with the same bits.  So a
// context whose full batch fills the CUs with long splits (few slabs, X staged once) has short ranges for a call
// with few of its right-hand sides, which would else run on a few CUs, and the FP32 chains stay short in both.
// o40 v300 N_Q1000 FP32, max_rhs 64, 4 splits of 32 ranges, per step: one RHS 1.5 ms (34.9 without ranges), all
// 64 35.6 (35.3).  o60 v400 N_Q1500, max_rhs 3, per two steps: one RHS 5.7 ms (13.9) in FP32, 42 splits of 3, and
// 2.3 (3.7) in split BF16, 42 of 2; all three 13.98 (13.92) and 3.69 (3.59).
// (The second phase's blocks, whose waves share the split's Q in eighths, are left out of that: the workgroup of
// a split's first range takes them, the others' slabs hold zeros there.)
template <bool BF, int JB, int KS, int NCBM, bool PK, int RANGES>
__global__ __launch_bounds__(64 * NWAVE, 1) void k_exchange_res(const char *__restrict__ Boo,
                                                                const char *__restrict__ Bvv,
                                                                const char *__restrict__ X,
                                                                const char *__restrict__ Xlo, int o, int v, int nq,
                                                                int ns, int n_sg, int nct, int ncg, int qs, int rem,
                                                                int nsplit, int m, float scale,
                                                                float *__restrict__ P) {
  using C = CfgR<BF, JB, KS, NCBM, PK>;
  constexpr int RB = C::RB, KB = C::KB, PL = C::PL, GV = C::GV, SZ = C::SZ;
  constexpr int D = 2;                       // double steps of B_vv in flight (of every other one, see the loop below)
  constexpr int HA = (RB + 1) / 2;           // row blocks of the first half of a step
  // K-product steps: pairs of row blocks (the last may be a single one); packed: each slice's JB
  constexpr int NP = BF ? (JB + 1) / 2 : PK ? 2 * JB : JB;
  extern __shared__ __attribute__((aligned(16))) char ldsr[];

  // XCD-aware logical block id (hardware deals workgroups to the 8 XCDs round robin): slice groups
  // fastest, so that the workgroups that read the same rows of B_vv^Q run together on one XCD
  const int total = n_sg * nct * nsplit;
  const int per_xcd = (int)gridDim.x / 8;
  const int lb = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if (lb >= total) return;
  const int sg = lb % n_sg, ct = (lb / n_sg) % nct, sp = lb / (n_sg * nct);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, n = lane & 15;
  const int s_base = sg * KS;
  const int ng = (v + GV - 1) / GV, nds = (ng + 7) / 8;  // groups per row, double steps
  const bool odd_k = ng - 8 * (nds - 1) <= 4;             // the last double step is a single one
  const int nst = 2 * nds - (odd_k ? 1 : 0);              // K steps

  // ---- X of this workgroup's slices into LDS, in operand order (1 KiB per K step, row block, plane)
  {
    const int nfrag = nst * RB;
    const int row = lane >> 2, gl = lane & 3;  // four groups of 16 rows: 64 contiguous bytes per row
    for (int f = wave; f < nfrag; f += NWAVE) {
      const int st = f / RB, rb = f - st * RB;
      int sl = s_base + rb / JB, j = slot_row<BF, JB>((rb % JB) * 16 + row, o);
      if constexpr (PK) {
        const int up = rb > JB - 1 || (rb == JB - 1 && row >= 8) ? 1 : 0;  // second slice
        sl = s_base + up;
        j = slot_row<BF, JB>(rb == JB - 1 ? row & 7 : 8 + 16 * (up ? rb - JB : rb) + row, o);
      }
      const int grp = odd_k && st == nst - 1 ? 4 * st + gl : 8 * (st >> 1) + 2 * gl + (st & 1);
      const bool live = sl < ns && j >= 0 && grp < ng;
      const int a0 = grp == ng - 1 ? v - GV : GV * grp;  // first value of the group's load
      const int dup = GV * grp - a0;                     // its leading values the previous group has
      const size_t off = ((size_t)(live ? sl : 0) * o + (live ? j : 0)) * v + (live ? a0 : 0);
#pragma unroll
      for (int p = 0; p < PL; ++p) {
        u4 x = *reinterpret_cast<const u4_unaligned *>((p ? Xlo : X) + off * SZ);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (BF) {
            const unsigned lo = live && 2 * e >= dup ? x[e] & 0xffffu : 0u;
            const unsigned hi = live && 2 * e + 1 >= dup ? x[e] & 0xffff0000u : 0u;
            x[e] = lo | hi;
          } else {
            x[e] = live && e >= dup ? x[e] : 0u;
          }
        }
        *reinterpret_cast<u4 *>(ldsr + ((size_t)f * PL + p) * 1024 + (gl * 16 + row) * 16) = x;
      }
    }
  }
  __syncthreads();

  const int nblk = (v + 15) / 16;
  const int t0 = tile_block(nblk, nct, ct), t1 = tile_block(nblk, nct, ct + 1);
  // ADD: in the slab, which all workgroups read and write at once (o60 v400, 3 RHS: 4 us a range in FP32, whose
  // ranges are long; 13 us in split BF16, where leaving them costs the launch 2 us and the stage update 5)
  constexpr bool EACH = RANGES == 1, RNG = RANGES == 2, ADD = !BF;
  const int n_split = EACH ? nsplit / m : nsplit, split = EACH ? sp / m : sp, range = EACH ? sp - split * m : 0;
  const int Qa = (int)((long long)split * nq / n_split), Qb = (int)((long long)(split + 1) * nq / n_split);
  auto bound = [&](int k) { return Qa + k * (Qb - Qa) / m; };  // the split's ranges

  // byte offset of this lane's load in the last double step of a row: the row's last group ends at v
  const int odd = n & 1;
  const int glast = 8 * (nds - 1) + (odd_k ? (odd ? 8 : g) : 2 * g + odd);
  const unsigned klast = glast < ng - 1 ? 16u * glast : glast == ng - 1 ? (unsigned)(v - GV) * SZ : 0u;

  // blocks [b0, b0 + NCB) over Q in [qa, qb): part `part` of nparts, whose waves are grp, grp + pstride, ...
  auto run = [&](auto ncb_tag, int b0, int qa, int qb, int part, int nparts, int grp, int pstride)
                 __attribute__((always_inline)) {
    constexpr int NCB = decltype(ncb_tag)::value;
    f4 K[KB][NCB], W[RB][NCB];
#pragma unroll
    for (int a = 0; a < KB; ++a)
#pragma unroll
      for (int c = 0; c < NCB; ++c) K[a][c] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
      for (int c = 0; c < NCB; ++c) W[a][c] = f4{0.f, 0.f, 0.f, 0.f};
    // byte offset of the first of the two rows (columns of the output) this lane loads; the second is
    // the row after it, or the last one
    unsigned roff[NCB];
    const unsigned row_bytes = (unsigned)(v * SZ), row_last = (unsigned)(v - 1) * row_bytes;
#pragma unroll
    for (int c = 0; c < NCB; ++c) roff[c] = (unsigned)min((b0 + c) * 16 + (n & ~1), v - 1) * row_bytes;
    // RNG: K, the sum of the split's range rg, to its slab, or added to what the split's holds
    auto flush = [&](int rg) __attribute__((always_inline)) {
      const bool add = ADD && rg > 0;
      const int to = ADD ? sp : sp * m + rg;
      int ln = lane;  // (opaque here: addresses made from it would be held in registers through the loop)
      asm volatile("" : "+v"(ln));
      unsigned col[NCB];  // byte offsets, from clamped places
#pragma unroll
      for (int c = 0; c < NCB; ++c) col[c] = 4u * min((b0 + c) * 16 + (ln & 15), v - 1);
      auto slab = [&](int a) __attribute__((always_inline)) {
        return reinterpret_cast<char *>(P + ((size_t)to * ns + min(s_base + a / JB, ns - 1)) * o * v);
      };
      auto row = [&](int a, int t) __attribute__((always_inline)) {
        return 4u * (unsigned)v * min((a % JB) * 16 + 4 * (ln >> 4) + t, o - 1);
      };
      f4 old[KB][NCB] = {};
      if (add) {  // (all of them on their way before the first is used)
#pragma unroll
        for (int a = 0; a < KB; ++a)
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int c = 0; c < NCB; ++c)
              old[a][c][t] = *reinterpret_cast<const float *>(slab(a) + (row(a, t) + col[c]));
      }
#pragma unroll
      for (int a = 0; a < KB; ++a)
#pragma unroll
        for (int c = 0; c < NCB; ++c) {
#pragma clang fp contract(off)  // (the stage update, which adds the ranges elsewhere, rounds each of them)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const float x = scale * K[a][c][t];
            if (s_base + a / JB < ns && (a % JB) * 16 + 4 * (ln >> 4) + t < o && (b0 + c) * 16 + (ln & 15) < v)
              *reinterpret_cast<float *>(slab(a) + (row(a, t) + col[c])) = add ? old[a][c][t] + x : x;
          }
        }
    };
    int rg = 0, qf = RNG && nparts == 1 ? bound(1) : qb;  // RNG: ranges done, and the next one's end
    auto next_range = [&]() __attribute__((always_inline)) {
      flush(rg);
#pragma unroll
      for (int a = 0; a < KB; ++a)
#pragma unroll
        for (int c = 0; c < NCB; ++c) K[a][c] = f4{0.f, 0.f, 0.f, 0.f};
      ++rg;
      qf = bound(rg + 1);
    };
    // split BF16 leaves the loop over its Q for a range's end: with that inside, the compiler spilled addresses of
    // the widest waves' loads and waited for every load to read them back (per two steps, 3 RHS of o48 v480 N_Q1500,
    // three blocks a wave, 4.32 ms, now 4.21, without ranges 4.19; 6 of o64 v440 N_Q1461, four, 13.6, 8.5 and 7.8,
    // see shape_xres).  FP32 spills more with that outside.
    constexpr bool NEST = RNG && BF;
    if (qa < qb) {
      const size_t qstride = (size_t)v * v * SZ;
      const char *ql = Bvv + (size_t)qa * qstride;  // Q and double step of the next load
      int lq = qa, lds_ = 0;
      u4 ring[D][2][NCB];
      auto load = [&](u4(&B)[2][NCB]) __attribute__((always_inline)) {
        const unsigned ko = lds_ == nds - 1 ? klast : 128u * lds_ + 32u * g + 16u * odd;
#pragma unroll
        for (int c = 0; c < NCB; ++c)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            B[u][c] = *reinterpret_cast<const u4_unaligned *>(
                ql + (size_t)((u ? min(roff[c] + row_bytes, row_last) : roff[c]) + ko));
        if (++lds_ == nds) {  // (past the last Q: its rows once more)
          lds_ = 0;
          if (++lq < qb) ql += qstride;
        }
      };
      // the pair's exchange: the even lane keeps its half of row 2a and takes the odd lane's, and the
      // other way round for row 2a + 1; then B[u] holds each lane's own row, step u
      auto exchange = [&](u4 &B0, u4 &B1) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const unsigned send = odd ? B0[e] : B1[e];
          const unsigned got = __builtin_amdgcn_update_dpp(0u, send, 0xB1, 0xF, 0xF, true);  // lane ^ 1
          B0[e] = odd ? got : B0[e];
          B1[e] = odd ? B1[e] : got;
        }
      };
      u4 xa[HA][PL], xb[HA][PL];
      auto read_x = [&](u4(&F)[HA][PL], int st, int r0, int r1) __attribute__((always_inline)) {
        const char *b = ldsr + (size_t)st * C::STEP_LDS + lane * 16;
#pragma unroll
        for (int r = 0; r < HA; ++r)
          if (r0 + r < r1)
#pragma unroll
            for (int p = 0; p < PL; ++p)
              F[r][p] = *reinterpret_cast<const u4 *>(b + ((r0 + r) * PL + p) * 1024);
      };
      auto mfma_w = [&](const u4(&F)[HA][PL], const u4 &B, int c, int r0, int r1) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < (BF ? PL : 4); ++p)
#pragma unroll
          for (int r = 0; r < HA; ++r)
            if (r0 + r < r1) {
              if constexpr (BF)
                W[r0 + r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf8, F[r][p]), __builtin_bit_cast(bf8, B), W[r0 + r][c], 0, 0, 0);
              else
                W[r0 + r][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                    __builtin_bit_cast(f4, F[r][0])[p], __builtin_bit_cast(f4, B)[p], W[r0 + r][c], 0, 0, 0);
            }
      };
      auto mfma_all = [&](const u4(&F)[HA][PL], const u4(&B)[NCB], int r0, int r1) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NCB; ++c) mfma_w(F, B[c], c, r0, r1);
      };
      // B_oo^Q fragments of K-product step p: row ib 16 + n, the j of this lane's accumulators
      auto load_o = [&](u4(&F)[JB], int q, int p) __attribute__((always_inline)) {
        const bool pair = BF && 2 * p + 1 < JB;
        const int w = pair ? 8 : 4;
        int ln = lane;  // (once per Q: offsets recomputed rather than held in registers)
        asm volatile("" : "+v"(ln));
        const int g = ln >> 4, n = ln & 15;
        // (packed: the middle block first, whose two halves are the slices' rows 0..7)
        const int j0 = PK ? (p % JB == 0 ? 4 * (g & 1) : 16 * (p % JB) - 8 + 4 * g)
                          : pair ? 32 * p + 8 * g : (BF ? 32 : 16) * p + 4 * g;
        const int j = j0 + w <= o ? j0 : j0 < o ? o - w : 0;
        const char *Oq = Boo + (size_t)q * o * o * SZ;
#pragma unroll
        for (int ib = 0; ib < JB; ++ib) {
          const char *src = Oq + (unsigned)((min(ib * 16 + n, o - 1) * o + j) * SZ);
          if (BF && !pair) {
            const u2 t = *reinterpret_cast<const u2_unaligned *>(src);
            F[ib] = u4{t[0], t[1], 0u, 0u};
          } else {
            F[ib] = *reinterpret_cast<const u4_unaligned *>(src);
          }
        }
      };
      // K += B_oo^Q W for K-product step p
      auto mfma_k = [&](const u4(&F)[JB], int p) __attribute__((always_inline)) {
        if constexpr (BF) {
          const bool pair = 2 * p + 1 < JB;
          u4 w[KS][NCB][2];
#pragma unroll
          for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int c = 0; c < NCB; ++c) {
              bf8 hi, lo;
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                if (e >= 4 && !pair) {
                  hi[e] = lo[e] = (__bf16)0.f;
                  continue;
                }
                const float x = W[s * JB + (pair ? 2 * p + (e >> 2) : 2 * p)][c][e & 3];
                hi[e] = (__bf16)x;
                lo[e] = (__bf16)(x - (float)hi[e]);
              }
              w[s][c][0] = __builtin_bit_cast(u4, hi);
              w[s][c][1] = __builtin_bit_cast(u4, lo);
            }
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int ib = 0; ib < JB; ++ib)
#pragma unroll
              for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int c = 0; c < NCB; ++c) {
                  f4 &k = K[s * JB + ib][c];
                  if (pair)
                    k = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, F[ib]),
                                                                __builtin_bit_cast(bf8, w[s][c][h]), k, 0, 0, 0);
                  else
                    k = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                        __builtin_bit_cast(s4v, u2{F[ib][0], F[ib][1]}),
                        __builtin_bit_cast(s4v, u2{w[s][c][h][0], w[s][c][h][1]}), k, 0, 0, 0);
                }
        } else if constexpr (PK) {
          const int s = p / JB, pp = p % JB, blk = pp == 0 ? JB - 1 : s * JB + pp - 1;
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int c = 0; c < NCB; ++c) {
              // (the other slice's half of the middle block is left out, whatever it holds)
              const float w = pp == 0 && (g >= 2) != (s == 1) ? 0.f : W[blk][c][t];
#pragma unroll
              for (int ib = 0; ib < JB; ++ib)
                K[s * JB + ib][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(f4, F[ib])[t], w,
                                                                         K[s * JB + ib][c], 0, 0, 0);
            }
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int ib = 0; ib < JB; ++ib)
#pragma unroll
              for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int c = 0; c < NCB; ++c)
                  K[s * JB + ib][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                      __builtin_bit_cast(f4, F[ib])[t], W[s * JB + p][c][t], K[s * JB + ib][c], 0, 0, 0);
        }
      };

#pragma unroll
      for (int d = 0; d < D; ++d) {
        load(ring[d]);
        __builtin_amdgcn_sched_barrier(0);  // (in ring order: the loop's waits count on it)
      }
      read_x(xa, 0, 0, HA);
      int q = qa, ds = 0;
      u4 of0[JB], of1[JB];
      // one double step: each half step's X is read behind the other half's products; the ring slot is
      // refilled D double steps ahead.  A Q's first B_oo^Q fragments are requested before its last
      // double step's products.
      auto step = [&](u4(&B)[2][NCB]) __attribute__((always_inline)) {
        const bool last = ds == nds - 1, two = !(last && odd_k);
        if (last) load_o(of0, q, 0);
        if constexpr (HA < RB) read_x(xb, 2 * ds, HA, RB);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < NCB; ++c) {
          exchange(B[0][c], B[1][c]);
          mfma_w(xa, B[0][c], c, 0, HA);
        }
        __builtin_amdgcn_sched_barrier(0);
        read_x(xa, two ? 2 * ds + 1 : 0, 0, HA);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (HA < RB) mfma_all(xb, B[0], HA, RB);
        if (two) {
          if constexpr (HA < RB) read_x(xb, 2 * ds + 1, HA, RB);
          __builtin_amdgcn_sched_barrier(0);
          mfma_all(xa, B[1], 0, HA);
          __builtin_amdgcn_sched_barrier(0);
          read_x(xa, last ? 0 : 2 * ds + 2, 0, HA);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (HA < RB) mfma_all(xb, B[1], HA, RB);
        }
        __builtin_amdgcn_sched_barrier(0);
        load(B);
        __builtin_amdgcn_sched_barrier(0);
        ++ds;
        if (last) {
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            if (p + 1 < NP) load_o(p & 1 ? of0 : of1, q, p + 1);
            mfma_k(p & 1 ? of1 : of0, p);
          }
          if constexpr (RNG && !NEST)
            if (q + 1 == qf && q + 1 < qb) next_range();
#pragma unroll
          for (int a = 0; a < RB; ++a)
#pragma unroll
            for (int c = 0; c < NCB; ++c) W[a][c] = f4{0.f, 0.f, 0.f, 0.f};
          ds = 0;
          ++q;
          // the two waves of a SIMD take turns at issue priority: the older one, favoured by default,
          // would finish a quarter earlier and leave the other alone
          if ((q ^ (wave >> 2)) & 1) __builtin_amdgcn_s_setprio(1); else __builtin_amdgcn_s_setprio(0);
        }
      };
      // (an exit after each slot.  The compiler makes the first one part of the loop's end, sees a path on which
      // slot 0 has just been loaded, and waits for every load in flight before slot 0's products, with slot
      // 1's two loads per block still in flight before its own: every second double step starts on an empty
      // ring)
      for (;;) {
        const int qe = NEST ? qf : qb;
        bool turn = false;  // slot 1 is the next one
        for (;;) {
          step(ring[0]);
          if (NEST) turn = q >= qe;
          if (q >= qe) break;
          step(ring[1]);
          if (q >= qe) break;
        }
        if (!NEST || q >= qb) break;
        next_range();
        if (turn) {
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int c = 0; c < NCB; ++c) {
              const u4 t = ring[0][u][c];
              ring[0][u][c] = ring[1][u][c];
              ring[1][u][c] = t;
            }
        }
      }
    }
    if constexpr (RNG) {
      if (nparts == 1) {
        flush(rg);
        return;
      }
    }
    int ln = lane;  // (opaque here too)
    asm volatile("" : "+v"(ln));
    auto store = [&](int a, int c, f4 k) __attribute__((always_inline)) {
      const int sl = s_base + a / JB, col = (b0 + c) * 16 + (ln & 15);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int i = (a % JB) * 16 + 4 * (ln >> 4) + t;
        if (sl < ns && i < o && col < v) {
          if constexpr (RNG && !ADD) {  // (the whole split's sum with its first range, zeros with the others)
            for (int r = 0; r < m; ++r)
              P[(((size_t)(sp * m + r) * ns + sl) * o + i) * v + col] = r ? 0.f : scale * k[t];
          } else {
            P[(((size_t)sp * ns + sl) * o + i) * v + col] = scale * k[t];
          }
        }
      }
    };
    if (nparts == 1) {
#pragma unroll
      for (int a = 0; a < KB; ++a)
#pragma unroll
        for (int c = 0; c < NCB; ++c) store(a, c, K[a][c]);
      return;
    }
    // the parts' sums meet in LDS (X is no longer needed), added in order, the blocks dealt to the parts
    constexpr int SLOT = KB * NCBM * 1024;
    __syncthreads();
#pragma unroll
    for (int a = 0; a < KB; ++a)
#pragma unroll
      for (int c = 0; c < NCB; ++c)
        *reinterpret_cast<f4 *>(ldsr + (size_t)wave * SLOT + (a * NCB + c) * 1024 + lane * 16) = K[a][c];
    __syncthreads();
    for (int f = part; f < KB * NCB; f += nparts) {
      f4 k = f4{0.f, 0.f, 0.f, 0.f};
      for (int p = 0; p < nparts; ++p)
        k += *reinterpret_cast<const f4 *>(ldsr + (size_t)(p * pstride + grp) * SLOT + f * 1024 + lane * 16);
      store(f / NCB, f % NCB, k);
    }
  };
  auto go = [&](int w, int b0, int qa, int qb, int part, int nparts, int grp, int pstride)
                __attribute__((always_inline)) {
    switch (w) {
      case 1: run(std::integral_constant<int, 1>{}, b0, qa, qb, part, nparts, grp, pstride); break;
      case 2: if constexpr (NCBM >= 2) run(std::integral_constant<int, 2>{}, b0, qa, qb, part, nparts, grp, pstride); break;
      case 3: if constexpr (NCBM >= 3) run(std::integral_constant<int, 3>{}, b0, qa, qb, part, nparts, grp, pstride); break;
      case 4: if constexpr (NCBM >= 4) run(std::integral_constant<int, 4>{}, b0, qa, qb, part, nparts, grp, pstride); break;
      case 5: if constexpr (NCBM >= 5) run(std::integral_constant<int, 5>{}, b0, qa, qb, part, nparts, grp, pstride); break;
      default:  // no columns for this wave: it keeps the barriers
        if (nparts > 1) {
          __syncthreads();
          __syncthreads();
        }
        break;
    }
  };
  for (int phase = 0; phase < (rem ? 2 : 1); ++phase) {
    int cg = wave % ncg, part = wave / ncg, nparts = qs, pstride = ncg, b0 = 0, w = 0;
    int qa0 = EACH ? bound(range) : Qa, qb0 = EACH ? bound(range + 1) : Qb;
    if (phase == 0) {
      if (part < qs) group_blocks(t1 - t0, rem, ncg, cg, b0, w);
    } else {
      cg = 0, part = wave, nparts = NWAVE, pstride = 1, b0 = t1 - t0 - rem, w = rem;
      if (EACH) qa0 = Qa, qb0 = range == 0 ? Qb : Qa;
    }
    const int qa = qa0 + (int)((long long)part * (qb0 - qa0) / nparts);
    const int qb = qa0 + (int)((long long)(part + 1) * (qb0 - qa0) / nparts);
    go(w, t0 + b0, qa, qb, part, nparts, cg, pstride);
  }
}

// nsplit splits of m ranges: a workgroup per split (whole), which leaves one slab (FP32) or m, or a workgroup and a
// slab per range
template <bool BF, int JB, int KS, int NCBM, bool PK>
hipError_t launch_xres_ranges(hipStream_t s, const void *Boo, const void *Bvv, const void *X, const void *Xlo, int o,
                              int v, int nq, int ns, int nsplit, int m, bool whole, float scale, float *P) {
  using C = CfgR<BF, JB, KS, NCBM, PK>;
  const Split sp = choose_split(v, NCBM);
  if (o > C::OMAX || o < 4 || (BF && JB > 1 && o < 8) || v < C::GV || v > C::VMAX || nsplit < 1 || m < 1 ||
      (long long)nsplit * m > nq || (m > 1 && sp.qs > 1))
    return hipErrorInvalidValue;
  const int nst = ((v + C::GV - 1) / C::GV + 3) / 4;  // K steps
  const size_t lds = std::max((size_t)nst * C::STEP_LDS, sp.qs > 1 || sp.rem ? (size_t)NWAVE * C::KB * NCBM * 1024 : (size_t)0);
  if (lds > LDS_MAX) return hipErrorInvalidValue;
  const int n_sg = (ns + KS - 1) / KS;
  const int per_tile = whole ? nsplit : nsplit * m, total = n_sg * sp.nct * per_tile;  // workgroups
  const dim3 grid((total + 7) / 8 * 8);
  auto go = [&](auto rng) {
    hipLaunchKernelGGL((k_exchange_res<BF, JB, KS, NCBM, PK, decltype(rng)::value>), grid, dim3(64 * NWAVE), lds, s,
                       static_cast<const char *>(Boo), static_cast<const char *>(Bvv), static_cast<const char *>(X),
                       static_cast<const char *>(Xlo), o, v, nq, ns, n_sg, sp.nct, sp.ncg, sp.qs, sp.rem, per_tile,
                       m, scale, P);
  };
  if (m == 1) go(std::integral_constant<int, 0>{});
  else if (whole) go(std::integral_constant<int, 2>{});
  else go(std::integral_constant<int, 1>{});
  return hipGetLastError();
}

template <bool BF, int JB, int KS, int NCBM, bool PK>
hipError_t launch_xres(hipStream_t s, const void *Boo, const void *Bvv, const void *X, const void *Xlo, int o, int v,
                       int nq, int ns, int nsplit, float scale, float *P, void *, size_t) {
  return launch_xres_ranges<BF, JB, KS, NCBM, PK>(s, Boo, Bvv, X, Xlo, o, v, nq, ns, nsplit, 1, true, scale, P);
}

template <bool BF, int JB, int KS, int NCBM, bool PK>
hipError_t prepare_xres() {
  const void *fn[] = {reinterpret_cast<const void *>(&k_exchange_res<BF, JB, KS, NCBM, PK, 0>),
                      reinterpret_cast<const void *>(&k_exchange_res<BF, JB, KS, NCBM, PK, 1>),
                      reinterpret_cast<const void *>(&k_exchange_res<BF, JB, KS, NCBM, PK, 2>)};
  for (const void *f : fn) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_MAX);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// What auto_splits needs of a shape: workgroups per Q split, Q subranges per workgroup, and the cycles
// of a workgroup per Q (of one subrange) and before its first.
template <bool BF, int JB, int KS, int NCBM, bool PK>
void shape_xres(int v, int ns, ResShape *r) {
  using C = CfgR<BF, JB, KS, NCBM, PK>;
  const Split sp = choose_split(v, NCBM);
  const int nst = ((v + C::GV - 1) / C::GV + 3) / 4;
  const double per_block = (double)nst * C::RB * (BF ? 2 * 16 : 4 * 32) +
                           (BF ? 2 * 16 * ((JB + 1) / 2) : 4 * 32 * JB) * (double)C::KB;  // matrix cycles per Q
  const int nb = ((v + 15) / 16 + sp.nct - 1) / sp.nct;
  r->tiles = (ns + KS - 1) / KS * sp.nct;
  // (split BF16 waves of 16 W and 16 K blocks spill even without ranges, more with them: 6 to 8 % of a full launch
  // of o64 v440 N_Q1461, 6 RHS, o32 v452 N_Q1461, 16, and o32 v470 N_Q1500, 8)
  r->ranges = sp.qs == 1 && !(BF && C::RB * ((nb - sp.rem + sp.ncg - 1) / sp.ncg) >= 16);
  r->qs = sp.qs;
  // (a wave of two row blocks waits longer for its operands per product than one of three or four)
  r->q_cycles = per_block * ((nb + sp.ncg - 1) / sp.ncg) * 2 / (BF ? (C::RB > 2 ? 0.45 : 0.35) : 0.85);
  r->start_cycles = 5000.0 + nst * C::STEP_LDS / 40.0;
}

// Column blocks per wave: as many as keep the accumulators, the ring and two halves of a step's X
// within (about) the 256 registers of two waves per SIMD.
#define XRES_(BF, JB, KS, NCBM, PK, NAME)                                                                          \
  ExchangeVariant {                                                                                                \
    BF ? RTTDA_PREC_MIXED_BF16 : RTTDA_PREC_FP32, CfgR<BF, JB, KS, NCBM, PK>::OMAX, KS, 16 * NWAVE * NCBM, NAME,   \
        &launch_xres<BF, JB, KS, NCBM, PK>, LDS_MAX, &prepare_xres<BF, JB, KS, NCBM, PK>,                          \
        CfgR<BF, JB, KS, NCBM, PK>::GV, 1, 1, JB > 1 ? 8 : 4, false, 3, CfgR<BF, JB, KS, NCBM, PK>::VMAX,          \
        &shape_xres<BF, JB, KS, NCBM, PK>, &launch_xres_ranges<BF, JB, KS, NCBM, PK>                               \
  }
#define XRES(BF, JB, KS, NCBM, NAME) XRES_(BF, JB, KS, NCBM, false, NAME)

const ExchangeVariant kResF32[] = {
    XRES(false, 4, 1, 4, "f32r_o64"), XRES(false, 3, 1, 4, "f32r_o48"), XRES(false, 2, 2, 4, "f32r_o32_s2"),
    XRES(false, 2, 1, 5, "f32r_o32_s1"), XRES(false, 1, 2, 5, "f32r_o16_s2"),
    XRES_(false, 3, 2, 3, true, "f32r_p40"), XRES_(false, 2, 2, 4, true, "f32r_p24"),
};
const ExchangeVariant kResBf16[] = {
    XRES(true, 4, 1, 4, "bf16x2r_o64"), XRES(true, 3, 1, 4, "bf16x2r_o48"), XRES(true, 2, 2, 4, "bf16x2r_o32_s2"),
    XRES(true, 2, 1, 5, "bf16x2r_o32_s1"), XRES(true, 1, 2, 5, "bf16x2r_o16_s2"),
};

}  // namespace

int exchange_res_variant_count(int prec) {
  return prec == RTTDA_PREC_FP32 ? (int)(sizeof(kResF32) / sizeof(kResF32[0])) : (int)(sizeof(kResBf16) / sizeof(kResBf16[0]));
}
const ExchangeVariant *exchange_res_variant(int prec, int k) {
  return prec == RTTDA_PREC_FP32 ? &kResF32[k] : &kResBf16[k];
}

}  // namespace rttda
