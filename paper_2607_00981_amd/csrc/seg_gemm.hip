// Segmented FP64 products over a device table of items: the accumulators of the
// (Q) tasks and the T2 drivers of a slab, one launch for every task or block.
#include <algorithm>
#include <climits>

#include "internal.h"

namespace cct {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double dbl2 __attribute__((ext_vector_type(2)));
constexpr int SBK = 16;

__device__ __forceinline__ long long map4(const Idx4& d, int i) {
  const unsigned u = (unsigned)i;
  const unsigned d3 = u % (unsigned)d.n3, r3 = u / (unsigned)d.n3;
  const unsigned d2 = r3 % (unsigned)d.n2, r2 = r3 / (unsigned)d.n2;
  const unsigned d1 = r2 % (unsigned)d.n1, d0 = r2 / (unsigned)d.n1;
  return (long long)d0 * d.s0 + (long long)d1 * d.s1 + (long long)d2 * d.s2 + (long long)d3 * d.s3;
}

// blockIdx.x -> item and output tile (xcd_place), tiles grouped by 8 rows of tiles.
__device__ __forceinline__ bool seg_tile(int tiles_m, int tiles_n, int batch, int& tm, int& tn, int& z) {
  int pid;
  if (!xcd_place(tiles_m * tiles_n, batch, pid, z)) return false;
  constexpr int GM = 8;
  const int group = pid / (GM * tiles_n);
  const int first_m = group * GM;
  const int gsize = min(tiles_m - first_m, GM);
  const int r = pid - group * GM * tiles_n;
  tm = first_m + r % gsize;
  tn = r / gsize;
  return true;
}

// C_z(m, n) (+)= sum_s coef_s sum_k A_s(m, k) B_s(k, n), one item z and tile per workgroup (xcd_place).
//
// Bound: at v = 48 the products of one task are 24 v^5 multiply-adds against
// 14 updates of a v^4 array, about 13 FLOP per byte of accumulator traffic, so
// the matrix cores and HBM are both near their limits; what the layout avoids
// is everything else.  The tile is BM x BN = (16 TM WM) x (16 TN WN) with
// WM x WN waves.  The K index runs over the item's segments without a gap (a
// K = o segment does not start on a K tile of its own: at o = 6 padding each
// to 16 would be 2.7x the work), every thread keeping the segment and the k of
// its load units.  SWAP exchanges the MFMA operands so that a wave's 16
// consecutive lanes run along m instead of n: the caller sets it where the
// unit-stride axis of C is among the rows, and the update stays in 128-byte
// runs for all seven groups of axes.
template <int TM, int TN, int WM, int WN, bool SWAP, bool VEC>
__global__ __launch_bounds__(64 * WM * WN) void seg_gemm_kernel(SegGemm g, int tiles_m, int tiles_n) {
  constexpr int NTH = 64 * WM * WN, BM = 16 * TM * WM, BN = 16 * TN * WN;
  constexpr int LA = BM + 2, LB = BN + 2;
  constexpr int W = VEC ? 2 : 1;
  constexpr int UA = BM * SBK / W, UB = BN * SBK / W;  // load units per K tile
  constexpr int NA = (UA + NTH - 1) / NTH, NB = (UB + NTH - 1) / NTH;
  __shared__ double As[2][SBK * LA];
  __shared__ double Bs[2][SBK * LB];
  int tm, tn, z;
  if (!seg_tile(tiles_m, tiles_n, g.nitems, tm, tn, z)) return;
  const int tid = threadIdx.x;
  const SegItem& it = g.items[z];
  const int m0 = tm * BM, n0 = tn * BN, nseg = it.nseg, K = g.K, ktot = nseg * K;
  int ak[NA], as_[NA], ar[NA], ad0[NA], ad1[NA], ad2[NA], bk[NB], bs_[NB], br[NB];
  const double *pa[NA], *pb[NB];
  double ca[NA];
  bool va[NA], vb[NB];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int u = tid + i * NTH;
    ar[i] = u / (SBK / W);
    ak[i] = (u % (SBK / W)) * W;
    as_[i] = 0;
    const unsigned m = (unsigned)(m0 + ar[i]);
    va[i] = u < UA && (int)m < g.M;
    ad2[i] = (int)(m % (unsigned)g.n2);
    const unsigned r = m / (unsigned)g.n2;
    ad1[i] = (int)(r % (unsigned)g.n1);
    ad0[i] = (int)(r / (unsigned)g.n1);
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int u = tid + i * NTH;
    bk[i] = u / (BN / W);
    br[i] = (u % (BN / W)) * W;
    bs_[i] = 0;
    vb[i] = u < UB && n0 + br[i] < g.N;
  }
  // the segment that holds the unit's k, and the unit's row in it
  auto enter_a = [&](int i) {
    while (ak[i] >= K && as_[i] < nseg) {
      ak[i] -= K;
      ++as_[i];
    }
    if (!va[i] || as_[i] >= nseg) return;
    const SegOp& s = it.seg[as_[i]];
    pa[i] = s.a + (long long)ad0[i] * s.rs0 + (long long)ad1[i] * s.rs1 + (long long)ad2[i] * s.rs2;
    ca[i] = s.coef;
  };
  auto enter_b = [&](int i) {
    while (bk[i] >= K && bs_[i] < nseg) {
      bk[i] -= K;
      ++bs_[i];
    }
    if (!vb[i] || bs_[i] >= nseg) return;
    pb[i] = it.seg[bs_[i]].b + (n0 + br[i]);
  };
#pragma unroll
  for (int i = 0; i < NA; ++i) enter_a(i);
#pragma unroll
  for (int i = 0; i < NB; ++i) enter_b(i);
  dbl2 ra[NA], rb[NB];
  // raw loads; masking happens at the LDS store, after the products
  bool oa[NA], ob[NB];
  double sa[NA];
  auto load = [&]() {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      oa[i] = va[i] && as_[i] < nseg;
      sa[i] = ca[i];
      if (oa[i]) {
        if constexpr (VEC) ra[i] = *(const dbl2*)(pa[i] + ak[i]);
        else ra[i].x = pa[i][ak[i]];
      }
      ak[i] += SBK;
      if (ak[i] >= K) enter_a(i);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      ob[i] = vb[i] && bs_[i] < nseg && bk[i] < g.kb;
      if (ob[i]) {
        const double* p = pb[i] + (long long)bk[i] * it.seg[bs_[i]].ldb;
        if constexpr (VEC) rb[i] = *(const dbl2*)p;
        else rb[i].x = *p;
      }
      bk[i] += SBK;
      if (bk[i] >= K) enter_b(i);
    }
  };
  auto store = [&](double* as, double* bs) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int u = tid + i * NTH;
      if (u >= UA) continue;
      const int k = (u % (SBK / W)) * W;
      as[k * LA + ar[i]] = oa[i] ? sa[i] * ra[i].x : 0.0;
      if constexpr (VEC) as[(k + 1) * LA + ar[i]] = oa[i] ? sa[i] * ra[i].y : 0.0;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int u = tid + i * NTH;
      if (u >= UB) continue;
      const int k = u / (BN / W);
      bs[k * LB + br[i]] = ob[i] ? rb[i].x : 0.0;
      if constexpr (VEC) bs[k * LB + br[i] + 1] = ob[i] ? rb[i].y : 0.0;
    }
  };

  const int wave = tid / 64, lane = tid & 63;
  const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
  d4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  const int total = (ktot + SBK - 1) / SBK;
  if (total > 0) {
    load();
    store(As[0], Bs[0]);
  }
  __syncthreads();
  for (int t = 0; t < total; ++t) {
    const int cur = t & 1;
    if (t + 1 < total) load();
    const double* as = As[cur];
    const double* bs = Bs[cur];
#pragma unroll
    for (int ks = 0; ks < SBK / 4; ++ks) {
      const int kr = ks * 4 + lane / 16;
      double af[TM], bf[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = as[kr * LA + wm0 + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < TN; ++j) bf[j] = bs[kr * LB + wn0 + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = SWAP ? __builtin_amdgcn_mfma_f64_16x16x4f64(bf[j], af[i], acc[i][j], 0, 0, 0)
                           : __builtin_amdgcn_mfma_f64_16x16x4f64(af[i], bf[j], acc[i][j], 0, 0, 0);
    }
    if (t + 1 < total) store(As[cur ^ 1], Bs[cur ^ 1]);
    __syncthreads();
  }
  // accumulator register r of lane l: first MFMA operand's index 4r + l/16,
  // second operand's l%16.  Per 16 rows every load of C precedes the stores.
  double* C = g.C + it.c;
  if constexpr (!SWAP) {
    long long cof[TN];
    bool cin[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn0 + j * 16 + (lane & 15);
      cin[j] = n < g.N;
      cof[j] = cin[j] ? map4(g.cn, n) : 0;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      double cur[4][TN];
      double* row[4];
      bool rin[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm0 + i * 16 + 4 * r + lane / 16;
        rin[r] = m < g.M;
        row[r] = C + (rin[r] ? map4(g.cm, m) : 0);
#pragma unroll
        for (int j = 0; j < TN; ++j) cur[r][j] = (g.accumulate && rin[r] && cin[j]) ? row[r][cof[j]] : 0.0;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          if (rin[r] && cin[j]) row[r][cof[j]] = cur[r][j] + acc[i][j][r];
    }
  } else {
    long long rof[TM];
    bool rin[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + wm0 + i * 16 + (lane & 15);
      rin[i] = m < g.M;
      rof[i] = rin[i] ? map4(g.cm, m) : 0;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      double cur[4][TM];
      double* col[4];
      bool cin[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int n = n0 + wn0 + j * 16 + 4 * r + lane / 16;
        cin[r] = n < g.N;
        col[r] = C + (cin[r] ? map4(g.cn, n) : 0);
#pragma unroll
        for (int i = 0; i < TM; ++i) cur[r][i] = (g.accumulate && cin[r] && rin[i]) ? col[r][rof[i]] : 0.0;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < TM; ++i)
          if (cin[r] && rin[i]) col[r][rof[i]] = cur[r][i] + acc[i][j][r];
    }
  }
}

template <int TM, int TN, int WM, int WN>
hipError_t seg_launch(const SegGemm& g, bool vec, hipStream_t s) {
  constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN;
  const long long tiles_m = ((long long)g.M + BM - 1) / BM, tiles_n = ((long long)g.N + BN - 1) / BN;
  const long long gx = xcd_grid(tiles_m * tiles_n, g.nitems);
  if (gx > INT_MAX) return hipErrorInvalidValue;
  const dim3 grid((unsigned)gx), block(64 * WM * WN);
  if (g.swap) {
    if (vec) hipLaunchKernelGGL((seg_gemm_kernel<TM, TN, WM, WN, true, true>), grid, block, 0, s, g, (int)tiles_m, (int)tiles_n);
    else hipLaunchKernelGGL((seg_gemm_kernel<TM, TN, WM, WN, true, false>), grid, block, 0, s, g, (int)tiles_m, (int)tiles_n);
  } else {
    if (vec) hipLaunchKernelGGL((seg_gemm_kernel<TM, TN, WM, WN, false, true>), grid, block, 0, s, g, (int)tiles_m, (int)tiles_n);
    else hipLaunchKernelGGL((seg_gemm_kernel<TM, TN, WM, WN, false, false>), grid, block, 0, s, g, (int)tiles_m, (int)tiles_n);
  }
  return hipGetLastError();
}

}  // namespace

long long idx4_max(const Idx4& d, long long n) {
  const long long r[4] = {0, d.n1, d.n2, d.n3}, st[4] = {d.s0, d.s1, d.s2, d.s3};
  long long dg[4], x = n - 1;
  for (int k = 3; k >= 1; --k) {
    dg[k] = x % r[k];
    x /= r[k];
  }
  dg[0] = x;
  long long best = 0;
  for (int k = 0; k < 4; ++k) best += dg[k] * st[k];
  for (int k = 0; k < 4; ++k) {
    if (dg[k] == 0) continue;
    long long alt = 0;
    for (int j = 0; j < k; ++j) alt += dg[j] * st[j];
    alt += (dg[k] - 1) * st[k];
    for (int j = k + 1; j < 4; ++j) alt += (r[j] - 1) * st[j];
    best = std::max(best, alt);
  }
  return best;
}

hipError_t seg_gemm(const SegGemm& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.nitems <= 0) return hipSuccess;
  if (g.K <= 0 || g.kb < 1 || g.kb > g.K || !g.items || g.n1 < 1 || g.n2 < 1) return hipErrorInvalidValue;
  if (g.vec && ((g.K | g.N) & 1)) return hipErrorInvalidValue;
  for (const Idx4* d : {&g.cm, &g.cn})
    if (d->n1 < 1 || d->n2 < 1 || d->n3 < 1 || d->s0 < 0 || d->s1 < 0 || d->s2 < 0 || d->s3 < 0)
      return hipErrorInvalidValue;
  if (g.c_last < 0 || g.c_last + idx4_max(g.cm, g.M) + idx4_max(g.cn, g.N) >= g.c_len) return hipErrorInvalidValue;
  const bool vec = g.vec;
  // A skinny side (the v labels of one axis) takes the narrowest tile of 32,
  // 48 or 64 that wastes least, against 64 of the long side: the update of C
  // and the short K want workgroups in flight more than operand reuse (o = 6,
  // v = 48, whole evaluation: 128 x 48 tiles 65.2 ms, 64 x 48 61.7, 256 x 48
  // 73.1; not measured anew at other v).  The square products take 128 x 128 with eight waves of 32 x 64
  // where those tiles are filled (four waves of 64 x 64 65.2 ms, eight 58.5,
  // 64 x 64 tiles 59.6), else 64 x 64.
  auto pad = [](int n, int b) { return (n + b - 1) / b * b; };
  if (g.N <= g.M / 4 || g.M <= g.N / 4) {
    const bool small_n = g.N <= g.M / 4;
    const int n = small_n ? g.N : g.M;
    int best = 64;
    for (int b : {48, 32})
      if (pad(n, b) < pad(n, best)) best = b;
    if (small_n) {
      if (best == 64) return seg_launch<1, 4, 4, 1>(g, vec, s);   // 64 x 64
      if (best == 48) return seg_launch<1, 3, 4, 1>(g, vec, s);   // 64 x 48
      return seg_launch<1, 2, 4, 1>(g, vec, s);                   // 64 x 32
    }
    if (best == 64) return seg_launch<4, 1, 1, 4>(g, vec, s);     // 64 x 64
    if (best == 48) return seg_launch<3, 1, 1, 4>(g, vec, s);     // 48 x 64
    return seg_launch<2, 1, 1, 4>(g, vec, s);                     // 32 x 64
  }
  if (pad(g.M, 128) * (long long)pad(g.N, 128) <= 1.1 * pad(g.M, 64) * (long long)pad(g.N, 64) && g.M >= 1024)
    return seg_launch<2, 4, 4, 2>(g, vec, s);  // 128 x 128
  return seg_launch<2, 2, 2, 2>(g, vec, s);    // 64 x 64
}

}  // namespace cct
