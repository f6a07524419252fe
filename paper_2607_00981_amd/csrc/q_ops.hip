// Kernels of the perturbative quadruples correction in the occupied-tuple
// order: the segmented products that accumulate a task's 24-permutation sums,
// and the task energies with the spin summation.
#include <algorithm>
#include <climits>
#include <cmath>

#include "internal.h"

namespace cct {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double dbl2 __attribute__((ext_vector_type(2)));
constexpr int QBK = 16;

__device__ __forceinline__ long long map4(const Idx4& d, int i) {
  const unsigned u = (unsigned)i;
  const unsigned d3 = u % (unsigned)d.n3, r3 = u / (unsigned)d.n3;
  const unsigned d2 = r3 % (unsigned)d.n2, r2 = r3 / (unsigned)d.n2;
  const unsigned d1 = r2 % (unsigned)d.n1, d0 = r2 / (unsigned)d.n1;
  return (long long)d0 * d.s0 + (long long)d1 * d.s1 + (long long)d2 * d.s2 + (long long)d3 * d.s3;
}

// blockIdx.x -> output tile: each XCD takes a contiguous range of a tile order
// grouped by 8 rows of tiles (see q_abc.hip).
__device__ __forceinline__ bool q_tile(int tiles_m, int tiles_n, int& tm, int& tn) {
  const int nb = tiles_m * tiles_n;
  const int per = (nb + 7) / 8;
  const int bid = blockIdx.x;
  const int pid = (bid % 8) * per + bid / 8;
  if (pid >= nb) return false;
  constexpr int GM = 8;
  const int group = pid / (GM * tiles_n);
  const int first_m = group * GM;
  const int gsize = min(tiles_m - first_m, GM);
  const int r = pid - group * GM * tiles_n;
  tm = first_m + r % gsize;
  tn = r / gsize;
  return true;
}

// C_z(m, n) (+)= sum_s coef_s sum_k A_s(m, k) B_s(k, n), one item z per grid z.
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
__global__ __launch_bounds__(64 * WM * WN) void qo_gemm_kernel(QoGemm g, int tiles_m, int tiles_n) {
  constexpr int NTH = 64 * WM * WN, BM = 16 * TM * WM, BN = 16 * TN * WN;
  constexpr int LA = BM + 2, LB = BN + 2;
  constexpr int W = VEC ? 2 : 1;
  constexpr int UA = BM * QBK / W, UB = BN * QBK / W;  // load units per K tile
  constexpr int NA = (UA + NTH - 1) / NTH, NB = (UB + NTH - 1) / NTH;
  __shared__ double As[2][QBK * LA];
  __shared__ double Bs[2][QBK * LB];
  int tm, tn;
  if (!q_tile(tiles_m, tiles_n, tm, tn)) return;
  const int tid = threadIdx.x;
  const QoItem& it = g.items[blockIdx.z];
  const int m0 = tm * BM, n0 = tn * BN, K = g.K, ktot = it.nseg * K;
  int ak[NA], as_[NA], ar[NA], ad0[NA], ad1[NA], ad2[NA], bk[NB], bs_[NB], br[NB];
  const double *pa[NA], *pb[NB];
  double ca[NA];
  bool va[NA], vb[NB];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int u = tid + i * NTH;
    ar[i] = u / (QBK / W);
    ak[i] = (u % (QBK / W)) * W;
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
    while (ak[i] >= K && as_[i] < it.nseg) {
      ak[i] -= K;
      ++as_[i];
    }
    if (!va[i] || as_[i] >= it.nseg) return;
    const QoSeg& s = it.seg[as_[i]];
    pa[i] = s.a + (long long)ad0[i] * s.rs0 + (long long)ad1[i] * s.rs1 + (long long)ad2[i] * s.rs2;
    ca[i] = s.coef;
  };
  auto enter_b = [&](int i) {
    while (bk[i] >= K && bs_[i] < it.nseg) {
      bk[i] -= K;
      ++bs_[i];
    }
    if (!vb[i] || bs_[i] >= it.nseg) return;
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
      oa[i] = va[i] && as_[i] < it.nseg;
      sa[i] = ca[i];
      if (oa[i]) {
        if constexpr (VEC) ra[i] = *(const dbl2*)(pa[i] + ak[i]);
        else ra[i].x = pa[i][ak[i]];
      }
      ak[i] += QBK;
      if (ak[i] >= K) enter_a(i);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      ob[i] = vb[i] && bs_[i] < it.nseg;
      if (ob[i]) {
        const double* p = pb[i] + (long long)bk[i] * it.seg[bs_[i]].ldb;
        if constexpr (VEC) rb[i] = *(const dbl2*)p;
        else rb[i].x = *p;
      }
      bk[i] += QBK;
      if (bk[i] >= K) enter_b(i);
    }
  };
  auto store = [&](double* as, double* bs) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int u = tid + i * NTH;
      if (u >= UA) continue;
      const int k = (u % (QBK / W)) * W;
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
  const int total = (ktot + QBK - 1) / QBK;
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
    for (int ks = 0; ks < QBK / 4; ++ks) {
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
hipError_t qo_launch(const QoGemm& g, bool vec, hipStream_t s) {
  constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN;
  const long long tiles_m = ((long long)g.M + BM - 1) / BM, tiles_n = ((long long)g.N + BN - 1) / BN;
  const long long gx = ((tiles_m * tiles_n + 7) / 8) * 8;
  if (gx > INT_MAX) return hipErrorInvalidValue;
  const dim3 grid((unsigned)gx, 1, (unsigned)g.nitems), block(64 * WM * WN);
  if (g.swap) {
    if (vec) hipLaunchKernelGGL((qo_gemm_kernel<TM, TN, WM, WN, true, true>), grid, block, 0, s, g, (int)tiles_m, (int)tiles_n);
    else hipLaunchKernelGGL((qo_gemm_kernel<TM, TN, WM, WN, true, false>), grid, block, 0, s, g, (int)tiles_m, (int)tiles_n);
  } else {
    if (vec) hipLaunchKernelGGL((qo_gemm_kernel<TM, TN, WM, WN, false, true>), grid, block, 0, s, g, (int)tiles_m, (int)tiles_n);
    else hipLaunchKernelGGL((qo_gemm_kernel<TM, TN, WM, WN, false, false>), grid, block, 0, s, g, (int)tiles_m, (int)tiles_n);
  }
  return hipGetLastError();
}

// The spin summation 2 (2 - P_cd)(2 - P_bc - P_bd)(2 - P_ab - P_ac - P_ad),
// multiplied out, is a class function of the permutation group: 16 on the
// identity, -8 on transpositions, 4 on three-cycles and on double
// transpositions, -2 on four-cycles.
double spin_class(const int p[4]) {
  int seen[4] = {0, 0, 0, 0}, longest = 0, cycles = 0;
  for (int k = 0; k < 4; ++k) {
    if (seen[k]) continue;
    int len = 0;
    for (int x = k; !seen[x]; x = p[x]) {
      seen[x] = 1;
      ++len;
    }
    longest = std::max(longest, len);
    ++cycles;
  }
  if (longest == 1) return 16.0;
  if (longest == 2 && cycles == 3) return -8.0;
  if (longest == 4) return -2.0;
  return 4.0;
}

// The 24 permutations in lexicographic order.
constexpr unsigned char QO_P[24][4] = {
    {0, 1, 2, 3}, {0, 1, 3, 2}, {0, 2, 1, 3}, {0, 2, 3, 1}, {0, 3, 1, 2}, {0, 3, 2, 1}, {1, 0, 2, 3}, {1, 0, 3, 2},
    {1, 2, 0, 3}, {1, 2, 3, 0}, {1, 3, 0, 2}, {1, 3, 2, 0}, {2, 0, 1, 3}, {2, 0, 3, 1}, {2, 1, 0, 3}, {2, 1, 3, 0},
    {2, 3, 0, 1}, {2, 3, 1, 0}, {3, 0, 1, 2}, {3, 0, 2, 1}, {3, 1, 0, 2}, {3, 1, 2, 0}, {3, 2, 0, 1}, {3, 2, 1, 0}};
// Per class of tasks (bit 0: i = j, bit 1: j = k, bit 2: k = l; no three are
// equal, so 0, 1, 2, 4 and 5 occur) the coefficients of U.
struct QoCoef {
  double c[6][24];
};

// The virtual index space v^4 is cut into blocks of 4^4; the axis permutations
// act on whole blocks, so an orbit of blocks (at most 24) is closed under
// them.  One workgroup takes one task and one orbit, each thread the same
// element of every block: it stages R = X + Y of the orbit's blocks in LDS
// (each element of X and Y read from memory once, one more read of X at the end) and
// evaluates U = (sum_pi c_pi R o pi) / den there.  The 24 permuted reads are
// LDS reads at offsets fixed per thread plus the block's slot, which is the
// same for the whole workgroup; the levels of a block are padded by one double
// each (85, 21, 5, 1) so that a permuted read does not put a level on one bank.
// Each XCD takes a contiguous range of orbits: neighbouring blocks share lines
// of X and Y.  Bound by the LDS reads.  o = 6, v = 48: 0.23 -> 0.087 ms per task
// against computed permutations with one block element per loop step.
constexpr int QOB = 4, QOB4 = QOB * QOB * QOB * QOB, QOLD = 4 * 85;
__global__ __launch_bounds__(QOB4) void qo_energy_kernel(const double* __restrict__ X, const double* __restrict__ Y,
                                                         const double* __restrict__ VVOO,
                                                         const double* __restrict__ t2,
                                                         const double* __restrict__ eps,
                                                         const int4* __restrict__ tasks,
                                                         const unsigned* __restrict__ orbits, QoCoef Q, int o, int v,
                                                         int norb, double* __restrict__ part) {
  __shared__ double Rl[24 * QOLD];
  __shared__ double red[QOB4];
  __shared__ int blk[24][4], slot_of[24], perm_of[24], nblk_s;
  __shared__ __attribute__((aligned(16))) unsigned short smap[24][24];  // slot of block o pi, times QOLD
  const int per = (norb + 7) / 8;
  const int orb = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  if (orb >= norb) return;
  const int4 tk = tasks[blockIdx.y];
  const int oc[4] = {tk.x, tk.y, tk.z, tk.w};
  const unsigned ob = orbits[orb];  // block coordinates b0 <= b1 <= b2 <= b3, a byte each
  if (threadIdx.x < 64) {
    // lane p < 24: block number p of the orbit, its slot the rank among the distinct ones
    const int p = min((int)threadIdx.x, 23);
    int q[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = (int)((ob >> (8 * QO_P[p][k])) & 255u);
    const unsigned code = (unsigned)q[0] | (unsigned)q[1] << 8 | (unsigned)q[2] << 16 | (unsigned)q[3] << 24;
    int first = 23;
    for (int t = 22; t >= 0; --t)
      if (__shfl(code, t) == code) first = t;
    first = min(first, p);
    const unsigned long long lead = __ballot(threadIdx.x < 24 && first == p);
    const int slot = __popcll(lead & ((1ull << first) - 1));
    if (threadIdx.x < 24) {
      slot_of[p] = slot;
      if (first == p) {
        for (int k = 0; k < 4; ++k) blk[slot][k] = q[k];
        perm_of[slot] = p;
      }
    }
    if (threadIdx.x == 0) nblk_s = __popcll(lead);
  }
  __syncthreads();
  const int nblk = nblk_s;
  for (int e = threadIdx.x; e < nblk * 24; e += QOB4) {
    // block number f composed with permutation p is block number f o p (lexicographic rank)
    const int sidx = e / 24, p = e % 24, f = perm_of[sidx];
    int t[4];
    for (int k = 0; k < 4; ++k) t[k] = QO_P[f][QO_P[p][k]];
    const int r = 6 * t[0] + 2 * (t[1] - (t[1] > t[0])) + (t[2] > t[3] ? 1 : 0);
    smap[sidx][p] = (unsigned short)(slot_of[r] * QOLD);
  }
  const int w = threadIdx.x;
  const int j[4] = {w >> 6, (w >> 4) & 3, (w >> 2) & 3, w & 3};
  const long long v1 = v, v2 = v1 * v, v4 = v2 * v2;
  const double* x = X + (long long)blockIdx.y * v4;
  const double* yy = Y + (long long)blockIdx.y * v4;
  const int at0 = j[0] * 85 + j[1] * 21 + j[2] * 5 + j[3];
#pragma unroll 4
  for (int k = 0; k < nblk; ++k) {
    const int w0 = blk[k][0] * QOB + j[0], w1 = blk[k][1] * QOB + j[1];
    const int w2 = blk[k][2] * QOB + j[2], w3 = blk[k][3] * QOB + j[3];
    const long long at = (w0 * v1 + w1) * v2 + w2 * v1 + w3;
    Rl[k * QOLD + at0] = (w0 < v && w1 < v && w2 < v && w3 < v) ? x[at] + yy[at] : 0.0;
  }
  int jj[24];
#pragma unroll
  for (int p = 0; p < 24; ++p) jj[p] = j[QO_P[p][0]] * 85 + j[QO_P[p][1]] * 21 + j[QO_P[p][2]] * 5 + j[QO_P[p][3]];
  __syncthreads();
  const int cls = (oc[0] == oc[1] ? 1 : 0) + (oc[1] == oc[2] ? 2 : 0) + (oc[2] == oc[3] ? 4 : 0);
  const double istab = cls == 0 ? 1.0 : (cls == 5 ? 0.25 : 0.5);
  const double eo = eps[oc[0]] + eps[oc[1]] + eps[oc[2]] + eps[oc[3]];
  const double* ev = eps + o;
  double acc = 0.0;
#pragma unroll 2
  for (int k = 0; k < nblk; ++k) {
    const int i[4] = {blk[k][0] * QOB + j[0], blk[k][1] * QOB + j[1], blk[k][2] * QOB + j[2], blk[k][3] * QOB + j[3]};
    if (i[0] >= v || i[1] >= v || i[2] >= v || i[3] >= v) continue;
    // U vanishes where three virtual labels are equal (the coefficients sum to
    // zero over the orders of the other label)
    if ((i[0] == i[1] && (i[1] == i[2] || i[1] == i[3])) || (i[2] == i[3] && (i[0] == i[2] || i[1] == i[2]))) continue;
    const double xk = x[(i[0] * v1 + i[1]) * v2 + i[2] * v1 + i[3]];
    const uint4* sp = (const uint4*)smap[k];
    const uint4 s0_ = sp[0], s1_ = sp[1], s2_ = sp[2];
    const unsigned sw[12] = {s0_.x, s0_.y, s0_.z, s0_.w, s1_.x, s1_.y, s1_.z, s1_.w, s2_.x, s2_.y, s2_.z, s2_.w};
    double u = 0.0;
#pragma unroll
    for (int p = 0; p < 24; ++p) {
      const int sl = __builtin_amdgcn_readfirstlane((int)((sw[p / 2] >> (16 * (p & 1))) & 0xffffu));
      u += Q.c[cls][p] * Rl[sl + jj[p]];
    }
    const double den = eo - (ev[i[0]] + ev[i[1]] + ev[i[2]] + ev[i[3]]);
    // the six splits {s0 < s1} | {s2 < s3} of v^{..}_{..} t_{..}^{..}
    double vs = 0.0;
#pragma unroll
    for (int s0 = 0; s0 < 4; ++s0)
#pragma unroll
      for (int s1 = s0 + 1; s1 < 4; ++s1) {
        int s2 = -1, s3 = -1;
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (t != s0 && t != s1) {
            if (s2 < 0) s2 = t;
            else s3 = t;
          }
        vs += VVOO[((long long)oc[s0] * o + oc[s1]) * v2 + (long long)i[s0] * v + i[s1]] *
              t2[((long long)oc[s2] * o + oc[s3]) * v2 + (long long)i[s2] * v + i[s3]];
      }
    acc += (xk + istab * vs) * (u / den);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int t = QOB4 / 2; t > 0; t >>= 1) {
    if ((int)threadIdx.x < t) red[threadIdx.x] += red[threadIdx.x + t];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[(long long)blockIdx.y * norb + orb] = red[0];
}

// orbits[r] = the r-th b0 <= b1 <= b2 <= b3 < nbk (lexicographic), a byte each.
__global__ __launch_bounds__(256) void qo_orbits_kernel(unsigned* __restrict__ orbits, int norb, int nbk) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= norb) return;
  long long r = i;
  unsigned code = 0;
  int lo = 0;
  for (int d = 0; d < 3; ++d) {
    const int left = 3 - d;  // coordinates after this one, each in [x, nbk)
    for (int x = lo;; ++x) {
      const long long m = nbk - x;
      const long long cnt = left == 3 ? m * (m + 1) * (m + 2) / 6 : (left == 2 ? m * (m + 1) / 2 : m);
      if (r < cnt) {
        code |= (unsigned)x << (8 * d);
        lo = x;
        break;
      }
      r -= cnt;
    }
  }
  orbits[i] = code | (unsigned)(lo + (int)r) << 24;
}

// out[at[y]] = sum over x of part[y][x], fixed order.
__global__ __launch_bounds__(256) void qo_reduce_kernel(const double* __restrict__ part, long long n,
                                                        const int* __restrict__ at, double* __restrict__ out) {
  __shared__ double red[256];
  const double* p = part + (long long)blockIdx.x * n;
  double s = 0.0;
  for (long long x = threadIdx.x; x < n; x += blockDim.x) s += p[x];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[at[blockIdx.x]] = red[0];
}

}  // namespace

hipError_t qo_gemm(const QoGemm& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.nitems <= 0) return hipSuccess;
  if (g.K <= 0 || !g.items || g.n1 < 1 || g.n2 < 1 || g.nitems > 65535) return hipErrorInvalidValue;
  const bool vec = g.vec;
  // A skinny side (the v labels of one axis) takes the narrowest tile of 32,
  // 48 or 64 that wastes least, against 64 of the long side: the update of C
  // and the short K want workgroups in flight more than operand reuse (o = 6,
  // v = 48, whole evaluation: 128 x 48 tiles 65.2 ms, 64 x 48 61.7, 256 x 48
  // 73.1).  The square products take 128 x 128 with eight waves of 32 x 64
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
      if (best == 64) return qo_launch<1, 4, 4, 1>(g, vec, s);   // 64 x 64
      if (best == 48) return qo_launch<1, 3, 4, 1>(g, vec, s);   // 64 x 48
      return qo_launch<1, 2, 4, 1>(g, vec, s);                   // 64 x 32
    }
    if (best == 64) return qo_launch<4, 1, 1, 4>(g, vec, s);     // 64 x 64
    if (best == 48) return qo_launch<3, 1, 1, 4>(g, vec, s);     // 48 x 64
    return qo_launch<2, 1, 1, 4>(g, vec, s);                     // 32 x 64
  }
  if (pad(g.M, 128) * (long long)pad(g.N, 128) <= 1.1 * pad(g.M, 64) * (long long)pad(g.N, 64) && g.M >= 1024)
    return qo_launch<2, 4, 4, 2>(g, vec, s);  // 128 x 128
  return qo_launch<2, 2, 2, 2>(g, vec, s);    // 64 x 64
}

long long qo_orbits(int v) {
  const long long n = (v + QOB - 1) / QOB;
  return n * (n + 1) * (n + 2) * (n + 3) / 24;
}

hipError_t qo_orbit_table(unsigned* orbits, int v, hipStream_t s) {
  const long long norb = qo_orbits(v), nbk = (v + QOB - 1) / QOB;
  if (v <= 0) return hipSuccess;
  if (nbk > 256 || norb > INT_MAX - 256) return hipErrorInvalidValue;
  hipLaunchKernelGGL(qo_orbits_kernel, dim3((unsigned)((norb + 255) / 256)), dim3(256), 0, s, orbits, (int)norb,
                     (int)nbk);
  return hipGetLastError();
}

hipError_t qo_energy(const double* X, const double* Y, const double* VVOO, const double* t2, const double* eps,
                     const int4* tasks, const int* at, int ntasks, const unsigned* orbits, int o, int v, double* part,
                     double* etask, hipStream_t s) {
  if (ntasks <= 0 || v <= 0) return hipSuccess;
  const long long norb = qo_orbits(v);
  if (norb > INT_MAX - 8 || ntasks > 65535) return hipErrorInvalidValue;
  QoCoef Q{};
  // c'_sigma = sum over the stabiliser tau of the task of c(sigma o tau)
  const int stab[4][4] = {{0, 1, 2, 3}, {1, 0, 2, 3}, {0, 2, 1, 3}, {0, 1, 3, 2}};  // 1, (01), (12), (23)
  const int both[4] = {1, 0, 3, 2};                                                 // (01)(23)
  for (int cls = 0; cls < 6; ++cls) {
    const int* taus[4];
    int nt = 0;
    taus[nt++] = stab[0];
    if (cls == 1 || cls == 5) taus[nt++] = stab[1];
    if (cls == 2) taus[nt++] = stab[2];
    if (cls == 4 || cls == 5) taus[nt++] = stab[3];
    if (cls == 5) taus[nt++] = both;
    for (int q = 0; q < 24; ++q) {
      double c = 0.0;
      for (int t = 0; t < nt; ++t) {
        int st[4];
        for (int k = 0; k < 4; ++k) st[k] = QO_P[q][taus[t][k]];
        c += spin_class(st);
      }
      Q.c[cls][q] = c;
    }
  }
  hipLaunchKernelGGL(qo_energy_kernel, dim3((unsigned)((norb + 7) / 8 * 8), (unsigned)ntasks), dim3(QOB4), 0, s, X, Y,
                     VVOO, t2, eps, tasks, orbits, Q, o, v, (int)norb, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(qo_reduce_kernel, dim3((unsigned)ntasks), dim3(256), 0, s, part, norb, at, etask);
  return hipGetLastError();
}

}  // namespace cct
