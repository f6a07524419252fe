// Energies of the perturbative quadruples correction in the occupied-tuple
// order, from the accumulators that the segmented products of seg_gemm.hip
// leave.
#include <algorithm>
#include <climits>
#include <cmath>

#include "internal.h"

namespace cct {

namespace {

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
