// IBS distance and complete-linkage clustering (section "Identity-by-state
// matrices, complete linkage clustering": an IBS matrix followed by complete
// linkage clustering, timed in Table 2).
//
// Distance (reading; the paper names the statistic but not its formula): the
// proportion of alleles not shared identical by state over the jointly
// non-missing markers, d = (2 IBS0 + IBS1) / (2 N), +inf when N = 0 -- the
// correctly rounded quotient of two integers, so any implementation gets the
// same double.
//
// Clustering: while more than one cluster remains, merge the two clusters
// with the smallest complete-linkage distance (largest member-to-member
// distance); ties go to the smallest (a, b) pair of cluster indices, a
// cluster being indexed by its smallest sample.  Every decision compares
// doubles that are maxima of the input doubles, so the merge sequence is
// exactly determined.
//
// GPU plan: the working matrix D (m x m doubles) lives in the workspace.  From
// kClMinSlots to kClMaxSlots samples the merges run in rounds of mutually
// nearest pairs, in one cooperative launch (k_cl_rounds below).  Other cohorts, and calls
// that cannot launch it (cluster_rounds_ok), merge one pair at a time:
// for each active cluster k the cached nearest neighbour among l > k,
// nn[k] = argmin over (D[k][l], l), is kept; the globally closest pair is the
// argmin over k of (nn_d[k], k), which is exactly the lexicographic rule.
// Each of the m - 1 steps picks the pair (i, j), folds row and column
// j into i with max(), retires j, then rescans only the rows whose cached
// neighbour could have changed -- row i, rows k < i whose neighbour was i or
// j, and rows i < k < j whose neighbour was j (distances only grow, so no
// other row's minimum moves).  A retired cluster's column and cache entry
// hold NaN, which never wins a minimum, so scans need no activity flags.
// One block runs the steps below kClusterSplitMin samples, two launches per
// step above.
#include <mutex>

#include "pg_internal.h"

namespace pg {

__global__ __launch_bounds__(256) void k_ibs_distance(const uint32_t* __restrict__ i0,
                                                      const uint32_t* __restrict__ i1,
                                                      const uint32_t* __restrict__ nm,
                                                      int64_t count, double* __restrict__ d) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
       e += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t n = nm[e];
    d[e] = n ? __ddiv_rn((double)(2 * (int64_t)i0[e] + i1[e]), (double)(2 * (int64_t)n))
             : __longlong_as_double(0x7ff0000000000000ll);
  }
}

int launch_ibs_distance(const uint32_t* i0, const uint32_t* i1, const uint32_t* nm, int64_t count,
                        double* d, hipStream_t st) {
  if (count <= 0) return PG_OK;
  const int64_t blocks = ceil_div(count, 256) < 65536 ? ceil_div(count, 256) : 65536;
  hipLaunchKernelGGL(k_ibs_distance, dim3((unsigned)blocks), dim3(256), 0, st, i0, i1, nm, count,
                     d);
  return check_launch("ibs_distance");
}

// ---- IBS similarity and the IBD report ---------------------------------------
// Similarity (the --distance ibs value; reading): s = (2 IBS2 + IBS1) / (2 N),
// the correctly rounded quotient of two integers, NaN when N = 0.
__global__ __launch_bounds__(256) void k_ibs_similarity(const uint32_t* __restrict__ i1,
                                                        const uint32_t* __restrict__ i2,
                                                        const uint32_t* __restrict__ nm,
                                                        int64_t count, double* __restrict__ s) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
       e += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t n = nm[e];
    s[e] = n ? __ddiv_rn((double)(2 * (int64_t)i2[e] + i1[e]), (double)(2 * (int64_t)n))
             : __longlong_as_double(0x7ff8000000000000ll);
  }
}

int launch_ibs_similarity(const uint32_t* i1, const uint32_t* i2, const uint32_t* nm,
                          int64_t count, double* s, hipStream_t st) {
  if (count <= 0) return PG_OK;
  const int64_t blocks = ceil_div(count, 256) < 65536 ? ceil_div(count, 256) : 65536;
  hipLaunchKernelGGL(k_ibs_similarity, dim3((unsigned)blocks), dim3(256), 0, st, i1, i2, nm,
                     count, s);
  return check_launch("ibs_similarity");
}

// IBD report (reading; the paper times it but gives no formulas).  A marker
// whose observed alleles among the selected samples are x copies of A2 and y
// of A1 (n = x + y >= 4) expects, for two samples sharing no allele IBD (four
// alleles drawn without replacement from those n) or one (three drawn),
//   P(IBS0|IBD0) = 2 x(x-1) y(y-1) / n(n-1)(n-2)(n-3),
//   P(IBS1|IBD0) = 4 [x(x-1)(x-2) y + x y(y-1)(y-2)] / n(n-1)(n-2)(n-3),
//   P(IBS2|IBD0) = [x(x-1)(x-2)(x-3) + y(y-1)(y-2)(y-3) + 4 x(x-1) y(y-1)] / n(n-1)(n-2)(n-3),
//   P(IBS1|IBD1) = 2 [x(x-1) y + x y(y-1)] / n(n-1)(n-2),
//   P(IBS2|IBD1) = [x(x-1)(x-2) + y(y-1)(y-2) + x(x-1) y + x y(y-1)] / n(n-1)(n-2).
// These are averaged over the markers with n >= 4 (E00, E10, E20, E11, E21),
// and per pair the IBS0 and IBS1 moment equations give
//   Z0 = min(P0 / E00, 1),  Z1 = (P1 - Z0 E10) / E11 clamped to [0, 1 - Z0],
//   Z2 = (1 - Z0) - Z1,  PI_HAT = 0.5 Z1 + Z2,  with P0 = IBS0 / N, P1 = IBS1 / N.
// Every term is evaluated in IEEE double in the order written (explicit
// round-to-nearest operations, no contraction) and the averages are sums in
// increasing marker order, so the results are the same doubles any
// implementation of these formulas in that order gets.

// A marker's five terms from its {calls, A2 alleles}; whether it counts.
__device__ __forceinline__ bool genome_terms(uint2 c, double (&t)[5]) {
#pragma unroll
  for (int q = 0; q < 5; ++q) t[q] = 0.0;
  const int64_t calls = c.x, a2 = c.y;
  if (2 * calls < 4) return false;
  const double X = (double)a2, Y = (double)(2 * calls - a2), n = (double)(2 * calls);
  const double d4 = __dmul_rn(__dmul_rn(__dmul_rn(n, __dsub_rn(n, 1.0)), __dsub_rn(n, 2.0)),
                              __dsub_rn(n, 3.0));
  const double d3 = __dmul_rn(__dmul_rn(n, __dsub_rn(n, 1.0)), __dsub_rn(n, 2.0));
  const double x2 = __dmul_rn(X, __dsub_rn(X, 1.0)), y2 = __dmul_rn(Y, __dsub_rn(Y, 1.0));
  const double x3 = __dmul_rn(x2, __dsub_rn(X, 2.0)), y3 = __dmul_rn(y2, __dsub_rn(Y, 2.0));
  t[0] = __ddiv_rn(__dmul_rn(__dmul_rn(2.0, x2), y2), d4);
  t[1] = __ddiv_rn(__dmul_rn(4.0, __dadd_rn(__dmul_rn(x3, Y), __dmul_rn(X, y3))), d4);
  t[2] = __ddiv_rn(__dadd_rn(__dadd_rn(__dmul_rn(x3, __dsub_rn(X, 3.0)),
                                       __dmul_rn(y3, __dsub_rn(Y, 3.0))),
                             __dmul_rn(__dmul_rn(4.0, x2), y2)),
                   d4);
  t[3] = __ddiv_rn(__dmul_rn(2.0, __dadd_rn(__dmul_rn(x2, Y), __dmul_rn(X, y2))), d3);
  t[4] = __ddiv_rn(__dadd_rn(__dadd_rn(__dadd_rn(x3, y3), __dmul_rn(x2, Y)), __dmul_rn(X, y2)),
                   d3);
  return true;
}

// The five sums and the count K of markers that count, in two levels: each
// run of kSumRun consecutive markers is summed in increasing marker order
// from 0, then the runs' sums are added in increasing run order from 0.
// k_genome_run_sums: one block per run; all threads evaluate their markers'
// terms into LDS, then threads 0..4 each add their column in order; a marker
// that does not count, and the padding past the last marker, add +0.0, which
// leaves a non-negative sum unchanged.  It writes part[q * n_runs + r] (q < 5)
// and the run's count at q = 5.
constexpr int kSumRun = 1024;
__global__ __launch_bounds__(256) void k_genome_run_sums(const uint2* __restrict__ counts,
                                                         int64_t nv, int64_t n_runs,
                                                         double* __restrict__ part) {
  __shared__ double buf[5][kSumRun + 1];
  __shared__ unsigned int kcount;
  const int t = threadIdx.x;
  const int64_t r = blockIdx.x, c0 = r * kSumRun;
  const int64_t len = nv - c0 < kSumRun ? nv - c0 : kSumRun;
  if (t == 0) kcount = 0;
  uint2 c[kSumRun / 256];
#pragma unroll
  for (int u = 0; u < kSumRun / 256; ++u)
    c[u] = t + 256 * u < len ? counts[c0 + t + 256 * u] : make_uint2(0, 0);
  unsigned int K = 0;
#pragma unroll
  for (int u = 0; u < kSumRun / 256; ++u) {
    double v[5];
    K += genome_terms(c[u], v);
#pragma unroll
    for (int q = 0; q < 5; ++q) buf[q][t + 256 * u] = v[q];
  }
  __syncthreads();
  if (K) atomicAdd(&kcount, K);
  if (t < 5) {
    const double* col = buf[t];
    double S = 0.0;
    for (int j = 0; j < len; j += 32) {
      double b[32];
#pragma unroll
      for (int u = 0; u < 32; ++u) b[u] = col[j + u];
#pragma unroll
      for (int u = 0; u < 32; ++u) S = __dadd_rn(S, b[u]);
    }
    part[t * n_runs + r] = S;
  }
  __syncthreads();
  if (t == 0) part[5 * n_runs + r] = (double)kcount;
}

// out = {S00, S10, S20, S11, S21, K}: wave q adds the runs' sums of its column
// in run order, 64 loaded at a time and taken from their lanes; column 5 holds
// the counts (integers, exact).
__global__ __launch_bounds__(384) void k_genome_total(const double* __restrict__ part,
                                                      int64_t n_runs, double* __restrict__ out) {
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  double S = 0.0;
  for (int64_t r0 = 0; r0 < n_runs; r0 += 64) {
    const double p = r0 + lane < n_runs ? part[q * n_runs + r0 + lane] : 0.0;
    const int n = n_runs - r0 < 64 ? (int)(n_runs - r0) : 64;
    for (int u = 0; u < n; ++u) S = __dadd_rn(S, __shfl(p, u));
  }
  if (lane == 0) out[q] = S;
}

__global__ __launch_bounds__(256) void k_genome_pairs(const double* __restrict__ sums,
                                                      const uint32_t* __restrict__ i0,
                                                      const uint32_t* __restrict__ i1,
                                                      const uint32_t* __restrict__ nm,
                                                      int64_t count, double* __restrict__ z0,
                                                      double* __restrict__ z1,
                                                      double* __restrict__ z2,
                                                      double* __restrict__ pi) {
  const double K = sums[5];
  const double E00 = __ddiv_rn(sums[0], K), E10 = __ddiv_rn(sums[1], K);
  const double E11 = __ddiv_rn(sums[3], K);
  const bool ok = K > 0.0 && E00 != 0.0 && E11 != 0.0;
  const double nan = __longlong_as_double(0x7ff8000000000000ll);
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
       e += (int64_t)gridDim.x * blockDim.x) {
    if (!ok || nm[e] == 0) {
      z0[e] = z1[e] = z2[e] = pi[e] = nan;
      continue;
    }
    const double N = (double)nm[e];
    const double p0 = __ddiv_rn((double)i0[e], N), p1 = __ddiv_rn((double)i1[e], N);
    double a = __ddiv_rn(p0, E00);
    if (a > 1.0) a = 1.0;
    double b = __ddiv_rn(__dsub_rn(p1, __dmul_rn(a, E10)), E11);
    if (b < 0.0) b = 0.0;
    if (b > __dsub_rn(1.0, a)) b = __dsub_rn(1.0, a);
    const double c = __dsub_rn(__dsub_rn(1.0, a), b);
    z0[e] = a;
    z1[e] = b;
    z2[e] = c;
    pi[e] = __dadd_rn(__dmul_rn(0.5, b), c);
  }
}

int launch_genome(const uint2* counts, int64_t nv, double* sums, const uint32_t* i0,
                  const uint32_t* i1, const uint32_t* nm, int64_t count, double* z0, double* z1,
                  double* z2, double* pi, hipStream_t st) {
  const int64_t n_runs = genome_runs(nv);
  double* part = sums + 8;
  hipLaunchKernelGGL(k_genome_run_sums, dim3((unsigned)n_runs), dim3(256), 0, st, counts, nv,
                     n_runs, part);
  int rc = check_launch("genome_run_sums");
  if (rc != PG_OK) return rc;
  hipLaunchKernelGGL(k_genome_total, dim3(1), dim3(384), 0, st, part, n_runs, sums);
  rc = check_launch("genome_total");
  mark_stage(1, st);
  if (rc != PG_OK || count <= 0) return rc;
  const int64_t blocks = ceil_div(count, 256) < 65536 ? ceil_div(count, 256) : 65536;
  hipLaunchKernelGGL(k_genome_pairs, dim3((unsigned)blocks), dim3(256), 0, st, sums, i0, i1, nm,
                     count, z0, z1, z2, pi);
  return check_launch("genome_pairs");
}

// (value, index) minimum with the smaller index on equal values.
__device__ __forceinline__ void take_min(double& bv, int& bi, double v, int i) {
  if (v < bv || (v == bv && (unsigned)i < (unsigned)bi)) {
    bv = v;
    bi = i;
  }
}

__device__ __forceinline__ void wave_min(double& v, int& i) {
  for (int d = 32; d > 0; d >>= 1) {
    const double ov = __shfl_xor(v, d, 64);
    const int oi = __shfl_xor(i, d, 64);
    take_min(v, i, ov, oi);
  }
}

constexpr uint64_t kNaN = 0x7ff8000000000000ull;

__global__ __launch_bounds__(256) void k_nn_init(const double* __restrict__ D, int64_t m,
                                                 double* nn_d, int* nn_j) {
  const int lane = threadIdx.x & 63;
  for (int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; k < m;
       k += ((int64_t)gridDim.x * blockDim.x) >> 6) {
    double bv = __longlong_as_double(0x7ff0000000000000ll);
    int bi = -1;
    const double* row = D + k * m;
    for (int64_t l = k + 1 + lane; l < m; l += 64) take_min(bv, bi, row[l], (int)l);
    wave_min(bv, bi);
    if (lane == 0) {
      nn_d[k] = bi >= 0 ? bv : __longlong_as_double(kNaN);
      nn_j[k] = bi;
    }
  }
}

constexpr int kCT = 1024;
constexpr int kCW = kCT / 64;   // waves
constexpr int kCU = 4;          // loads in flight per thread in the argmin and the fold
constexpr int kCR = 8;          // loads in flight per thread in row rescans

__global__ __launch_bounds__(kCT) void k_cluster(double* __restrict__ D, int64_t m,
                                                 double* __restrict__ nn_d, int* __restrict__ nn_j,
                                                 pg_merge* __restrict__ merges) {
  __shared__ double s_v[kCW];
  __shared__ int s_i[kCW];
  __shared__ int s_rows[kCT];
  __shared__ int s_nrows;
  const double inf = __longlong_as_double(0x7ff0000000000000ll);
  const double nan = __longlong_as_double(kNaN);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int64_t t = 0; t + 1 < m; ++t) {
    // (a) the globally closest pair: argmin over k of (nn_d[k], k); retired
    // rows and rows without a neighbour hold NaN
    double bv = inf;
    int bi = -1;
    for (int64_t k0 = tid; k0 < m; k0 += kCT * kCU) {
      double v[kCU];
#pragma unroll
      for (int u = 0; u < kCU; ++u) v[u] = k0 + u * kCT < m ? nn_d[k0 + u * kCT] : nan;
#pragma unroll
      for (int u = 0; u < kCU; ++u) take_min(bv, bi, v[u], (int)(k0 + u * kCT));
    }
    wave_min(bv, bi);
    if (lane == 0) {
      s_v[wave] = bv;
      s_i[wave] = bi;
    }
    __syncthreads();
    double hv = s_v[0];
    int i = s_i[0];
    for (int w = 1; w < kCW; ++w) take_min(hv, i, s_v[w], s_i[w]);
    if (i < 0) break;   // unreachable: two active clusters always pair
    const int j = nn_j[i];
    if (tid == 0) {
      merges[t].a = i;
      merges[t].b = j;
      merges[t].height = hv;
      s_nrows = 0;
    }
    // (b) fold j into i: D[i][k] = D[k][i] = max(D[i][k], D[j][k]) for the
    // active k (a retired k has NaN in row i); retire j: its column and its
    // cache entry become NaN
    const double* ri = D + (int64_t)i * m;
    const double* rj = D + (int64_t)j * m;
    for (int64_t k0 = tid; k0 < m; k0 += kCT * kCU) {
      double a[kCU], b[kCU];
#pragma unroll
      for (int u = 0; u < kCU; ++u) {
        const int64_t k = k0 + u * kCT;
        a[u] = k < m ? ri[k] : nan;
        b[u] = k < m ? rj[k] : nan;
      }
#pragma unroll
      for (int u = 0; u < kCU; ++u) {
        const int64_t k = k0 + u * kCT;
        if (k >= m || k == j || a[u] != a[u]) continue;
        if (k != i) {
          const double v = a[u] > b[u] ? a[u] : b[u];
          D[(int64_t)i * m + k] = v;
          D[k * m + i] = v;
        }
        D[k * m + j] = nan;
      }
    }
    __syncthreads();
    if (tid == 0) nn_d[j] = nan;
    // (c) active rows (cache entry not NaN) whose neighbour may have moved
    for (int64_t k = tid; k < j; k += kCT) {
      const double dk = nn_d[k];
      if (dk != dk) continue;
      const int nk = nn_j[k];
      if (k == i || (k < i && (nk == i || nk == j)) || (k > i && nk == j)) {
        const int slot = atomicAdd(&s_nrows, 1);
        if (slot < kCT) s_rows[slot] = (int)k;
      }
    }
    __syncthreads();
    const int nrows = s_nrows;
    // (d) rescan them: groups of g waves per row, kCW / g rows at a time
    // (more rows than the list holds: walk every row below j, g = 1)
    const bool listed = nrows <= kCT;
    const int64_t nscan = listed ? nrows : j;
    int g = kCW;
    while (g > 1 && (int64_t)(kCW / g) < nscan) g >>= 1;
    const int groups = kCW / g, grp = wave / g, gt = tid - grp * g * 64;
    for (int64_t r0 = 0; r0 < nscan; r0 += groups) {
      const int64_t rr = r0 + grp;
      int k = -1;
      if (rr < nscan) {
        if (listed) {
          k = s_rows[rr];
        } else {
          const int kk = (int)rr;
          const double dk = nn_d[kk];
          const int nk = nn_j[kk];
          if (dk == dk && (kk == i || (kk < i && (nk == i || nk == j)) || (kk > i && nk == j)))
            k = kk;
        }
      }
      double v = inf;
      int l = -1;
      if (k >= 0) {
        const double* row = D + (int64_t)k * m;
        for (int64_t c0 = k + 1 + gt; c0 < m; c0 += (int64_t)g * 64 * kCR) {
          double x[kCR];
#pragma unroll
          for (int u = 0; u < kCR; ++u) {
            const int64_t c = c0 + (int64_t)u * g * 64;
            x[u] = c < m ? row[c] : nan;
          }
#pragma unroll
          for (int u = 0; u < kCR; ++u) take_min(v, l, x[u], (int)(c0 + (int64_t)u * g * 64));
        }
      }
      wave_min(v, l);
      __syncthreads();   // s_v / s_i free (their last readers are past here)
      if (lane == 0) {
        s_v[wave] = v;
        s_i[wave] = l;
      }
      __syncthreads();
      if (k >= 0 && gt == 0) {
        double rv = s_v[grp * g];
        int rl = s_i[grp * g];
        for (int w = 1; w < g; ++w) take_min(rv, rl, s_v[grp * g + w], s_i[grp * g + w]);
        nn_d[k] = rl >= 0 ? rv : nan;
        nn_j[k] = rl;
      }
    }
    __syncthreads();
  }
}

// ---- the merge loop as two launches per merge (large cohorts) ---------------
// The same steps as k_cluster, each spread over the chip.  k_cl_fold: every
// block finds the pair itself (the argmin over the cached neighbours, the
// same in every block; a block that already sees j retired by another block
// still finds i, since i != j), block 0 records the merge, and each thread
// folds sample k = its global index: j into i, j retired, and k appended to
// the list of rows to rescan when its neighbour may have moved.  k_cl_rescan
// (a block per listed row) rescans them.  The list's length for merge t is
// cnt[t % 2]; merge t clears cnt[(t + 1) % 2], whose last reader was merge
// t - 1's rescan, so the host only enqueues.
constexpr int kClT = 1024;
constexpr int kClScanBlocks = 64;

__global__ __launch_bounds__(kClT) void k_cl_fold(double* __restrict__ D, int64_t m,
                                                 double* __restrict__ nn_d,
                                                 const int* __restrict__ nn_j, int64_t t,
                                                 pg_merge* __restrict__ merges,
                                                 int* __restrict__ cnt, int* __restrict__ rows) {
  __shared__ double s_v[kClT / 64];
  __shared__ int s_i[kClT / 64];
  __shared__ int s_pair[2];
  const double inf = __longlong_as_double(0x7ff0000000000000ll);
  const double nan = __longlong_as_double(kNaN);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double bv = inf;
  int bi = -1;
  for (int64_t k0 = tid; k0 < m; k0 += kClT * kCU) {
    double v[kCU];
#pragma unroll
    for (int u = 0; u < kCU; ++u) v[u] = k0 + u * kClT < m ? nn_d[k0 + u * kClT] : nan;
#pragma unroll
    for (int u = 0; u < kCU; ++u) take_min(bv, bi, v[u], (int)(k0 + u * kClT));
  }
  wave_min(bv, bi);
  if (lane == 0) {
    s_v[wave] = bv;
    s_i[wave] = bi;
  }
  __syncthreads();
  if (tid == 0) {
    double hv = s_v[0];
    int pi = s_i[0];
    for (int w = 1; w < kClT / 64; ++w) take_min(hv, pi, s_v[w], s_i[w]);
    const int pj = pi >= 0 ? nn_j[pi] : -1;
    s_pair[0] = pi;
    s_pair[1] = pj;
    if (blockIdx.x == 0) {
      if (pi >= 0) {   // always: two active clusters always pair
        merges[t].a = pi;
        merges[t].b = pj;
        merges[t].height = hv;
      }
      cnt[(t + 1) & 1] = 0;
    }
  }
  __syncthreads();
  const int i = s_pair[0], j = s_pair[1];
  const int64_t k = (int64_t)blockIdx.x * kClT + tid;
  if (i < 0 || k >= m) return;
  // fold: D[i][k] = D[k][i] = max(D[i][k], D[j][k]) for the active k (a
  // retired k has NaN in row i); retire j: its column becomes NaN
  const double a = D[(int64_t)i * m + k];
  if (k != j && a == a) {
    if (k != i) {
      const double b = D[(int64_t)j * m + k];
      const double v = a > b ? a : b;
      D[(int64_t)i * m + k] = v;
      D[k * m + i] = v;
    }
    D[k * m + j] = nan;
  }
  if (k == j) nn_d[j] = nan;
  // active rows below j whose cached neighbour may have moved (their cache
  // entries are not touched by this kernel, except j's, which is not listed)
  if (k < j) {
    const double dk = nn_d[k];
    const int nk = nn_j[k];
    if (dk == dk && (k == i || (k < i && (nk == i || nk == j)) || (k > i && nk == j)))
      rows[atomicAdd(&cnt[t & 1], 1)] = (int)k;
  }
}

__global__ __launch_bounds__(kClT) void k_cl_rescan(const double* __restrict__ D, int64_t m,
                                                    double* __restrict__ nn_d,
                                                    int* __restrict__ nn_j, int64_t t,
                                                    const int* __restrict__ cnt,
                                                    const int* __restrict__ rows) {
  __shared__ double s_v[kClT / 64];
  __shared__ int s_i[kClT / 64];
  const int nrows = cnt[t & 1];
  const double inf = __longlong_as_double(0x7ff0000000000000ll);
  const double nan = __longlong_as_double(kNaN);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int r = blockIdx.x; r < nrows; r += gridDim.x) {   // block-uniform
    const int64_t k = rows[r];
    const double* row = D + k * m;
    double v = inf;
    int l = -1;
    for (int64_t c0 = k + 1 + tid; c0 < m; c0 += (int64_t)kClT * kCR) {
      double x[kCR];
#pragma unroll
      for (int u = 0; u < kCR; ++u) {
        const int64_t c = c0 + (int64_t)u * kClT;
        x[u] = c < m ? row[c] : nan;
      }
#pragma unroll
      for (int u = 0; u < kCR; ++u) take_min(v, l, x[u], (int)(c0 + (int64_t)u * kClT));
    }
    wave_min(v, l);
    __syncthreads();   // s_v / s_i free (the previous row's reader is done)
    if (lane == 0) {
      s_v[wave] = v;
      s_i[wave] = l;
    }
    __syncthreads();
    if (tid == 0) {
      double rv = s_v[0];
      int rl = s_i[0];
      for (int w = 1; w < kClT / 64; ++w) take_min(rv, rl, s_v[w], s_i[w]);
      nn_d[k] = rl >= 0 ? rv : nan;
      nn_j[k] = rl;
    }
  }
}

// ---- the merge loop in rounds (one cooperative launch) ------------------------
// Order cluster pairs by (distance, a, b): a strict total order, and the merge
// of the sequential rule is always its minimum.  A pair that is mutually
// nearest in that order stays so until it merges: a merge elsewhere leaves
// the labels of the pairs around it and only raises their distances.  And the
// pairs the sequential rule merges come in increasing order, since a merged
// cluster's pairs are no smaller than the pairs they replace.  So every
// mutually nearest pair of a round can merge at once, and the sequence is the
// list of all merges sorted by (height, a, b) (reciprocal nearest neighbours, a
// known form of agglomerative clustering).  47 rounds for 1,000 samples of
// independent variants, 77 for 10,000 of a founder mosaic, each merging 5-20% of
// the clusters.
//
// Active clusters occupy slots in increasing label, so the nearest neighbour
// of slot k is argmin over l of (d, l).  A round, in every block alike:
//   1. the neighbours of all slots go to LDS; slot k merges with l = nn[k]
//      when nn[l] = k.  The wave that writes a pair's row records the merge,
//      block 0 the last one;
//   2. with at least 1 pair per kClFew slots (or a quarter of the slots
//      retired) the matrix is rebuilt without the retired slots into the
//      other buffer: entry (i, j) is the maximum over the members of both
//      slots, and the wave that writes a row finds its neighbour on the way.
//      The matrix shrinks with the clusters, so all rounds together move
//      about twelve times the first matrix;
//   3. with fewer pairs, the rows and columns of the pairs are folded in place
//      (a retired slot's column becomes NaN, which never wins a minimum) and
//      only rows whose neighbour moved are scanned again.
// Bound: HBM while the matrix is large, then the grid barrier per round.  Every
// block is resident (cooperative launch), so the barriers end.  A round has a
// pair on a symmetric matrix; on another one, where the nearest neighbours may
// form a cycle, the slot with the smallest distance merges with its neighbour,
// so that every call writes m - 1 merges.
//
// Measured: 10,000 samples 155 -> 3.7 ms (0.4 ms of it the distances), 1,000
// samples 7.6 -> 0.43 ms (47 rounds of about 8 us).  What it costs where a round
// finds one pair: equal distances, 6,000 samples 73 -> 93 to 96 ms, 1,000 samples
// 7.8 ms either way.
constexpr int kClMaxSlots = 24576;   // 6 bytes of LDS per slot
// Below, the one block's loop is as fast as the rounds' three launches (us a
// call, loop / rounds: 2 samples 23 / 42, 5 41 / 56, 10 72 / 66, 20 129 / 105).
constexpr int kClMinSlots = 10;
constexpr int kClFew = 32;
constexpr int kClWaves = kClT / 64;
constexpr unsigned kClNone = 0xFFFFu;
constexpr int kClU = 4;              // columns in flight per lane in the rebuild
constexpr int kClPerBlock = 8;       // slots per block at least
constexpr int kClRows = 32;          // rows between two reductions of a block
constexpr int kClBarWords = 32 * 17; // grid barrier: a 128-byte line per word

struct ClRounds {
  double* D[2];        // slots x ld, ping-pong
  double* nn_d[2];
  int* nn_j[2];        // -1: retired
  int* lab[2];         // smallest sample of the slot's cluster
  pg_merge* found;     // found[b - 1]: the merge that retires label b
  unsigned* bar;       // kClBarWords words, 0 at launch
  int m;
};

// Barrier over the blocks [0, nb): all earlier writes of each are visible to
// all of them afterwards.  Arrivals count in eight words (one per XCD, as
// blocks are dealt round robin) and then in one, since 256 additions to one
// word take 10 us; the last one raises the epoch that the others wait for.
// Every wave waits for its own stores to be in L2 before the block's barrier
// (which waits for LDS only), so that the write-back of the one wave that
// signals the arrival covers them all.  A write-back by every wave costs more:
// 10,000 samples 3.7 -> 5.4 ms, equal distances of 6,000 96 -> 278 ms.
// nb may only fall from one barrier to the next.
struct ClBarrier {
  unsigned* bar;
  unsigned group_target, root_target, epoch;
  __device__ __forceinline__ void wait(unsigned nb) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (nb > 1) {
      const unsigned g = blockIdx.x & 7u;
      group_target += (nb - g + 7u) >> 3;
      root_target += nb < 8u ? nb : 8u;
      ++epoch;
      if (threadIdx.x == 0) {
        unsigned* flag = bar + 32 * 9;
        if (__hip_atomic_fetch_add(bar + 32 * g, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) +
                1u == group_target &&
            __hip_atomic_fetch_add(bar + 32 * 8, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) +
                1u == root_target)
          __hip_atomic_store(flag, epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < epoch)
          __builtin_amdgcn_s_sleep(1);
        __threadfence();
      }
    }
    __syncthreads();
  }
};

__device__ __forceinline__ double cl_max(double a, double b) { return a > b ? a : b; }

template <typename T>
__device__ __forceinline__ void cl_swap(T& a, T& b) {
  const T t = a;
  a = b;
  b = t;
}

// Argmin over the active columns of a row by one wave.
__device__ __forceinline__ void cl_scan_row(const double* row, int A, int lane, double& v,
                                            int& l) {
  const double nan = __longlong_as_double(kNaN);
  for (int c0 = lane; c0 < A; c0 += 64 * kCR) {
    double x[kCR];
#pragma unroll
    for (int u = 0; u < kCR; ++u) x[u] = c0 + 64 * u < A ? row[c0 + 64 * u] : nan;
#pragma unroll
    for (int u = 0; u < kCR; ++u) take_min(v, l, x[u], c0 + 64 * u);
  }
  wave_min(v, l);
}

__global__ __launch_bounds__(kClT) void k_cl_rounds(ClRounds p) {
  __shared__ uint16_t s_nn[kClMaxSlots];
  __shared__ uint32_t s_map[kClMaxSlots];   // k | l << 16 (kClNone: no second member)
  __shared__ double s_pv[kClRows][kClWaves];
  __shared__ int s_pi[kClRows][kClWaves];
  __shared__ int s_cnt[2][kClWaves];
  const double inf = __longlong_as_double(0x7ff0000000000000ll);
  const double nan = __longlong_as_double(kNaN);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = ((uint64_t)1 << lane) - 1;
  ClBarrier bar{p.bar, 0u, 0u, 0u};
  unsigned nb = gridDim.x;
  int A = p.m, active = p.m;   // slots, clusters
  double *D = p.D[0], *D2 = p.D[1], *nn_d = p.nn_d[0], *nn_d2 = p.nn_d[1];
  int *nn_j = p.nn_j[0], *nn_j2 = p.nn_j[1], *lab = p.lab[0], *lab2 = p.lab[1];
  while (active > 1) {
    const int64_t ld = (A + 15) & ~15;
    for (int k0 = tid; k0 < A; k0 += kClT * kCR) {
      int l[kCR];
#pragma unroll
      for (int u = 0; u < kCR; ++u) l[u] = k0 + u * kClT < A ? nn_j[k0 + u * kClT] : 0;
#pragma unroll
      for (int u = 0; u < kCR; ++u)
        if (k0 + u * kClT < A) s_nn[k0 + u * kClT] = (uint16_t)l[u];
    }
    __syncthreads();
    // survivors and pairs of this wave's run of slots, then their places
    const int run = ((A + kClT - 1) / kClT) * 64;
    const int r0 = wave * run, r1 = r0 + run < A ? r0 + run : A;
    int n_live, n_pairs, live_at, pair_at;
    for (;;) {
      int live = 0, pairs = 0;
      for (int k = r0 + lane; k - lane < r1; k += 64) {
        const unsigned l = k < r1 ? s_nn[k] : kClNone;
        const bool on = l != kClNone;
        const bool merge = on && s_nn[on ? l : 0] == (unsigned)k;
        live += __popcll(__ballot(on && !(merge && l < (unsigned)k)));
        pairs += __popcll(__ballot(merge && l > (unsigned)k));
      }
      if (lane == 0) {
        s_cnt[0][wave] = live;
        s_cnt[1][wave] = pairs;
      }
      __syncthreads();
      n_live = n_pairs = live_at = pair_at = 0;
      for (int w = 0; w < kClWaves; ++w) {
        if (w < wave) {
          live_at += s_cnt[0][w];
          pair_at += s_cnt[1][w];
        }
        n_live += s_cnt[0][w];
        n_pairs += s_cnt[1][w];
      }
      if (n_pairs > 0) break;
      // asymmetric counts: the slot nearest to another merges with it
      double v = inf;
      int k = -1;
      for (int x = tid; x < A; x += kClT)
        if (s_nn[x] != kClNone) take_min(v, k, nn_d[x], x);
      wave_min(v, k);
      if (lane == 0) {
        s_pv[0][wave] = v;
        s_pi[0][wave] = k;
      }
      __syncthreads();
      if (tid == 0) {
        for (int w = 1; w < kClWaves; ++w) take_min(v, k, s_pv[0][w], s_pi[0][w]);
        s_nn[s_nn[k]] = (uint16_t)k;
      }
      __syncthreads();
    }
    const bool rebuild = n_pairs * kClFew >= A || n_live * 4 <= A * 3;
    for (int k = r0 + lane; k - lane < r1; k += 64) {
      const unsigned l = k < r1 ? s_nn[k] : kClNone;
      const bool on = l != kClNone;
      const bool merge = on && s_nn[on ? l : 0] == (unsigned)k;
      const bool stays = on && !(merge && l < (unsigned)k), first = merge && l > (unsigned)k;
      const uint64_t bl = __ballot(stays), bp = __ballot(first);
      if (rebuild && stays)
        s_map[live_at + __popcll(bl & below)] = (unsigned)k | (merge ? l : kClNone) << 16;
      if (!rebuild && first) s_map[pair_at + __popcll(bp & below)] = (unsigned)k | l << 16;
      live_at += __popcll(bl);
      pair_at += __popcll(bp);
      if (n_live == 1 && blockIdx.x == 0 && first)   // the last merge
        p.found[lab[l] - 1] = pg_merge{lab[k], lab[l], nn_d[k]};
    }
    __syncthreads();
    active = n_live;
    if (active <= 1) break;
    if (rebuild) {
      const int64_t ld2 = (n_live + 15) & ~15;
      // wpr waves share a row, the number that gives the fewest trips times
      // column steps (half a step more for each trip's reduction)
      int wpr = 1, least = 0x7fffffff;
      for (int w = 1; w <= kClWaves; w <<= 1) {
        const int rows = (int)nb * (kClWaves / w), cols = 64 * kClU * w;
        const int cost = ((n_live + rows - 1) / rows) * (2 * ((n_live + cols - 1) / cols) + 1);
        if (cost < least) {
          least = cost;
          wpr = w;
        }
      }
      const int rpb = kClWaves / wpr, grp = wave / wpr, sub = wave % wpr;
      const int step = (int)nb * rpb, batch = kClRows / rpb;
      const int trips = (n_live + step - 1) / step;
      for (int t0 = 0; t0 < trips; t0 += batch) {
        const int t1 = t0 + batch < trips ? t0 + batch : trips;
        for (int t = t0; t < t1; ++t) {
          const int i = t * step + grp * (int)nb + (int)blockIdx.x;
          double v = inf;
          int at = -1;
          if (i < n_live) {
            const uint32_t me = s_map[i];
            const bool two = (me >> 16) != kClNone;
            const double* a0 = D + (int64_t)(me & 0xFFFFu) * ld;
            const double* a1 = two ? D + (int64_t)(me >> 16) * ld : a0;
            double* out = D2 + (int64_t)i * ld2;
            for (int c0 = sub * 64 + lane; c0 < n_live; c0 += 64 * wpr * kClU) {
              double x[kClU], y[kClU];
              uint32_t mp[kClU];
#pragma unroll
              for (int u = 0; u < kClU; ++u) {
                const int c = c0 + 64 * wpr * u;
                mp[u] = c < n_live ? s_map[c] : kClNone << 16;
                x[u] = c < n_live ? a0[mp[u] & 0xFFFFu] : nan;
              }
#pragma unroll
              for (int u = 0; u < kClU; ++u) {
                y[u] = -inf;
                if ((mp[u] >> 16) != kClNone) y[u] = a0[mp[u] >> 16];
              }
              if (two) {
                double z[kClU], w[kClU];
#pragma unroll
                for (int u = 0; u < kClU; ++u) {
                  z[u] = c0 + 64 * wpr * u < n_live ? a1[mp[u] & 0xFFFFu] : nan;
                  w[u] = -inf;
                  if ((mp[u] >> 16) != kClNone) w[u] = a1[mp[u] >> 16];
                }
#pragma unroll
                for (int u = 0; u < kClU; ++u) x[u] = cl_max(cl_max(x[u], z[u]), w[u]);
              }
#pragma unroll
              for (int u = 0; u < kClU; ++u) {
                const int c = c0 + 64 * wpr * u;
                x[u] = c == i ? nan : cl_max(x[u], y[u]);
                if (c < n_live) {
                  out[c] = x[u];
                  take_min(v, at, x[u], c);
                }
              }
            }
          }
          wave_min(v, at);
          if (lane == 0) {
            s_pv[(t - t0) * rpb + grp][sub] = v;
            s_pi[(t - t0) * rpb + grp][sub] = at;
          }
        }
        __syncthreads();
        if (tid < (t1 - t0) * rpb) {
          const int i = (t0 + tid / rpb) * step + (tid % rpb) * (int)nb + (int)blockIdx.x;
          if (i < n_live) {
            double v = s_pv[tid][0];
            int at = s_pi[tid][0];
            for (int w = 1; w < wpr; ++w) take_min(v, at, s_pv[tid][w], s_pi[tid][w]);
            nn_d2[i] = v;
            nn_j2[i] = at;
            const int k = s_map[i] & 0xFFFFu, l = s_map[i] >> 16, a = lab[k];
            lab2[i] = a;
            if (l != (int)kClNone) p.found[lab[l] - 1] = pg_merge{a, lab[l], nn_d[k]};
          }
        }
        __syncthreads();
      }
      cl_swap(D, D2);
      cl_swap(nn_d, nn_d2);
      cl_swap(nn_j, nn_j2);
      cl_swap(lab, lab2);
      A = n_live;
    } else {
      // the pairs' rows, a block each: the maximum over the members of the
      // row's slot and of the column's (the lane of a column pair's first
      // slot writes both; row l is not written by anyone)
      for (int q = blockIdx.x; q < n_pairs; q += nb) {
        const int k = s_map[q] & 0xFFFFu, l = s_map[q] >> 16;
        double* a0 = D + (int64_t)k * ld;
        const double* a1 = D + (int64_t)l * ld;
        double v = inf;
        int at = -1;
        for (int c0 = tid; c0 < A; c0 += kClT * kClU) {
          double x[kClU], y[kClU];
#pragma unroll
          for (int u = 0; u < kClU; ++u) {
            const int c = c0 + u * kClT;
            x[u] = c < A ? a0[c] : nan;
            y[u] = c < A ? a1[c] : nan;
          }
#pragma unroll
          for (int u = 0; u < kClU; ++u) {
            const int c = c0 + u * kClT;
            const unsigned nc = c < A ? s_nn[c] : kClNone;
            if (nc == kClNone) continue;
            const bool merge = s_nn[nc] == (unsigned)c;
            if (merge && nc < (unsigned)c) continue;
            x[u] = cl_max(x[u], y[u]);
            if (merge) {
              x[u] = cl_max(x[u], cl_max(a0[nc], a1[nc]));
              a0[nc] = nan;
            }
            if (c == k) continue;
            a0[c] = x[u];
            take_min(v, at, x[u], c);
          }
        }
        wave_min(v, at);
        __syncthreads();   // s_pv, s_pi free
        if (lane == 0) {
          s_pv[0][wave] = v;
          s_pi[0][wave] = at;
        }
        __syncthreads();
        if (tid == 0) {
          for (int w = 1; w < kClWaves; ++w) take_min(v, at, s_pv[0][w], s_pi[0][w]);
          p.found[lab[l] - 1] = pg_merge{lab[k], lab[l], nn_d[k]};
          nn_d2[k] = v;
          nn_j2[k] = at;
          nn_j2[l] = -1;
        }
      }
      // the pairs' columns in the other rows, a wave each; a row is scanned
      // again when its neighbour retired, or merged and moved away.  Every
      // neighbour goes to the other buffer: a slower block may still be
      // reading this round's
      for (int x = wave * (int)nb + (int)blockIdx.x; x < A; x += (int)nb * kClWaves) {
        const unsigned nx = s_nn[x];
        if (nx == kClNone) {
          if (lane == 0) nn_j2[x] = -1;
          continue;
        }
        if (s_nn[nx] == (unsigned)x) continue;
        double* row = D + (int64_t)x * ld;
        const double near = nn_d[x];
        bool moved = false;
        for (int q = lane; q < n_pairs; q += 64) {
          const int k = s_map[q] & 0xFFFFu, l = s_map[q] >> 16;
          const double y = cl_max(row[k], row[l]);
          row[k] = y;
          row[l] = nan;
          moved |= l == (int)nx || (k == (int)nx && y > near);
        }
        double v = near;
        int at = (int)nx;
        if (__any(moved)) {
          __threadfence_block();   // the other lanes' columns
          v = inf;
          at = -1;
          cl_scan_row(row, A, lane, v, at);
        }
        if (lane == 0) {
          nn_d2[x] = v;
          nn_j2[x] = at;
        }
      }
      cl_swap(nn_d, nn_d2);
      cl_swap(nn_j, nn_j2);
    }
    bar.wait(nb);
    // one block per kClPerBlock slots is enough; the others are done
    const unsigned need = (unsigned)((A + kClPerBlock - 1) / kClPerBlock);
    if (need < nb) nb = need;
    if (blockIdx.x >= nb) return;
  }
}

// The merges in increasing (height, a, b): each finds its place by counting
// the smaller ones (all differ in b).  64 merges per block, each counted by 16
// threads over a sixteenth of the others.
__global__ __launch_bounds__(1024) void k_cl_order(const pg_merge* __restrict__ found, int n,
                                                   pg_merge* __restrict__ merges) {
  __shared__ pg_merge s[1024];
  __shared__ int s_place[64];
  const int tid = threadIdx.x, slice = tid >> 6, e = blockIdx.x * 64 + (tid & 63);
  pg_merge me{};
  if (e < n) me = found[e];
  if (tid < 64) s_place[tid] = 0;
  int place = 0;
  for (int c0 = 0; c0 < n; c0 += 1024) {
    __syncthreads();
    if (c0 + tid < n) s[tid] = found[c0 + tid];
    __syncthreads();
    const int end = n - c0 < slice * 64 + 64 ? n - c0 : slice * 64 + 64;
    for (int q = slice * 64; q < end; ++q) {
      const pg_merge o = s[q];
      place += o.height < me.height ||
               (o.height == me.height && (o.a < me.a || (o.a == me.a && o.b < me.b)));
    }
  }
  atomicAdd(&s_place[tid & 63], place);
  __syncthreads();
  if (tid < 64 && e < n) merges[s_place[tid]] = me;
}

// Distances, and each sample's nearest neighbour: a block per row.
__global__ __launch_bounds__(256) void k_cl_start(const uint32_t* __restrict__ i0,
                                                  const uint32_t* __restrict__ i1,
                                                  const uint32_t* __restrict__ nm, ClRounds p) {
  __shared__ double s_v[4];
  __shared__ int s_i[4];
  const int m = p.m, k = blockIdx.x, tid = threadIdx.x;
  const int64_t at = (int64_t)k * m, ld = (m + 15) & ~15;
  const double inf = __longlong_as_double(0x7ff0000000000000ll);
  if (k == 0)
    for (int w = tid; w < kClBarWords; w += 256) p.bar[w] = 0u;
  double v = inf;
  int l = -1;
  for (int c0 = tid; c0 < m; c0 += 256 * kCU) {
    uint32_t a[kCU], b[kCU], n[kCU];
#pragma unroll
    for (int u = 0; u < kCU; ++u) {
      const int64_t c = at + (c0 + 256 * u < m ? c0 + 256 * u : k);
      a[u] = i0[c];
      b[u] = i1[c];
      n[u] = nm[c];
    }
#pragma unroll
    for (int u = 0; u < kCU; ++u) {
      const int c = c0 + 256 * u;
      if (c >= m) continue;
      double d = n[u] ? __ddiv_rn((double)(2 * (int64_t)a[u] + b[u]),
                                  (double)(2 * (int64_t)n[u]))
                      : inf;
      if (c == k) d = __longlong_as_double(kNaN);
      p.D[0][k * ld + c] = d;
      take_min(v, l, d, c);
    }
  }
  wave_min(v, l);
  if ((tid & 63) == 0) {
    s_v[tid >> 6] = v;
    s_i[tid >> 6] = l;
  }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 4; ++w) take_min(v, l, s_v[w], s_i[w]);
    p.nn_d[0][k] = v;
    p.nn_j[0][k] = l;
    p.lab[0][k] = k;
  }
}

int64_t cluster_rounds_bytes(int64_t m) {
  if (m > kClMaxSlots) return 0;
  const int64_t ld = round_up(m, 16);
  return 2 * m * ld * 8 + 2 * round_up(m, 32) * (8 + 4 + 4) + round_up(m, 32) * 16 +
         kClBarWords * 4;
}

// Whether the rounds can run and pay: the slots fit, the stream is not capturing (a
// captured call takes the launches per merge, plain kernel nodes) and has the
// whole chip (no CU mask), and the device launches cooperatively and holds a
// block per CU.  `blocks`: one per CU, or one per kClPerBlock rows.
static bool cluster_rounds_ok(int64_t m, hipStream_t st, unsigned& blocks) {
  if (m < kClMinSlots || m > kClMaxSlots) return false;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  int dev = 0, coop = 0, cus = 0, resident = 0;
  if (hipStreamIsCapturing(st, &cap) != hipSuccess || hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &resident, reinterpret_cast<const void*>(k_cl_rounds), kClT, 0) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (cap != hipStreamCaptureStatusNone || dev < 0 || dev >= kMaxDevices || !coop || cus < 1 ||
      resident < 1)
    return false;
  uint32_t mask[32] = {};
  if (hipExtStreamGetCUMask(st, 32, mask) == hipSuccess) {
    int on = 0;
    for (uint32_t w : mask) on += __builtin_popcount(w);
    if (on < cus) return false;
  } else {
    (void)hipGetLastError();
  }
  blocks = (unsigned)(ceil_div(m, kClPerBlock) < cus ? ceil_div(m, kClPerBlock) : cus);
  return true;
}

// The last launch of the rounds on each device, kept until the process ends.
// The grid barriers need every block resident, so a launch waits for the one
// before it, whatever their streams, beside the cooperative launch's own
// check that the grid fits.
static std::mutex g_rounds_mu;
static hipEvent_t g_rounds_done[kMaxDevices] = {};

// `launched`: whether the device took the grid; if not, nothing ran.
static int launch_rounds_kernel(ClRounds& p, unsigned blocks, hipStream_t st, bool& launched) {
  std::lock_guard<std::mutex> lock(g_rounds_mu);
  launched = false;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess && !g_rounds_done[dev])
    e = hipEventCreateWithFlags(&g_rounds_done[dev], hipEventDisableTiming);
  if (e == hipSuccess) e = hipStreamWaitEvent(st, g_rounds_done[dev], 0);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return fail(PG_EDEVICE, "cluster_rounds: %s", hipGetErrorString(e));
  }
  void* args[] = {&p};
  if (hipLaunchCooperativeKernel(reinterpret_cast<const void*>(k_cl_rounds), dim3(blocks),
                                 dim3(kClT), args, 0, st) != hipSuccess) {
    (void)hipGetLastError();
    return PG_OK;
  }
  launched = true;
  e = hipEventRecord(g_rounds_done[dev], st);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return fail(PG_EDEVICE, "cluster_rounds: %s", hipGetErrorString(e));
  }
  return PG_OK;
}

// `done` false: the rounds did not run, and the merges are still to be made.
static int launch_cluster_rounds(const uint32_t* i0, const uint32_t* i1, const uint32_t* nm,
                                 int64_t m, char* ws, unsigned blocks, pg_merge* merges,
                                 hipStream_t st, bool& done) {
  done = true;
  const int64_t ld = round_up(m, 16), mp = round_up(m, 32);
  ClRounds p;
  char* at = ws;
  for (int b = 0; b < 2; ++b, at += m * ld * 8) p.D[b] = (double*)at;
  for (int b = 0; b < 2; ++b, at += mp * 8) p.nn_d[b] = (double*)at;
  for (int b = 0; b < 2; ++b, at += mp * 4) p.nn_j[b] = (int*)at;
  for (int b = 0; b < 2; ++b, at += mp * 4) p.lab[b] = (int*)at;
  p.found = (pg_merge*)at;
  at += mp * 16;
  p.bar = (unsigned*)at;
  p.m = (int)m;
  hipLaunchKernelGGL(k_cl_start, dim3((unsigned)m), dim3(256), 0, st, i0, i1, nm, p);
  int rc = check_launch("cluster_start");
  mark_stage(1, st);
  if (rc != PG_OK || m < 2) return rc;
  rc = launch_rounds_kernel(p, blocks, st, done);
  if (rc != PG_OK || !done) return rc;
  hipLaunchKernelGGL(k_cl_order, dim3((unsigned)ceil_div(m - 1, 64)), dim3(1024), 0, st, p.found,
                     (int)(m - 1), merges);
  rc = check_launch("cluster_order");
  mark_stage(2, st);
  return rc;
}

int launch_ibs_cluster(const uint32_t* i0, const uint32_t* i1, const uint32_t* nm, int64_t m,
                       double* D, double* nn_d, int* nn_j, int* ctl, int* rows,
                       pg_merge* merges, hipStream_t st) {
  unsigned round_blocks;
  if (cluster_rounds_ok(m, st, round_blocks)) {
    bool done;
    const int rc = launch_cluster_rounds(i0, i1, nm, m, reinterpret_cast<char*>(D), round_blocks,
                                         merges, st, done);
    if (rc != PG_OK || done) return rc;
  }
  int rc = launch_ibs_distance(i0, i1, nm, m * m, D, st);
  if (rc != PG_OK) return rc;
  const int64_t blocks = ceil_div(m, 4) < 65536 ? ceil_div(m, 4) : 65536;
  hipLaunchKernelGGL(k_nn_init, dim3((unsigned)blocks), dim3(256), 0, st, D, m, nn_d, nn_j);
  rc = check_launch("cluster_init");
  mark_stage(1, st);
  if (rc != PG_OK || m < 2) return rc;
  if (m < kClusterSplitMin) {
    hipLaunchKernelGGL(k_cluster, dim3(1), dim3(kCT), 0, st, D, m, nn_d, nn_j, merges);
    rc = check_launch("cluster");
  } else {
    const unsigned fold_blocks = (unsigned)ceil_div(m, kClT);
    rc = fill_u32(reinterpret_cast<uint32_t*>(ctl), 2, 0u, st);   // the two list lengths
    for (int64_t t = 0; t + 1 < m && rc == PG_OK; ++t) {
      hipLaunchKernelGGL(k_cl_fold, dim3(fold_blocks), dim3(kClT), 0, st, D, m, nn_d, nn_j, t,
                         merges, ctl, rows);
      hipLaunchKernelGGL(k_cl_rescan, dim3(kClScanBlocks), dim3(kClT), 0, st, D, m, nn_d, nn_j, t,
                         ctl, rows);
      rc = check_launch("cluster_step");
    }
  }
  mark_stage(2, st);
  return rc;
}

}  // namespace pg
