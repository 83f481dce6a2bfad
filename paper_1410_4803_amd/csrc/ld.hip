// Linkage-disequilibrium window kernels (section "Bit population count").
//
// For variants a < b <= a + window, with x = -1 / 0 / +1 for homozygous A1 /
// heterozygous / homozygous A2, the six sums over the samples where neither
// call is missing are six contractions over samples of per-call int8
// features (all zero for a missing call): m = 1, x, h = x^2:
//   n = <m_a, m_b>, Sx = <x_a, m_b>, Sy = <m_a, x_b>, Sxx = <h_a, m_b>,
//   Syy = <m_a, h_b>, Sxy = <x_a, x_b>.
// The main kernel runs these on the int8 matrix cores over a band of 64x64
// variant tiles and, per pair, evaluates r^2 and the emission test.  Emitted
// pairs are marked in a per-row bitmap and counted per row (atomic OR / add:
// the result does not depend on their order).  A scan turns row counts into
// offsets, and the emit kernel writes each marked pair at its offset in (a, b)
// order, recomputing its sums with popcounts over the same 2-bit words -- an
// independent integer route to the same exact values.
#include "tiles.h"

namespace pg {

// The emission scratch: bitmap words, then row counts.
__global__ void k_ld_clear(LdScratch sc, int64_t n_bits, int64_t n_rows) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_bits) sc.bitmap[i] = 0u;
  else if (i - n_bits < n_rows) sc.rowcnt[i - n_bits] = 0u;
}

__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

int fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t st) {
  if (n <= 0) return PG_OK;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, p, n, v);
  return check_launch("fill");
}

int ld_clear(const LdScratch& sc, int64_t rows_pad, hipStream_t st) {
  const int64_t n_bits = rows_pad * sc.bm_words;
  hipLaunchKernelGGL(k_ld_clear, dim3((unsigned)ceil_div(n_bits + rows_pad, 256)), dim3(256), 0,
                     st, sc, n_bits, rows_pad);
  return check_launch("ld_clear");
}

__global__ __launch_bounds__(256) void k_ld_popc(const uint32_t* __restrict__ P, int64_t words_pad,
                                                 int64_t nv, int64_t rows_pad, int64_t n_band,
                                                 int32_t window, double r2_min, LdScratch sc) {
  const int64_t b = xcd_swizzle(blockIdx.x, gridDim.x);
  const int64_t I = b / n_band;
  const int64_t J = I + b % n_band;
  if (J >= rows_pad / kLP) return;
  __shared__ __attribute__((aligned(16))) uint32_t smem[kLdPopcSmem];
  ld_popc_tile(P, words_pad, nv, rows_pad, I, J, window, r2_min, sc, (lds_t*)smem);
}

int launch_ld_popc(const uint32_t* P, int64_t words_pad, int64_t nv, int64_t rows_pad,
                   int32_t window, double r2_min, const LdScratch& sc, hipStream_t st) {
  const int64_t n_band = ((int64_t)window + kLP - 1) / kLP + 1;
  const int64_t blocks = rows_pad / kLP * n_band;
  hipLaunchKernelGGL(k_ld_popc, dim3((unsigned)blocks), dim3(256), 0, st, P, words_pad, nv,
                     rows_pad, n_band, window, r2_min, sc);
  int rc = check_launch("ld_popc");
  mark_stage(2, st);
  return rc;
}

constexpr int kLdTileNib = 0, kLdTileFp4 = 1, kLdTileInt8 = 2;

template <int kTile>
__global__ __launch_bounds__(256, 2) void k_ld_mfma(const uint32_t* __restrict__ D, int64_t wn,
                                                    int64_t nv, int64_t n_row_tiles, int64_t n_band,
                                                    int32_t window, double r2_min, LdScratch sc,
                                                    const int64_t* __restrict__ gsum,
                                                    const int* __restrict__ gmax,
                                                    const uint32_t* __restrict__ groups_ok,
                                                    uint32_t min_groups, int cap, int64_t budget) {
  __shared__ __attribute__((aligned(16))) uint32_t smem[kLdMfmaSmem];
  // all of them the correction path's: decided by one word
  if (gsum && groups_ok[0] >= min_groups && groups_ok[2] == 0) return;
  const int64_t b = xcd_swizzle(blockIdx.x, gridDim.x);
  const int64_t I = b / n_band;
  const int64_t J = I + b % n_band;
  if (J >= n_row_tiles) return;
  if (gsum && ld_tile_sparse(gsum, gmax, groups_ok, min_groups, I, J, cap, budget))
    return;   // the correction path's
  if constexpr (kTile == kLdTileNib)   // the operand is E
    ld_nib_tile(D, wn / 4, nv, I, J, window, r2_min, sc, (lds_t*)smem);
  else if constexpr (kTile == kLdTileFp4)
    ld_fp4_tile_pipe(D, wn, nv, I, J, window, r2_min, sc, (lds_t*)smem);
  else
    ld_mfma_tile(D, wn, nv, I, J, window, r2_min, sc, (lds_t*)smem);
}

int launch_ld_mfma(const uint32_t* D, const uint32_t* E, bool fp4, int64_t wn, int64_t nv,
                   int64_t rows_pad, int32_t window, double r2_min, const LdScratch& sc,
                   hipStream_t st, const LdSparse* sp) {
  int rc;
  const int64_t n_row_tiles = rows_pad / kL;
  const int64_t n_band = ((int64_t)window + kL - 1) / kL + 1;
  const int64_t blocks = n_row_tiles * n_band;
  hipLaunchKernelGGL((E ? k_ld_mfma<kLdTileNib>
                        : fp4 ? k_ld_mfma<kLdTileFp4> : k_ld_mfma<kLdTileInt8>),
                     dim3((unsigned)blocks), dim3(256), 0, st, E ? E : D, wn, nv, n_row_tiles,
                     n_band, window, r2_min, sc, sp ? sp->gsum : nullptr,
                     sp ? sp->gmax : nullptr, sp ? sp->groups_ok : nullptr,
                     sp ? sp->min_groups : 0u, sp ? sp->cap : 0, sp ? sp->budget : 0);
  rc = check_launch("ld_mfma");
  if (!sp) mark_stage(2, st);
  return rc;
}

// ---- scan: row counts -> row offsets, total -> *n_out ----------------------------
// Up to kScanOneRows rows: one block, 32 rows a thread held in registers, wave
// scans by lane shuffles and one exchange of wave sums: bound by latency, 6.4
// us at 20,011 rows against 4 + 4 + 8.5 us and two gaps for three kernels.
// More: per-block sums (4096 rows per block), one block scanning the block
// sums, then per-block exclusive scans plus the block's offset (5.5 + 4.8 + 9
// us at 500,000 rows).
constexpr int kScanOneU = 8;                                  // groups of 4 rows per thread
constexpr int64_t kScanOneRows = 4 * 1024 * (int64_t)kScanOneU;

// Rows [base, base + kScanOneRows) of nv from the offset `carry` on; returns
// the offset past them.  1024 threads.  The sums within are 32 bits wide: at
// most 32,768 rows of fewer than kLdScanJobRows pairs each.
static_assert(kScanOneRows * (kLdScanJobRows - 1) < ((int64_t)1 << 32), "row sums in 32 bits");
__device__ __forceinline__ int64_t scan_rows_block(const LdScratch& sc, int64_t nv, int64_t base,
                                                   int64_t carry, uint32_t* s_w) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  uint4 c[kScanOneU];
  uint32_t incl[kScanOneU];
#pragma unroll
  for (int u = 0; u < kScanOneU; ++u) {   // rows past nv within the padding count 0
    const int64_t r = base + 4 * (1024 * u + t);
    c[u] = r < nv ? *reinterpret_cast<const uint4*>(sc.rowcnt + r) : make_uint4(0, 0, 0, 0);
    incl[u] = c[u].x + c[u].y + c[u].z + c[u].w;
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1)
#pragma unroll
    for (int u = 0; u < kScanOneU; ++u) {
      const uint32_t o = __shfl_up(incl[u], d);
      incl[u] += lane >= d ? o : 0u;
    }
  if (lane == 63)
#pragma unroll
    for (int u = 0; u < kScanOneU; ++u) s_w[16 * u + wave] = incl[u];
  __syncthreads();
  // every wave scans the 128 wave sums itself
  const uint32_t w0 = s_w[2 * lane], w1 = s_w[2 * lane + 1];
  uint32_t ws = w0 + w1;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(ws, d);
    ws += lane >= d ? o : 0u;
  }
#pragma unroll
  for (int u = 0; u < kScanOneU; ++u) {
    const int k = 16 * u + wave;   // this wave's place among the sums
    const uint32_t to = __shfl(ws, k >> 1), b1 = __shfl(w1, k >> 1), b0 = __shfl(w0, k >> 1);
    const uint32_t before = to - b1 - ((k & 1) ? 0u : b0);
    const int64_t o = carry + before + (incl[u] - (c[u].x + c[u].y + c[u].z + c[u].w));
    const int64_t r = base + 4 * (1024 * u + t);
    if (r < nv) {   // off has rows_pad + 1 places, rows_pad a multiple of 4
      longlong2* p = reinterpret_cast<longlong2*>(sc.rowoff + r);
      p[0] = make_longlong2(o, o + c[u].x);
      p[1] = make_longlong2(o + c[u].x + c[u].y, o + c[u].x + c[u].y + c[u].z);
    }
  }
  const int64_t total = carry + __shfl(ws, 63);
  __syncthreads();
  return total;
}

__device__ __forceinline__ void scan_rows_all(const LdScratch& sc, int64_t nv, int64_t* n_out) {
  __shared__ uint32_t s_w[16 * kScanOneU];
  int64_t carry = 0;
  for (int64_t base = 0; base < nv; base += kScanOneRows)
    carry = scan_rows_block(sc, nv, base, carry, s_w);
  if (threadIdx.x == 0) {
    sc.rowoff[nv] = carry;
    *n_out = carry;
  }
}

__global__ __launch_bounds__(1024) void k_scan_one(LdScratch sc, int64_t nv, int64_t* n_out) {
  scan_rows_all(sc, nv, n_out);
}

__global__ __launch_bounds__(1024) void k_scan_jobs(const LdFinishJob* __restrict__ jobs) {
  const LdFinishJob j = jobs[blockIdx.x];
  if (j.nv <= kLdScanJobRows) scan_rows_all(j.sc, j.nv, j.n_out);
}

constexpr int kScanPer = 16;                  // rows per thread
constexpr int kScanBlock = 256 * kScanPer;    // rows per block

__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t* sh, int64_t* total) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int d = 1; d < (int)blockDim.x; d <<= 1) {
    const int64_t add = t >= d ? sh[t - d] : 0;
    __syncthreads();
    sh[t] += add;
    __syncthreads();
  }
  const int64_t incl = sh[t];
  if (total) *total = sh[blockDim.x - 1];
  __syncthreads();
  return incl - v;
}

__global__ __launch_bounds__(256) void k_scan_sums(const uint32_t* __restrict__ cnt, int64_t nv,
                                                   int64_t* __restrict__ bsum) {
  __shared__ int64_t sh[256];
  const int64_t base = (int64_t)blockIdx.x * kScanBlock + threadIdx.x * kScanPer;
  int64_t s = 0;
  for (int i = 0; i < kScanPer; ++i)
    if (base + i < nv) s += cnt[base + i];
  int64_t tot;
  block_exclusive_scan(s, sh, &tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void k_scan_top(int64_t* __restrict__ bsum, int64_t nb,
                                                   int64_t nv, int64_t* __restrict__ off,
                                                   int64_t* n_out) {
  __shared__ int64_t sh[1024];
  const int64_t per = ceil_div(nb, 1024);
  const int64_t lo = threadIdx.x * per;
  int64_t s = 0;
  for (int64_t i = lo; i < lo + per && i < nb; ++i) s += bsum[i];
  int64_t tot;
  int64_t run = block_exclusive_scan(s, sh, &tot);
  for (int64_t i = lo; i < lo + per && i < nb; ++i) {
    const int64_t v = bsum[i];
    bsum[i] = run;
    run += v;
  }
  if (threadIdx.x == 0) {
    off[nv] = tot;
    *n_out = tot;
  }
}

__global__ __launch_bounds__(256) void k_scan_apply(const uint32_t* __restrict__ cnt, int64_t nv,
                                                    const int64_t* __restrict__ bsum,
                                                    int64_t* __restrict__ off) {
  __shared__ int64_t sh[256];
  const int64_t base = (int64_t)blockIdx.x * kScanBlock + threadIdx.x * kScanPer;
  int64_t s = 0;
  for (int i = 0; i < kScanPer; ++i)
    if (base + i < nv) s += cnt[base + i];
  int64_t run = block_exclusive_scan(s, sh, nullptr) + bsum[blockIdx.x];
  for (int i = 0; i < kScanPer; ++i)
    if (base + i < nv) {
      off[base + i] = run;
      run += cnt[base + i];
    }
}

// ---- emit: one record per thread ---------------------------------------------------
// Record r (< min(total, capacity)) belongs to the row a with off[a] <= r <
// off[a+1] (binary search), and to the (r - off[a])-th marked bit of that
// row's bitmap.  Its sums are recomputed with popcounts over the operand the
// pair kernel used (2-bit words or bit planes) -- an independent integer route
// to the same exact values.
struct Sums6 {
  int n, sx, sy, sxx, syy, sxy;
};

__device__ __forceinline__ void add_plane_sums(Sums6& z, uint32_t pa, uint32_t qa, uint32_t ma,
                                               uint32_t pb, uint32_t qb, uint32_t mb) {
  z.n += __builtin_popcount(ma & mb);
  z.sx += __builtin_popcount(pa & mb) - __builtin_popcount(qa & mb);
  z.sy += __builtin_popcount(pb & ma) - __builtin_popcount(qb & ma);
  z.sxx += __builtin_popcount((pa | qa) & mb);
  z.syy += __builtin_popcount((pb | qb) & ma);
  z.sxy += __builtin_popcount((pa & pb) | (qa & qb)) - __builtin_popcount((pa & qb) | (qa & pb));
}

constexpr int kEmitU = 4;

template <bool kPlanes>
__device__ __forceinline__ void emit_records(const uint32_t* __restrict__ X, int64_t words,
                                             int64_t rows_pad, int64_t nv, int64_t v0,
                                             const LdScratch& sc, pg_ld_pair* __restrict__ out,
                                             int64_t capacity) {
  const int64_t total = sc.rowoff[nv] < capacity ? sc.rowoff[nv] : capacity;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < total;
       r += (int64_t)gridDim.x * blockDim.x) {
    int64_t lo = 0, hi = nv;                       // find last a with off[a] <= r
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (sc.rowoff[mid] <= r) lo = mid; else hi = mid;
    }
    const int64_t a = lo;
    int64_t k = r - sc.rowoff[a];
    int64_t b = -1;
    for (int64_t q = 0; q < sc.bm_words; ++q) {
      uint32_t bits = sc.bitmap[a * sc.bm_words + q];
      const int pc = __builtin_popcount(bits);
      if (k < pc) {
        for (; k > 0; --k) bits &= bits - 1;
        b = a + 1 + q * 32 + __builtin_ctz(bits);
        break;
      }
      k -= pc;
    }
    if (b < 0) continue;   // unreachable when counts and bitmap agree
    // the row loops load kEmitU steps ahead, so a thread has that many
    // loads in flight instead of waiting on each
    Sums6 z{0, 0, 0, 0, 0, 0};
    if constexpr (kPlanes) {
      int64_t w = 0;
      for (; w + kEmitU <= words; w += kEmitU) {
        uint32_t v[kEmitU][6];
#pragma unroll
        for (int u = 0; u < kEmitU; ++u) {
          const uint32_t* pw = X + (w + u) * 3 * rows_pad;
          v[u][0] = pw[a]; v[u][1] = pw[rows_pad + a]; v[u][2] = pw[2 * rows_pad + a];
          v[u][3] = pw[b]; v[u][4] = pw[rows_pad + b]; v[u][5] = pw[2 * rows_pad + b];
        }
#pragma unroll
        for (int u = 0; u < kEmitU; ++u)
          add_plane_sums(z, v[u][0], v[u][1], v[u][2], v[u][3], v[u][4], v[u][5]);
      }
      for (; w < words; ++w) {
        const uint32_t* pw = X + w * 3 * rows_pad;
        add_plane_sums(z, pw[a], pw[rows_pad + a], pw[2 * rows_pad + a], pw[b],
                       pw[rows_pad + b], pw[2 * rows_pad + b]);
      }
    } else {
      const uint4* ra = reinterpret_cast<const uint4*>(X + a * words);
      const uint4* rb = reinterpret_cast<const uint4*>(X + b * words);
      auto add4 = [&z](const uint4& A, const uint4& B) {
        const uint32_t xs[4] = {A.x, A.y, A.z, A.w}, ys[4] = {B.x, B.y, B.z, B.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t pa, qa, ma, pb, qb, mb;
          masks_of_word(xs[e], pa, qa, ma);
          masks_of_word(ys[e], pb, qb, mb);
          add_plane_sums(z, pa, qa, ma, pb, qb, mb);
        }
      };
      const int64_t n4 = words / 4;
      int64_t w4 = 0;
      for (; w4 + kEmitU <= n4; w4 += kEmitU) {
        uint4 A[kEmitU], B[kEmitU];
#pragma unroll
        for (int u = 0; u < kEmitU; ++u) { A[u] = ra[w4 + u]; B[u] = rb[w4 + u]; }
#pragma unroll
        for (int u = 0; u < kEmitU; ++u) add4(A[u], B[u]);
      }
      for (; w4 < n4; ++w4) add4(ra[w4], rb[w4]);
    }
    pg_ld_pair rec;
    rec.a = (int32_t)(v0 + a);
    rec.b = (int32_t)(v0 + b);
    rec.n = z.n; rec.sx = z.sx; rec.sy = z.sy; rec.sxx = z.sxx; rec.syy = z.syy; rec.sxy = z.sxy;
    rec.r2 = ld_r2(z.n, z.sx, z.sy, z.sxx, z.syy, z.sxy);
    out[r] = rec;
  }
}

template <bool kPlanes>
__global__ __launch_bounds__(256) void k_ld_emit(const uint32_t* __restrict__ X, int64_t words,
                                                 int64_t rows_pad, int64_t nv, int64_t v0,
                                                 LdScratch sc, pg_ld_pair* __restrict__ out,
                                                 int64_t capacity) {
  emit_records<kPlanes>(X, words, rows_pad, nv, v0, sc, out, capacity);
}

// Problem blockIdx.y of the table.
template <bool kPlanes>
__global__ __launch_bounds__(256) void k_ld_emit_jobs(const LdFinishJob* __restrict__ jobs) {
  const LdFinishJob j = jobs[blockIdx.y];
  emit_records<kPlanes>(j.X, j.words, j.rows_pad, j.nv, j.v0, j.sc, j.out, j.capacity);
}

int ld_scan_blocks(int64_t nv) { return (int)ceil_div(nv, kScanBlock); }

int scan_ld_rows(const LdScratch& sc, int64_t nv, int64_t* n_out, hipStream_t st) {
  if (nv <= kScanOneRows) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(1024), 0, st, sc, nv, n_out);
    return check_launch("ld_scan_one");
  }
  const int64_t nb = ceil_div(nv, kScanBlock);
  hipLaunchKernelGGL(k_scan_sums, dim3((unsigned)nb), dim3(256), 0, st, sc.rowcnt, nv, sc.bsum);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, st, sc.bsum, nb, nv, sc.rowoff, n_out);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(256), 0, st, sc.rowcnt, nv, sc.bsum,
                     sc.rowoff);
  return check_launch("ld_scan");
}

int launch_ld_finish_jobs(const LdFinishJob* jobs, int n_words, int n_planes,
                          const int64_t* max_capacity, hipStream_t st) {
  if (n_words + n_planes <= 0) return PG_OK;
  hipLaunchKernelGGL(k_scan_jobs, dim3((unsigned)(n_words + n_planes)), dim3(1024), 0, st, jobs);
  int rc = check_launch("ld_scan_jobs");
  auto gx = [](int64_t capacity) {
    return (unsigned)(ceil_div(capacity, 256) < 2048 ? ceil_div(capacity, 256) : 2048);
  };
  constexpr int kMaxY = 32768;   // table slices a launch's grid takes
  for (int i = 0; rc == PG_OK && max_capacity[0] > 0 && i < n_words; i += kMaxY) {
    const unsigned gy = (unsigned)(n_words - i < kMaxY ? n_words - i : kMaxY);
    hipLaunchKernelGGL(k_ld_emit_jobs<false>, dim3(gx(max_capacity[0]), gy), dim3(256), 0, st,
                       jobs + i);
    rc = check_launch("ld_emit_jobs");
  }
  for (int i = 0; rc == PG_OK && max_capacity[1] > 0 && i < n_planes; i += kMaxY) {
    const unsigned gy = (unsigned)(n_planes - i < kMaxY ? n_planes - i : kMaxY);
    hipLaunchKernelGGL(k_ld_emit_jobs<true>, dim3(gx(max_capacity[1]), gy), dim3(256), 0, st,
                       jobs + n_words + i);
    rc = check_launch("ld_emit_jobs");
  }
  return rc;
}

int launch_ld_finish(const uint32_t* X, bool planes, int64_t words, int64_t rows_pad, int64_t nv,
                     int64_t v0, const LdScratch& sc, pg_ld_pair* out, int64_t capacity,
                     int64_t* n_out, hipStream_t st) {
  int rc = scan_ld_rows(sc, nv, n_out, st);
  mark_stage(3, st);
  if (rc == PG_OK && capacity > 0) {
    if (planes)
      hipLaunchKernelGGL(k_ld_emit<true>, dim3(2048), dim3(256), 0, st, X, words, rows_pad, nv, v0,
                         sc, out, capacity);
    else
      hipLaunchKernelGGL(k_ld_emit<false>, dim3(2048), dim3(256), 0, st, X, words, rows_pad, nv, v0,
                         sc, out, capacity);
    rc = check_launch("ld_emit");
  }
  mark_stage(4, st);
  return rc;
}

}  // namespace pg
