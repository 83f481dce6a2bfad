// Layout kernels: turn the caller's variant-major .bed selection into the
// operand layouts of the pair kernels.  All are single passes over the input,
// bound by HBM traffic.  Padding positions are written as missing calls, so
// they contribute nothing to any count.
#include "tiles.h"

namespace pg {

// ---- helpers for whole-matrix selections (no sample list) -------------------
__device__ __forceinline__ uint32_t spread16(uint32_t x) {
  // bit k -> bit 2k, for the low 16 bits
  x &= 0xFFFFu;
  x = (x | (x << 8)) & 0x00FF00FFu;
  x = (x | (x << 4)) & 0x0F0F0F0Fu;
  x = (x | (x << 2)) & 0x33333333u;
  x = (x | (x << 1)) & 0x55555555u;
  return x;
}

// Word g of selected variant v: sixteen consecutive samples of the row as a
// 2-bit word (sample 16g + k at bits 2k), with the missing mask applied and
// samples >= m (and variants >= nv) forced to missing.  This reads the words
// of N (v, g) pairs and issues every load before any result is used (a reader
// that branches per word waits on each load in turn).  Dword-aligned rows take
// one dword per word, other rows two aligned dwords, shifted; a word whose
// dwords would leave the selected rows (a row's last partial dword, the edges
// of the selection) is read byte by byte afterwards.  Words read in place of
// those come from the first dwords of the selection and are discarded.
template <int N>
__device__ __forceinline__ void row_words16(const Sel& s, const int64_t (&v)[N],
                                            const int64_t (&g)[N], bool aligned,
                                            uint32_t (&w)[N]) {
  const uint8_t* first = s.bed + s.v0 * s.bpv;
  const uint8_t* end = first + s.nv * s.bpv;
  const uint8_t* safe =
      reinterpret_cast<const uint8_t*>((reinterpret_cast<uintptr_t>(first) + 3) & ~(uintptr_t)3);
  const bool loads = aligned ? s.nv > 0 && s.bpv >= 4 : safe + 8 <= end;   // same for all lanes
  bool fast[N];
  uint32_t lo[N], hi[N];
  if (loads && aligned) {
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const uint8_t* p = first + v[r] * s.bpv + 4 * g[r];
      fast[r] = v[r] < s.nv && s.bpv - 4 * g[r] >= 4;
      lo[r] = *reinterpret_cast<const uint32_t*>(fast[r] ? p : first);
      hi[r] = 0;
    }
  } else if (loads) {
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const uint8_t* p = first + v[r] * s.bpv + 4 * g[r];
      const uint8_t* pa =
          reinterpret_cast<const uint8_t*>(reinterpret_cast<uintptr_t>(p) & ~(uintptr_t)3);
      fast[r] = v[r] < s.nv && s.bpv - 4 * g[r] >= 4 && pa >= first && pa + 8 <= end;
      const uint32_t* q = reinterpret_cast<const uint32_t*>(fast[r] ? pa : safe);
      lo[r] = q[0];
      hi[r] = q[1];
    }
  } else {
#pragma unroll
    for (int r = 0; r < N; ++r) { fast[r] = false; lo[r] = hi[r] = 0; }
  }
  uint64_t mw[N];
  if (s.mask) {
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const bool in = v[r] < s.nv && s.m - 16 * g[r] > 0;
      mw[r] = s.mask[in ? (s.v0 + v[r]) * s.wpm + ((16 * g[r]) >> 6) : 0];
    }
  }
#pragma unroll
  for (int r = 0; r < N; ++r) {
    uint32_t x;
    if (fast[r]) {
      const uintptr_t p = reinterpret_cast<uintptr_t>(first + v[r] * s.bpv + 4 * g[r]);
      x = aligned ? lo[r] : (uint32_t)((((uint64_t)hi[r] << 32) | lo[r]) >> (8 * (p & 3)));
    } else if (v[r] >= s.nv) {
      x = kAllMissing16;
    } else {
      const uint8_t* p = first + v[r] * s.bpv + 4 * g[r];
      const int64_t avail = s.bpv - 4 * g[r];
      x = 0;
      for (int b = 0; b < 4; ++b)
        if (b < avail) x |= (uint32_t)p[b] << (8 * b);
    }
    const int64_t valid = s.m - 16 * g[r];
    if (valid < 16) {
      const uint32_t keep = valid <= 0 ? 0u : ((1u << (2 * valid)) - 1u);
      x = (x & keep) | (kAllMissing16 & ~keep);
    }
    if (s.mask && valid > 0 && v[r] < s.nv) {
      const uint32_t lanes = spread16((uint32_t)(mw[r] >> ((16 * g[r]) & 63)));
      x = (x & ~(lanes | (lanes << 1))) | lanes;  // masked calls -> code 01
    }
    w[r] = x;
  }
}

// Sample-major 2-bit words without a sample list, 512 samples x 256 variants
// per block: lanes read consecutive words of one .bed row (whole lines), the
// 16x16 transposes land in LDS, and the block writes 64-byte runs of T rows.
// The block's 34 KB of LDS let four blocks share a CU (512 x 512 blocks, 68
// KB: two per CU, 17% slower at 10,000 x 100,000).
// Samples past the matrix and variants past the selection are missing calls.
// Where those blocks would leave CUs idle, blocks of 128 samples x 256 variants
// by 128 threads, each with one word's sixteen loads: 500 x 5,000, 20 blocks in
// two passes 14 us, 80 blocks 9 us.
constexpr int kSmTG = 32;            // sample groups (16 samples) per block
constexpr int kSmTGSmall = 8;
constexpr int kSmTW = 16;            // T words (16 variants) per block
constexpr int kSmTS = kSmTW + 1;     // LDS row stride (words)

// Block `bid` of the tiled layout of one operand: kTG sample groups, kThreads
// threads.
template <int kTG, int kThreads>
__device__ __forceinline__ void sample_major_tiled_block(const Sel& s, uint32_t* __restrict__ T,
                                                         int64_t rows_pad, int64_t wp,
                                                         int aligned, int64_t bid,
                                                         uint32_t* s_out) {
  const int64_t nb_g = ceil_div(rows_pad / 16, kTG);
  const int64_t g0 = (bid % nb_g) * kTG;     // sample group (16 samples)
  const int64_t a0 = (bid / nb_g) * kSmTW;   // T word (16 variants)
  const int t = threadIdx.x;
  const int gl = t % kTG;
#pragma unroll 1
  for (int i = 0; i < kSmTW * kTG / kThreads; ++i) {
    const int al = t / kTG + kThreads / kTG * i;
    const int64_t a = a0 + al, g = g0 + gl;
    int64_t vr[16], gr[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) { vr[r] = 16 * a + r; gr[r] = g; }   // (16 wp >= nv)
    uint32_t x[16];
    row_words16(s, vr, gr, aligned != 0, x);
    transpose16_2bit(x);
#pragma unroll
    for (int c = 0; c < 16; ++c) s_out[(c * kTG + gl) * kSmTS + al] = x[c];
  }
  __syncthreads();
  for (int e = t; e < 16 * kTG * kSmTW; e += kThreads) {
    const int row = e / kSmTW, col = e % kSmTW;
    const int64_t k = 16 * g0 + row, a = a0 + col;
    if (k < rows_pad && a < wp)   // T row 16 gl + c is LDS row c * kTG + gl
      T[k * wp + a] = s_out[((row & 15) * kTG + (row >> 4)) * kSmTS + col];
  }
}

template <int kTG, int kThreads>
__global__ __launch_bounds__(kThreads) void k_sample_major_tiled(Sel s, uint32_t* __restrict__ T,
                                                                 int64_t rows_pad, int64_t wp,
                                                                 int aligned) {
  __shared__ uint32_t s_out[16 * kTG * kSmTS];
  // blocks of one XCD take consecutive sample groups of the same variants, so
  // the row pieces that straddle two blocks' reads meet in that XCD's L2
  sample_major_tiled_block<kTG, kThreads>(s, T, rows_pad, wp, aligned,
                                          xcd_swizzle(blockIdx.x, gridDim.x), s_out);
}

// Many operands in one launch: block b lays out block b - block_begin of the
// job whose block range holds b (jobs in increasing block_begin).
__global__ __launch_bounds__(256) void k_sample_major_jobs(const LayoutJob* __restrict__ jobs,
                                                           int n_jobs) {
  __shared__ uint32_t s_out[16 * kSmTG * kSmTS];
  const int64_t b = blockIdx.x;
  int lo = 0, hi = n_jobs - 1;
  while (lo < hi) {   // the last job with block_begin <= b
    const int mid = (lo + hi + 1) / 2;
    if (jobs[mid].block_begin <= b) lo = mid; else hi = mid - 1;
  }
  const LayoutJob j = jobs[lo];
  sample_major_tiled_block<kSmTG, 256>(j.s, j.T, j.rows_pad, j.wp, j.aligned, b - j.block_begin,
                                       s_out);
}

int64_t sample_major_job_blocks(int64_t rows_pad, int64_t wp) {
  return ceil_div(wp, kSmTW) * ceil_div(rows_pad, 16 * kSmTG);
}

int launch_sample_major_jobs(const LayoutJob* jobs, int n_jobs, int64_t total_blocks,
                             hipStream_t st) {
  if (n_jobs <= 0 || total_blocks <= 0) return PG_OK;
  hipLaunchKernelGGL(k_sample_major_jobs, dim3((unsigned)total_blocks), dim3(256), 0, st, jobs,
                     n_jobs);
  return check_launch("sample_major_jobs");
}

// Every other bit (bits 0, 2, 4, ... of x) packed into the low 16 bits.
__device__ __forceinline__ uint32_t compact_even_bits(uint32_t x) {
  x &= 0x55555555u;
  x = (x | (x >> 1)) & 0x33333333u;
  x = (x | (x >> 2)) & 0x0F0F0F0Fu;
  x = (x | (x >> 4)) & 0x00FF00FFu;
  x = (x | (x >> 8)) & 0x0000FFFFu;
  return x;
}

// Bit planes without a sample list: a thread owns 16 samples x 32 variants
// (two 16x16 transposes), then splits each sample's 32 codes into the high
// bit, low bit and non-missing planes; it writes 16 consecutive samples of
// each plane word.
__global__ __launch_bounds__(256) void k_ibs_planes_fast(Sel s, uint32_t* __restrict__ P,
                                                         int64_t rows_pad, int64_t words_pad,
                                                         int aligned) {
  const int64_t groups = rows_pad / 16;
  const int64_t total = groups * words_pad;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t g = e % groups;
    const int64_t w = e / groups;
    uint32_t lo16[16], hi16[16];
    int64_t vr[16], gr[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) { vr[r] = 32 * w + r; gr[r] = g; }
    row_words16(s, vr, gr, aligned != 0, lo16);
#pragma unroll
    for (int r = 0; r < 16; ++r) vr[r] += 16;
    row_words16(s, vr, gr, aligned != 0, hi16);
    transpose16_2bit(lo16);
    transpose16_2bit(hi16);
    uint32_t H[16], L[16], M[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const uint32_t a = lo16[c], b = hi16[c];   // variants 0-15 and 16-31 of sample c
      const uint32_t miss_a = a & ~(a >> 1) & 0x55555555u;   // code 01
      const uint32_t miss_b = b & ~(b >> 1) & 0x55555555u;
      H[c] = compact_even_bits(a >> 1) | (compact_even_bits(b >> 1) << 16);
      L[c] = compact_even_bits(a) | (compact_even_bits(b) << 16);
      M[c] = ~(compact_even_bits(miss_a) | (compact_even_bits(miss_b) << 16));
    }
    uint32_t* dst = P + (w * 3) * rows_pad + 16 * g;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      *reinterpret_cast<uint4*>(dst + 4 * q) = make_uint4(H[4 * q], H[4 * q + 1], H[4 * q + 2], H[4 * q + 3]);
      *reinterpret_cast<uint4*>(dst + rows_pad + 4 * q) =
          make_uint4(L[4 * q], L[4 * q + 1], L[4 * q + 2], L[4 * q + 3]);
      *reinterpret_cast<uint4*>(dst + 2 * rows_pad + 4 * q) =
          make_uint4(M[4 * q], M[4 * q + 1], M[4 * q + 2], M[4 * q + 3]);
    }
  }
}

// Variant-major bit planes for the popcount LD path: for 32-sample word w,
// plane p (0 = homozygous A2, 1 = homozygous A1, 2 = non-missing) of selected
// variant v at P[(w*3 + p)*rows_pad + v].  One plane word per thread.
__device__ __forceinline__ void ld_planes_of(uint32_t x, uint32_t& hom2, uint32_t& hom1,
                                             uint32_t& nonmiss) {
  const uint32_t lo = x & 0x55555555u, hi = (x >> 1) & 0x55555555u;
  hom2 = compact_even_bits(lo & hi);
  hom1 = compact_even_bits(~(lo | hi) & 0x55555555u);
  nonmiss = compact_even_bits(~(lo & ~hi) & 0x55555555u);
}

__global__ __launch_bounds__(256) void k_ld_planes(Sel s, uint32_t* __restrict__ P, int64_t rows_pad,
                                                   int64_t words_pad) {
  const int64_t total = rows_pad * words_pad;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t v = e % rows_pad;
    const int64_t w = e / rows_pad;
    uint32_t x0 = 0, x1 = 0;
    for (int b = 0; b < 16; ++b) {
      x0 |= code_at(s, v, 32 * w + b) << (2 * b);
      x1 |= code_at(s, v, 32 * w + 16 + b) << (2 * b);
    }
    uint32_t p0, q0, m0, p1, q1, m1;
    ld_planes_of(x0, p0, q0, m0);
    ld_planes_of(x1, p1, q1, m1);
    P[(w * 3 + 0) * rows_pad + v] = p0 | (p1 << 16);
    P[(w * 3 + 1) * rows_pad + v] = q0 | (q1 << 16);
    P[(w * 3 + 2) * rows_pad + v] = m0 | (m1 << 16);
  }
}

// Replicated fp4 operand: for each sample and each group of 8 variants, two
// words.  HR holds each code's high bit at nibble bits 1 and 3; LR holds its
// low bit at nibble bits 1 and 3 and ones at nibble bits 0 and 2.  Missing
// positions (and padding) are HR = 0, LR = ~0.  With this layout every fp4
// feature nibble is one three-input bit function of (HR, LR, bit-1 mask).
__device__ __forceinline__ void rep_pair(uint32_t codes8, uint32_t& hr, uint32_t& lr) {
  // codes8: 8 codes in the low 16 bits, code t at bits 2t -> code t at bits 4t (nibbles)
  uint32_t x = codes8 & 0xFFFFu;
  x = (x | (x << 8)) & 0x00FF00FFu;
  x = (x | (x << 4)) & 0x0F0F0F0Fu;
  x = (x | (x << 2)) & 0x33333333u;
  const uint32_t hi = (x >> 1) & 0x11111111u, lo = x & 0x11111111u;
  hr = (hi << 1) | (hi << 3);
  lr = (lo << 1) | (lo << 3) | 0x55555555u;
}

// Replicated operand without a sample list: a thread owns 16 samples x 64
// variants (four 16x16 transposes) and writes 16 words per sample row.
__global__ __launch_bounds__(256) void k_sample_major_rep(Sel s, uint32_t* __restrict__ R,
                                                          int64_t rows_pad, int64_t rp,
                                                          int aligned) {
  const int64_t groups = rows_pad / 16;
  const int64_t quads = rp / 16;               // 64 variants = 16 words per sample
  const int64_t total = groups * quads;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t g = e % groups;
    const int64_t q = e / groups;
    uint32_t out[4][16];
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) {
      const int64_t w = 4 * q + ww;
      int64_t vr[16], gr[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) { vr[r] = 16 * w + r; gr[r] = g; }
      row_words16(s, vr, gr, aligned != 0, out[ww]);
      transpose16_2bit(out[ww]);
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      uint32_t v[16];
#pragma unroll
      for (int ww = 0; ww < 4; ++ww) {
        rep_pair(out[ww][c], v[4 * ww + 0], v[4 * ww + 1]);
        rep_pair(out[ww][c] >> 16, v[4 * ww + 2], v[4 * ww + 3]);
      }
      uint4* dst = reinterpret_cast<uint4*>(R + (16 * g + c) * rp + 16 * q);
#pragma unroll
      for (int k = 0; k < 4; ++k) dst[k] = make_uint4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
    }
  }
}

// Replicated operand with a sample list: one 8-variant group per thread.
__global__ __launch_bounds__(256) void k_sample_major_rep_gather(Sel s, uint32_t* __restrict__ R,
                                                                 int64_t rows_pad, int64_t rp) {
  const int64_t ngroups = rp / 2;
  const int64_t total = rows_pad * ngroups;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / ngroups;
    const int64_t q = e % ngroups;
    uint32_t codes = 0;
    for (int b = 0; b < 8; ++b) codes |= code_at(s, 8 * q + b, i) << (2 * b);
    uint32_t hr, lr;
    rep_pair(codes, hr, lr);
    R[i * rp + 2 * q] = hr;
    R[i * rp + 2 * q + 1] = lr;
  }
}

// Calls and A2 alleles of every selected variant: one wave per variant, its
// words straight from the rows (kFromD: from D, a sample list's layout), kU a
// lane in flight.  Bound by reading the calls once: 62 us for 10,000 x 71,307,
// against 82 us for laying them out and 67 us for counting in that copy (two
// variants a wave, 20 loads in flight at one address a row: 56 us, and the same
// 0.47 ms for the whole report).
template <bool kFromD, int kU>
__global__ __launch_bounds__(256) void k_allele_counts(Sel s, const uint32_t* __restrict__ D,
                                                       int64_t wn, int aligned,
                                                       uint2* __restrict__ counts) {
  const int lane = threadIdx.x & 63;
  const int64_t v = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (v >= s.nv) return;
  uint32_t calls = 0, a2 = 0;
  for (int64_t w0 = 0; w0 < wn; w0 += 64 * kU) {
    int64_t vr[kU], gr[kU];
    uint32_t x[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      vr[u] = v;
      gr[u] = w0 + 64 * u + lane;
    }
    if constexpr (kFromD) {
#pragma unroll
      for (int u = 0; u < kU; ++u) x[u] = gr[u] < wn ? D[v * wn + gr[u]] : kAllMissing16;
    } else {
      row_words16(s, vr, gr, aligned != 0, x);   // missing past the row
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint32_t lo = x[u] & 0x55555555u, hi = (x[u] >> 1) & 0x55555555u;
      calls += __popc((hi | ~lo) & 0x55555555u);          // codes 00, 10, 11
      a2 += 2 * __popc(hi & lo) + __popc(hi & ~lo);       // 11 twice, 10 once
    }
  }
  for (int d = 32; d > 0; d >>= 1) {
    calls += __shfl_xor(calls, d, 64);
    a2 += __shfl_xor(a2, d, 64);
  }
  if (lane == 0) counts[v] = make_uint2(calls, a2);
}

bool rows_dword_aligned(const Sel& s) {
  return (s.bpv % 4) == 0 && (reinterpret_cast<uintptr_t>(s.bed) % 4) == 0;
}

static unsigned stride_grid(int64_t items) {
  const int64_t b = ceil_div(items, 256);
  return (unsigned)(b < 65536 ? b : 65536);
}

// ---- sample-major 2-bit words with a sample list (IBS, matrix-core path) -----
// A wave owns 64 samples x 4 words (64 variants), a block four consecutive
// word quads of the same samples (64-byte runs of T rows).  Each lane keeps
// one sample: its list entry is read once, and the 16 bytes of a word are
// loaded before any is used, so a wave has 32 loads in flight.  Bound by the
// latency of those loads; a reader that took one code at a time (list entry,
// bounds, byte, mask) 174 us for 1,733 of 6,011 samples x 10,121 variants,
// this one 18 us.
constexpr int kSmSamples = 64;
constexpr int kSmWords = 16;

__global__ __launch_bounds__(256) void k_sample_major_2bit(Sel s, uint32_t* __restrict__ T,
                                                           int64_t rows_pad, int64_t wp) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nbi = ceil_div(rows_pad, kSmSamples);
  const int64_t i = ((int64_t)blockIdx.x % nbi) * kSmSamples + lane;
  const int64_t w0 = ((int64_t)blockIdx.x / nbi) * kSmWords + 4 * wave;
  if (w0 >= wp) return;
  const int64_t smp = i < s.m ? (int64_t)s.idx[i] : -1;
  const bool in = smp >= 0 && smp < s.n;      // a sample without calls otherwise
  // row addresses are uniform, the sample's place in a row 32 bits
  const uint32_t k = in ? (uint32_t)smp : 0u;
  const int shift = 2 * (int)(k & 3);
  uint32_t out[4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint32_t byte[32], miss[32];
#pragma unroll
    for (int b = 0; b < 32; ++b) {
      const int64_t v = 16 * w0 + 32 * h + b;
      byte[b] = (s.bed + (s.v0 + (v < s.nv ? v : s.nv - 1)) * s.bpv)[k >> 2];
      miss[b] = 0u;
    }
    if (s.mask) {
#pragma unroll
      for (int b = 0; b < 32; ++b) {
        const int64_t v = 16 * w0 + 32 * h + b;
        miss[b] = reinterpret_cast<const uint32_t*>(
                      s.mask + (s.v0 + (v < s.nv ? v : s.nv - 1)) * s.wpm)[k >> 5] >> (k & 31);
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      uint32_t word = 0;
#pragma unroll
      for (int b = 0; b < 16; ++b) {
        const int64_t v = 16 * w0 + 32 * h + 16 * q + b;
        const bool there = v < s.nv && !(miss[16 * q + b] & 1u);
        word |= (there ? (byte[16 * q + b] >> shift) & 3u : 1u) << (2 * b);
      }
      out[2 * h + q] = in ? word : kAllMissing16;
    }
  }
  if (i < rows_pad)   // wp is a multiple of 4
    *reinterpret_cast<uint4*>(T + i * wp + w0) = make_uint4(out[0], out[1], out[2], out[3]);
}

int launch_sample_major_2bit(const Sel& s, uint32_t* T, int64_t rows_pad, int64_t wp,
                             hipStream_t st) {
  if (!s.idx) {
    const int64_t blocks = sample_major_job_blocks(rows_pad, wp);
    const int aligned = (int)rows_dword_aligned(s);
    if (blocks >= 256) {
      hipLaunchKernelGGL((k_sample_major_tiled<kSmTG, 256>), dim3((unsigned)blocks), dim3(256), 0,
                         st, s, T, rows_pad, wp, aligned);
    } else {
      const int64_t small = ceil_div(wp, kSmTW) * ceil_div(rows_pad, 16 * kSmTGSmall);
      hipLaunchKernelGGL((k_sample_major_tiled<kSmTGSmall, 128>), dim3((unsigned)small), dim3(128),
                         0, st, s, T, rows_pad, wp, aligned);
    }
    return check_launch("sample_major_tiled");
  }
  dim3 grid((unsigned)(ceil_div(rows_pad, kSmSamples) * ceil_div(wp, kSmWords)));
  hipLaunchKernelGGL(k_sample_major_2bit, grid, dim3(256), 0, st, s, T, rows_pad, wp);
  return check_launch("sample_major_2bit");
}

// ---- sample-major bit planes (IBS, popcount path) ---------------------------
__global__ __launch_bounds__(256) void k_ibs_planes(Sel s, uint32_t* __restrict__ P,
                                                    int64_t rows_pad, int64_t words_pad) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = g % rows_pad;
  const int64_t w = g / rows_pad;
  if (w >= words_pad) return;
  uint32_t hi = 0, lo = 0, nm = 0;
  for (int b = 0; b < 32; ++b) {
    const uint32_t c = code_at(s, w * 32 + b, i);
    hi |= (c >> 1) << b;
    lo |= (c & 1u) << b;
    nm |= (uint32_t)(c != 1u) << b;
  }
  P[(w * 3 + 0) * rows_pad + i] = hi;
  P[(w * 3 + 1) * rows_pad + i] = lo;
  P[(w * 3 + 2) * rows_pad + i] = nm;
}

int launch_ibs_planes(const Sel& s, uint32_t* P, int64_t rows_pad, int64_t words_pad,
                      hipStream_t st) {
  if (!s.idx) {
    hipLaunchKernelGGL(k_ibs_planes_fast, dim3(stride_grid(rows_pad / 16 * words_pad)), dim3(256),
                       0, st, s, P, rows_pad, words_pad, (int)rows_dword_aligned(s));
    return check_launch("ibs_planes_fast");
  }
  dim3 grid((unsigned)ceil_div(rows_pad * words_pad, 256));
  hipLaunchKernelGGL(k_ibs_planes, grid, dim3(256), 0, st, s, P, rows_pad, words_pad);
  return check_launch("ibs_planes");
}

// ---- variant-major 2-bit words with a sample list (LD) -----------------------
// One word per thread; the 16 list entries, then the 16 bytes, are loaded
// before any is used.
__global__ __launch_bounds__(256) void k_variant_major_2bit(Sel s, uint32_t* __restrict__ D,
                                                            int64_t rows_pad, int64_t wn) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t w = g % wn;
  const int64_t v = g / wn;
  if (v >= rows_pad) return;
  uint32_t word = kAllMissing16;
  if (v < s.nv && 16 * w < s.m) {
    const uint8_t* row = s.bed + (s.v0 + v) * s.bpv;
    int64_t k[16];
    uint32_t byte[16], miss[16];
#pragma unroll
    for (int b = 0; b < 16; ++b) k[b] = 16 * w + b < s.m ? (int64_t)s.idx[16 * w + b] : -1;
#pragma unroll
    for (int b = 0; b < 16; ++b) {
      byte[b] = row[k[b] >= 0 && k[b] < s.n ? k[b] >> 2 : 0];
      miss[b] = 0u;
    }
    if (s.mask) {
      const uint32_t* m = reinterpret_cast<const uint32_t*>(s.mask + (s.v0 + v) * s.wpm);
#pragma unroll
      for (int b = 0; b < 16; ++b)
        miss[b] = m[k[b] >= 0 && k[b] < s.n ? k[b] >> 5 : 0] >> (k[b] & 31);
    }
    word = 0;
#pragma unroll
    for (int b = 0; b < 16; ++b) {
      const bool there = k[b] >= 0 && k[b] < s.n && !(miss[b] & 1u);
      word |= (there ? (byte[b] >> (2 * (k[b] & 3))) & 3u : 1u) << (2 * b);
    }
  }
  D[v * wn + w] = word;
}

int launch_allele_counts(const Sel& s, uint32_t* D, int64_t wn, uint2* counts, hipStream_t st) {
  if (s.nv <= 0) return PG_OK;
  const dim3 grid((unsigned)ceil_div(s.nv, 4));
  if (!s.idx) {
    // ten words a lane where five do not cover a row
    hipLaunchKernelGGL((wn <= 320 ? k_allele_counts<false, 5> : k_allele_counts<false, 10>), grid,
                       dim3(256), 0, st, s, D, wn, (int)rows_dword_aligned(s), counts);
    return check_launch("allele_counts");
  }
  hipLaunchKernelGGL(k_variant_major_2bit, dim3((unsigned)ceil_div(s.nv * wn, 256)), dim3(256), 0,
                     st, s, D, s.nv, wn);
  int rc = check_launch("variant_major_2bit");
  if (rc != PG_OK) return rc;
  hipLaunchKernelGGL((k_allele_counts<true, 5>), grid, dim3(256), 0, st, s, D, wn, 0, counts);
  return check_launch("allele_counts");
}

// ---- LD operands: 2-bit words D and nibbles E ------------------------------------
// Sixteen codes to the fp4 nibbles of the LD tile (ld_nib_tile): homozygous A1
// 1001, heterozygous 0001, homozygous A2 0011, missing 0000; even codes in
// the first word, odd codes in the second.
__device__ __forceinline__ uint2 ld_nibbles(uint32_t w) {
  uint32_t n[2];
#pragma unroll
  for (int par = 0; par < 2; ++par) {
    const uint32_t lo = (w >> (2 * par)) & 0x11111111u, hi = (w >> (2 * par + 1)) & 0x11111111u;
    n[par] = (~(lo & ~hi) & 0x11111111u) | (lo & hi) << 1 | (~(lo | hi) & 0x11111111u) << 3;
  }
  return make_uint2(n[0], n[1]);
}

// D (rows_pad x wn words of 16 samples) and E: 64 variants x 64 samples in 512
// words, [half of the samples][variant][4 words], the steps of a 64-variant
// group in order.  A block takes 64 variants x 32 words: 128-byte runs of a
// row in, the same of D out, and whole 2 KB steps of E by way of LDS (a step's
// halves lie 260 words apart there, so the 16 a half-wave writes fall in
// different banks).  E and cn.part may be NULL.  cn.part: per block and variant
// the homozygous A2, homozygous A1 and missing calls of its 512 samples (padding
// counts as missing), 10 bits each, from the nibbles in LDS.  The blocks of a
// group also clear its rows of the emission scratch, the first one cn.any.
// kFromD: D is there already (a sample list's layout).
constexpr int kLyRows = 64, kLyWords = 32;

template <bool kFromD>
__device__ __forceinline__ void ld_layout_block(const Sel& s, uint32_t* __restrict__ D,
                                                uint32_t* __restrict__ E, int64_t rows_pad,
                                                int64_t wn, bool aligned, const LdScratch& sc,
                                                const LdCounts& cn, int64_t blk, uint32_t* s_e) {
  const int64_t nb_w = ceil_div(wn, kLyWords);
  const int64_t G = blk / nb_w, w0 = blk % nb_w * kLyWords;
  const int t = threadIdx.x, g = t & 31;
  const int64_t bits = kLyRows * sc.bm_words;
  for (int64_t i = blk % nb_w * 256 + t; i < bits; i += nb_w * 256) sc.bitmap[G * bits + i] = 0u;
  if (w0 == 0 && t < kLyRows) sc.rowcnt[G * kLyRows + t] = 0u;
  if (cn.any && blk == 0 && t < 3) cn.any[t] = 0u;
  int64_t vr[8], gr[8];
  uint32_t x[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    vr[u] = G * kLyRows + (t >> 5) + 8 * u;
    gr[u] = w0 + g;
  }
  if constexpr (kFromD) {
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = gr[u] < wn ? D[vr[u] * wn + gr[u]] : kAllMissing16;
  } else {
    row_words16(s, vr, gr, aligned, x);
  }
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    if (!kFromD && gr[u] < wn) D[vr[u] * wn + gr[u]] = x[u];
    const uint2 n = ld_nibbles(x[u]);
    uint32_t* d = &s_e[(g >> 1) * 260 + ((t >> 5) + 8 * u) * 4 + 2 * (g & 1)];
    d[0] = n.x;
    d[1] = n.y;
  }
  __syncthreads();
  const int64_t nsteps = wn / 4, step0 = w0 / 4;
  if (E) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int o = u * 256 + t;             // 16-byte piece: step o / 128 of the block's eight
      const int64_t step = step0 + (o >> 7);
      if (step < nsteps)
        *reinterpret_cast<uint4*>(E + (G * nsteps + step) * 512 + 4 * (o & 127)) =
            *reinterpret_cast<const uint4*>(&s_e[(o >> 6) * 260 + 4 * (o & 63)]);
    }
  }
  if (!cn.part) return;
  // a quarter of a variant's samples per thread (a wave: 64 variants)
  uint32_t n3 = 0, n0 = 0, called = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint4 q = *reinterpret_cast<const uint4*>(&s_e[(4 * (t >> 6) + u) * 260 + 4 * (t & 63)]);
    const uint32_t n[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      n3 += __popc(n[e] & 0x22222222u);
      n0 += __popc(n[e] & 0x88888888u);
      called += __popc(n[e] & 0x11111111u);
    }
  }
  __syncthreads();
  s_e[t] = n3 | n0 << 10 | (128 - called) << 20;
  __syncthreads();
  if (t < kLyRows) {
    const int64_t words = wn - w0 < kLyWords ? wn - w0 : kLyWords;   // those past wn: missing
    cn.part[w0 / kLyWords * rows_pad + G * kLyRows + t] =
        s_e[t] + s_e[64 + t] + s_e[128 + t] + s_e[192 + t] -
        ((uint32_t)(16 * (kLyWords - words)) << 20);
  }
}

template <bool kFromD>
__global__ __launch_bounds__(256) void k_ld_layout(Sel s, uint32_t* __restrict__ D,
                                                   uint32_t* __restrict__ E, int64_t rows_pad,
                                                   int64_t wn, int aligned, LdScratch sc,
                                                   LdCounts cn) {
  __shared__ __attribute__((aligned(16))) uint32_t s_e[16 * 260];
  ld_layout_block<kFromD>(s, D, E, rows_pad, wn, aligned != 0, sc, cn,
                          xcd_swizzle(blockIdx.x, gridDim.x), s_e);
}

// Many problems in one launch, as k_sample_major_jobs.
__global__ __launch_bounds__(256) void k_ld_layout_jobs(const LdLayoutJob* __restrict__ jobs,
                                                        int n_jobs) {
  __shared__ __attribute__((aligned(16))) uint32_t s_e[16 * 260];
  const int64_t b = blockIdx.x;
  int lo = 0, hi = n_jobs - 1;
  while (lo < hi) {   // the last job with block_begin <= b
    const int mid = (lo + hi + 1) / 2;
    if (jobs[mid].block_begin <= b) lo = mid; else hi = mid - 1;
  }
  const LdLayoutJob j = jobs[lo];
  ld_layout_block<false>(j.s, j.D, j.E, 0, j.wn, j.aligned != 0, j.sc, LdCounts{}, b - j.block_begin,
                         s_e);
}

int64_t ld_layout_blocks(int64_t rows_pad, int64_t wn) {
  return rows_pad / kLyRows * ceil_div(wn, kLyWords);
}

int launch_ld_layout_jobs(const LdLayoutJob* jobs, int n_jobs, int64_t total_blocks,
                          hipStream_t st) {
  if (n_jobs <= 0 || total_blocks <= 0) return PG_OK;
  hipLaunchKernelGGL(k_ld_layout_jobs, dim3((unsigned)total_blocks), dim3(256), 0, st, jobs,
                     n_jobs);
  return check_launch("ld_layout_jobs");
}

int launch_ld_layout(const Sel& s, uint32_t* D, uint32_t* E, int64_t rows_pad, int64_t wn,
                     const LdScratch& sc, const LdCounts& cn, hipStream_t st) {
  const dim3 grid((unsigned)ld_layout_blocks(rows_pad, wn));
  if (!s.idx) {
    hipLaunchKernelGGL(k_ld_layout<false>, grid, dim3(256), 0, st, s, D, E, rows_pad, wn,
                       (int)rows_dword_aligned(s), sc, cn);
    return check_launch("ld_layout");
  }
  hipLaunchKernelGGL(k_variant_major_2bit, dim3((unsigned)ceil_div(rows_pad * wn, 256)), dim3(256),
                     0, st, s, D, rows_pad, wn);
  int rc = check_launch("variant_major_2bit");
  if (rc != PG_OK) return rc;
  if (!E && !cn.part) return ld_clear(sc, rows_pad, st);
  hipLaunchKernelGGL(k_ld_layout<true>, grid, dim3(256), 0, st, s, D, E, rows_pad, wn, 0, sc,
                     cn);
  return check_launch("ld_layout");
}

// LD bit planes without a sample list, staged through LDS: a block owns 64
// variants x 32 plane words (1,024 samples).  Lanes read consecutive dwords of
// one variant row (coalesced), the three 16-bit half-planes of each dword go
// to LDS, and lanes then write consecutive variants of one plane word
// (coalesced).
__global__ __launch_bounds__(256) void k_ld_planes_tiled(Sel s, uint32_t* __restrict__ P,
                                                         int64_t rows_pad, int64_t words_pad,
                                                         int aligned) {
  __shared__ uint16_t half[3][64][65];
  const int t = threadIdx.x;
  const int64_t nrb = rows_pad / 64;
  const int64_t v0 = ((int64_t)blockIdx.x % nrb) * 64;
  const int64_t w0 = ((int64_t)blockIdx.x / nrb) * 32;      // first plane word
  const int d = t & 63;                                      // 16-sample group in the block
#pragma unroll 1
  for (int k0 = 0; k0 < 16; k0 += 8) {
    int64_t vr[8], gr[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) { vr[k] = v0 + (t >> 6) + 4 * (k0 + k); gr[k] = 2 * w0 + d; }
    uint32_t xs[8];
    row_words16(s, vr, gr, aligned != 0, xs);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int row = (t >> 6) + 4 * (k0 + k);
      const uint32_t lo = xs[k] & 0x55555555u, hi = (xs[k] >> 1) & 0x55555555u;
      half[0][row][d] = (uint16_t)compact_even_bits(lo & hi);
      half[1][row][d] = (uint16_t)compact_even_bits(~(lo | hi) & 0x55555555u);
      half[2][row][d] = (uint16_t)compact_even_bits(~(lo & ~hi) & 0x55555555u);
    }
  }
  __syncthreads();
#pragma unroll 4
  for (int k = 0; k < 24; ++k) {
    const int e = t + 256 * k;
    const int row = e & 63;
    const int pw = e >> 6;                                   // 0..95
    const int p = pw % 3, w = pw / 3;
    if (w0 + w < words_pad)
      P[((w0 + w) * 3 + p) * rows_pad + v0 + row] =
          (uint32_t)half[p][row][2 * w] | ((uint32_t)half[p][row][2 * w + 1] << 16);
  }
}

int launch_ld_planes(const Sel& s, uint32_t* P, int64_t rows_pad, int64_t words_pad,
                     hipStream_t st) {
  if (!s.idx) {
    const int64_t blocks = (rows_pad / 64) * ceil_div(words_pad, 32);
    hipLaunchKernelGGL(k_ld_planes_tiled, dim3((unsigned)blocks), dim3(256), 0, st, s, P, rows_pad,
                       words_pad, (int)rows_dword_aligned(s));
  } else {
    hipLaunchKernelGGL(k_ld_planes, dim3(stride_grid(rows_pad * words_pad)), dim3(256), 0, st, s,
                       P, rows_pad, words_pad);
  }
  return check_launch("ld_planes");
}

int launch_sample_major_rep(const Sel& s, uint32_t* R, int64_t rows_pad, int64_t rp,
                            hipStream_t st) {
  if (!s.idx) {
    hipLaunchKernelGGL(k_sample_major_rep, dim3(stride_grid(rows_pad / 16 * (rp / 16))), dim3(256),
                       0, st, s, R, rows_pad, rp, (int)rows_dword_aligned(s));
  } else {
    hipLaunchKernelGGL(k_sample_major_rep_gather, dim3(stride_grid(rows_pad * (rp / 2))), dim3(256),
                       0, st, s, R, rows_pad, rp);
  }
  return check_launch("sample_major_rep");
}

}  // namespace pg
