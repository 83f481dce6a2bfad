// Relationship matrix on the int8 matrix cores, by an exact fixed-point split.
//
// With x in {0, 1, 2} the count of the marker's minor allele, m = 1 for a
// call (a missing one has x = m = 0), p the minor allele frequency and
// w = 1 / (2p(1-p)), the numerator of a pair is
//   S[i,j] = sum_v w (x_i - 2p m_i)(x_j - 2p m_j)
//          = sum_v x_i F1(j) + m_i F2(j),
//   F1 = w (x_j - 2p) m_j,   F2 = -2p w (x_j - 2p) m_j.
// The factors of sample i are small integers, those of sample j are one of
// three rationals per marker.  Each is rounded once, from the exact rational,
// to a multiple of 2^-53 and written in balanced base-256 digits, so S is a
// sum over digit places of int8 products with int32 sums, all exact (Ozaki's
// splitting of a product, one factor being small integers already):
//   S = 2^-53 sum_s 256^s (sum_v x_i F1_s(j) + m_i F2_s(j)).
// |F2| <= 2 takes 7 digits; |F1| <= 1/p takes 8 down to p = 1/1019, and 7, 9
// or 10 where the panel's smallest p asks for it.  The only roundings are
// the one per marker and class (half of 2^-53) and the few that add the digit
// places at the end, against one per marker in a double sum.  Measured against
// extended precision over 100 to 2,500 samples x 1,000 to 40,000 variants:
// relative error 0.7-2.6e-16, the fp64 kernel's 2.9e-16 to 3.3e-15.
//
// Half of 2^-53 is too much for an increment that is small itself: two common
// homozygotes' is 2p/(1-p), two heterozygotes' (1-2p)^2/(2p(1-p)), and equal
// markers round alike.  So the markers of a chunk of 64 that holds one with
// p < 1/512 are rounded to multiples of 2^-77, in three more digits of each
// factor (a pass over the listed chunks alone); and where 15 of 16 markers have
// an increment below 1/8 (p < 1/16, or 1 - 2p < 1/8) every chunk's are, to 2^-77,
// 2^-69 or 2^-85, in the ordinary passes.  The line: sums of equal increments at p
// of 1/512 to 1/256, relative error at most 1.3e-14 (rms 6e-15) here, the fp64
// product's rms 1.2e-14 over 800 to 2,000 markers.  10,000 samples x 1,000 alleles
// seen once, a pair without one: 3.2e-13 without these digits, 4e-17 with them,
// the fp64 kernel 6.1e-15.  10,000 x 71,307, all p from 0.0005 to 0.005: 47.8 ms a
// call, p from 0.001 to 0.5 57.7, from 0.01 on 40.0; 1,000 x 76,124 1.07, 0.91 from
// 0.01 on (the fp64 kernel 130 and 1.65).
//
// 16 products of 2 operations at the int8 rate replace one fp64 product at
// 1/64 of it: 10,000 x 71,307 130 -> 40.4 ms, 1,000 x 76,124 1.65 -> 0.80 ms.
// The operand is never expanded in memory: the 2-bit codes of 64
// markers of a 32-sample block are 512 contiguous bytes (G), rows expand to x
// and m in registers, and the digits of the block's columns are selected from
// the markers' tables into LDS once for all its waves.
#include "grm_int.h"

namespace pg {

typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v16i_t __attribute__((ext_vector_type(16)));

constexpr int kGiChunk = 64;                  // variants per chunk
constexpr int kGiBlockWords = 128;            // words of G per 32 samples and chunk
constexpr int kGiSeg = 128;                   // rows per counting segment
constexpr int kGiQuadWords = 20;              // table words per four variants (18 used)
constexpr int kGiTabWords = 16 * kGiQuadWords;   // table words per chunk and pass
constexpr int kGiListedSlot = 4;              // the listed chunks' low places among the
                                              // tables (of passes 0-4)

// What k_gi_stats finds over all markers.
struct GiPanel {
  unsigned long long counts;   // markers with defined increments; << 32 those of
                               // them with an increment below 1/8
  uint32_t top;                // largest ceil(n / a)
};

// The digit places of a panel: F1's and F2's, `low` of them below 2^-53 in every
// chunk; the count of pairs takes the place after F1's.  |F1| 2^53 < 0.498 *
// 256^digits for n/a (alleles over minor alleles) up to top.  A panel that takes
// its low places in every chunk takes so many that the last pass of three
// places is filled (11 and 1 places in four passes, or 14 and 1 in five).
struct GiPlaces {
  int n1, n2, low, passes;
};
__device__ __forceinline__ GiPlaces gi_places(const GiPanel& p) {
  const uint64_t used = p.counts & 0xFFFFFFFFu, coarse = p.counts >> 32;
  const bool all = coarse > 0 && 16 * coarse >= 15 * used;
  const int n1 = p.top <= 3u && !all ? 7 : p.top <= 1019u ? 8 : p.top <= 261000u ? 9 : 10;
  const int low = !all ? 0 : n1 < 10 ? 11 - n1 : 4;
  return GiPlaces{n1 + low, 7 + low, low, (n1 + low + 3) / 3};
}

// ---- per-marker counts ------------------------------------------------------
// One thread per word column of T and 128 rows: the calls, heterozygotes and
// homozygous A2 of its 16 variants (each at most 128), packed in bytes 0-2 of
// cnt[seg * nv_pad + v].  Counters of three rows share 2-bit fields, then
// byte fields.
__global__ __launch_bounds__(256) void k_gi_counts(const uint32_t* __restrict__ T, int64_t wp,
                                                   uint32_t* __restrict__ cnt,
                                                   GiPanel* __restrict__ panel,
                                                   uint32_t* __restrict__ fine) {
  const int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x, seg = blockIdx.y;
  if (w == 0 && seg == 0) *panel = GiPanel{0ull, 0u};
  if (seg == 0 && w < ceil_div(wp / 4, 32)) fine[w] = 0u;
  if (w >= wp) return;
  const uint32_t* src = T + seg * kGiSeg * wp + w;
  uint32_t c8[3][4] = {};
  for (int r0 = 0; r0 < kGiSeg; r0 += 12) {
    uint32_t x[12];
#pragma unroll
    for (int r = 0; r < 12; ++r)
      x[r] = r0 + r < kGiSeg ? src[(int64_t)(r0 + r) * wp] : kAllMissing16;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint32_t f[3] = {0, 0, 0};
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        uint32_t a2, a1, m;
        masks_of_word(x[3 * g + r], a2, a1, m);
        f[0] += m;
        f[1] += m & ~(a1 | a2);
        f[2] += a2;
      }
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) c8[k][e] += (f[k] >> (2 * e)) & 0x03030303u;
    }
  }
  uint4* out = reinterpret_cast<uint4*>(cnt + (seg * wp + w) * 16);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    uint32_t v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = ((c8[0][e] >> (8 * b)) & 0xFFu) | ((c8[1][e] >> (8 * b)) & 0xFFu) << 8 |
             ((c8[2][e] >> (8 * b)) & 0xFFu) << 16;
    out[b] = make_uint4(v[0], v[1], v[2], v[3]);
  }
}

// Per variant: {alleles n = 2 calls, minor alleles a}, a = 0 for an undefined
// marker; per 16 variants a word with the undefined ones in the low half and
// those whose minor allele is A1 in the high half; the panel's figures; and a
// bit per chunk (a wave's variants) that holds a rare allele (p < 1/512).
__global__ __launch_bounds__(256) void k_gi_stats(const uint32_t* __restrict__ cnt, int64_t nv_pad,
                                                  int segs, uint2* __restrict__ stat,
                                                  uint32_t* __restrict__ marks,
                                                  GiPanel* __restrict__ panel,
                                                  uint32_t* __restrict__ fine) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool in = v < nv_pad;
  uint32_t calls = 0, het = 0, h2 = 0;
  if (in)
    for (int s = 0; s < segs; ++s) {
      const uint32_t c = cnt[s * nv_pad + v];
      calls += c & 0xFFu;
      het += (c >> 8) & 0xFFu;
      h2 += c >> 16;
    }
  const uint32_t n = 2 * calls, a2 = het + 2 * h2;
  const bool used = a2 > 0 && a2 < n, flip = used && a2 > calls;
  const uint32_t a = !used ? 0u : flip ? n - a2 : a2;
  if (in) stat[v] = make_uint2(n, a);
  const uint64_t undef = __ballot(!used), flips = __ballot(flip);
  const int lane = threadIdx.x & 63;
  if (in && (lane & 15) == 0)
    marks[v >> 4] = (uint32_t)(undef >> lane & 0xFFFFu) | (uint32_t)(flips >> lane & 0xFFFFu) << 16;
  uint32_t r = used ? (n + a - 1) / a : 0u;
  for (int d = 32; d > 0; d >>= 1) {
    const uint32_t o = __shfl_xor(r, d, 64);
    r = o > r ? o : r;
  }
  const uint64_t rare = __ballot(used && 512 * a < n);
  const uint64_t coarse = __ballot(used && (16 * a < n || (2 * a < n && 8 * (n - 2 * a) < n)));
  __shared__ uint32_t s_n[2];
  if (threadIdx.x < 2) s_n[threadIdx.x] = 0u;
  __syncthreads();
  if (lane == 0) {
    // few waves raise it: most see a larger one and leave it
    if (r > __hip_atomic_load(&panel->top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&panel->top, r);
    if (rare) atomicOr(&fine[v >> 11], 1u << (v >> 6 & 31));
    atomicAdd(&s_n[0], (uint32_t)__popcll(~undef));
    atomicAdd(&s_n[1], (uint32_t)__popcll(coarse));
  }
  __syncthreads();
  // one addition per block: additions to one word queue up
  if (threadIdx.x == 0) atomicAdd(&panel->counts, (unsigned long long)s_n[1] << 32 | s_n[0]);
}

// ---- digit tables --------------------------------------------------------------
// num / den (den < 2^63, num / den < 2^22) times 2^bits, rounded to nearest, as
// a 128-bit two's complement pair, negated if `neg`.
__device__ __forceinline__ void gi_fixed(uint64_t num, uint64_t den, int bits, bool neg,
                                         uint64_t& lo, uint64_t& hi) {
  uint64_t r = num % den;
  lo = num / den;
  hi = 0;
  for (int b = 0; b < bits; ++b) {
    r <<= 1;
    hi = hi << 1 | lo >> 63;
    lo <<= 1;
    if (r >= den) {
      r -= den;
      lo |= 1;
    }
  }
  if ((r << 1) >= den) {
    ++lo;
    if (lo == 0) ++hi;
  }
  if (neg) {
    lo = ~lo + 1;
    hi = ~hi + (lo == 0);
  }
}

// Takes the lowest balanced digit off a 128-bit value.
__device__ __forceinline__ int gi_digit(uint64_t& lo, uint64_t& hi) {
  const int d = (int)(int8_t)(lo & 0xFFu);
  const bool up = d < 0;                  // the value minus d: add |d|
  lo = lo >> 8 | hi << 56;
  hi = (uint64_t)((int64_t)hi >> 8);
  if (up && ++lo == 0) ++hi;
  return d;
}

// tab[((pass * nch + chunk) * 16 + quad) * 20 + plane * 3 + class]: byte b is
// the digit of variant 16 * word + 4 b + e of the chunk (quad = 4 * word + e)
// for a column call of class x = 0, 1, 2.  Pass t holds the digit places
// 3t .. 3t + 2: planes 0-2 those of F1 (rows enter with x), 3-5 those of F2
// (rows enter with m), where the place after F1's last holds the count of
// pairs (1 in every class).  Pass kGiListedSlot holds three places below 2^-53
// for the chunks that are listed in `fine`, where not every chunk has them.
__global__ __launch_bounds__(256) void k_gi_tables(const uint2* __restrict__ stat, int64_t nch,
                                                   const GiPanel* __restrict__ panel,
                                                   const uint32_t* __restrict__ fine,
                                                   uint32_t* __restrict__ tab) {
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  // four neighbouring lanes hold the four variants of a quad; a row of blocks
  // per factor and class, k
  const int b = (int)(id & 3), quad = (int)(id >> 2 & 15), k = blockIdx.y;
  const int64_t c = id >> 6;
  if (c >= nch) return;
  const uint2 s = stat[c * kGiChunk + 16 * (quad >> 2) + 4 * b + (quad & 3)];
  const uint64_t n = s.x, a = s.y;
  const GiPlaces at = gi_places(*panel);
  const bool listed = at.low == 0 && (fine[c >> 5] >> (c & 31) & 1u);   // the wave's chunk
  uint64_t lo = 0, hi = 0;
  if (a) {
    const uint64_t z = n - a, h = n - 2 * a;      // a <= n / 2
    const uint64_t num = k == 1 ? n * h : k == 3 ? 2 * a : k == 4 ? h : k == 5 ? 2 : n;
    const uint64_t den = k == 1 ? 2 * a * z : k == 2 ? a : k == 5 ? 1 : z;
    // F1: -1/(1-p), (1-2p)/(2p(1-p)), 1/p; F2: 2p/(1-p), -(1-2p)/(1-p), -2
    gi_fixed(num, den, 53 + (listed ? 24 : 8 * at.low), k == 0 || k >= 4, lo, hi);
  }
  const int digits = k < 3 ? at.n1 : at.n2;
  for (int t = listed ? -1 : 0; t < at.passes; ++t) {
    uint32_t* out = tab + (((t < 0 ? kGiListedSlot : t) * nch + c) * 16 + quad) * kGiQuadWords;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int place = 3 * t + q;
      const int d = place < digits ? gi_digit(lo, hi) : a && k >= 3 && place == at.n1 ? 1 : 0;
      uint32_t x = (uint32_t)d & 0xFFu;
      x |= __shfl_xor(x, 1, 64) << 8;
      x |= __shfl_xor(x, 2, 64) << 16;
      if (b == 0) out[(k / 3 * 3 + q) * 3 + k % 3] = x;
    }
    if (b == 0 && k == 0) out[18] = out[19] = 0u;
  }
}

// ---- operand --------------------------------------------------------------------
// G: the codes of T with the minor allele counted (homozygotes swapped where
// A1 is the minor one) and undefined markers missing, in blocks of 32 samples
// x 64 variants: word [half][sample][s] holds word 2 * half + s of the chunk.
// A block of 256 threads moves 32 samples x 16 chunks through LDS: 256-byte
// runs of T in, 512-byte runs of G out.
__global__ __launch_bounds__(256) void k_gi_operand(const uint32_t* __restrict__ T, int64_t rows,
                                                    int64_t wp, const uint32_t* __restrict__ marks,
                                                    uint32_t* __restrict__ G) {
  __shared__ uint32_t s[32][65];
  const int tid = threadIdx.x;
  const int64_t rb = blockIdx.y, w0 = (int64_t)blockIdx.x * 64;
  const int64_t w = w0 + (tid & 63);
  uint32_t undef = 0x55555555u, flip = 0u;
  if (w < wp) {
    auto spread = [](uint32_t x) {   // 16 bits to the even bits of 32
      x = (x | x << 8) & 0x00FF00FFu;
      x = (x | x << 4) & 0x0F0F0F0Fu;
      x = (x | x << 2) & 0x33333333u;
      return (x | x << 1) & 0x55555555u;
    };
    undef = spread(marks[w] & 0xFFFFu);
    flip = spread(marks[w] >> 16);
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int row = r * 4 + (tid >> 6);
    const int64_t i = rb * 32 + row;
    uint32_t x = w < wp && i < rows ? T[i * wp + w] : kAllMissing16;
    const uint32_t hom = ~(x ^ x >> 1) & flip;
    x ^= hom | hom << 1;
    x = (x & ~(undef | undef << 1)) | undef;
    s[row][tid & 63] = x;
  }
  __syncthreads();
  const int64_t nch = wp / 4;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int o = r * 256 + tid, ch = o >> 7, in = o & 127;
    const int64_t c = w0 / 4 + ch;
    if (c < nch)
      G[(rb * nch + c) * kGiBlockWords + in] =
          s[(in >> 1) & 31][4 * ch + 2 * (in >> 6) + (in & 1)];
  }
}

// ---- the pair kernel ---------------------------------------------------------------
__device__ __forceinline__ uint32_t gi_perm(uint32_t table, uint32_t sel) {
  return __builtin_amdgcn_perm(table, table, sel);
}

// Tile t of the upper triangle: rows [128 NR I, ..), columns [128 / NR J, ..).
template <int NR>
__host__ __device__ inline void gi_tile(int64_t t, int64_t nj, int64_t& I, int64_t& J) {
  constexpr int64_t k = NR * NR;   // column strips per row tile
  I = 0;
  while (t >= nj - k * I) {
    t -= nj - k * I;
    ++I;
  }
  J = k * I + t;
}

template <int NR>
static int64_t gi_tiles(int64_t m, int64_t& ni, int64_t& nj) {
  constexpr int64_t k = NR * NR;
  ni = ceil_div(m, 128 * NR);
  nj = ceil_div(m, 128 / NR);
  return ni * nj - k * ni * (ni - 1) / 2;
}

struct GiOut {
  double* grm;
  uint32_t* n;
  int64_t m;
  int full;
  int64_t nj;
  // tiles [0, head) whole, then `tail` tiles in n_split ranges of cps chunks
  int64_t head, tail, n_split, cps;
  double* part_s;         // 16,384 sums and counts per range and tail tile
  uint32_t* part_n;
};

// A finished entry i <= j: S / N (NaN without a marker), and its mirror.
__device__ __forceinline__ void gi_store(const GiOut& o, int64_t i, int64_t j, double S,
                                         uint32_t n) {
  const double v = n ? __ddiv_rn(S, (double)n) : __longlong_as_double(0x7ff8000000000000ll);
  if (o.full) {
    o.grm[i * o.m + j] = v;
    o.n[i * o.m + j] = n;
    if (i != j) {
      o.grm[j * o.m + i] = v;
      o.n[j * o.m + i] = n;
    }
  } else if (i < j) {
    const int64_t e = i * o.m - i * (i + 1) / 2 + (j - i - 1);
    o.grm[e] = v;
    o.n[e] = n;
  }
}

// One pass's share S of entry (i, j), `n` its count with the last pass: parked
// in the outputs (or the range's partial sums) until then.
__device__ __forceinline__ void gi_put(const GiOut& o, bool begin, bool end, int64_t park,
                                       int64_t i, int64_t j, double S, uint32_t n) {
  if (park >= 0) {
    if (!begin) S += o.part_s[park];
    o.part_s[park] = S;
    if (end) o.part_n[park] = n;
  } else if (j < o.m && i <= j && (o.full || i < j)) {
    double* at = o.full ? &o.grm[i * o.m + j] : &o.grm[i * o.m - i * (i + 1) / 2 + (j - i - 1)];
    if (!begin) S += *at;
    if (end)
      gi_store(o, i, j, S, n);
    else
      *at = S;
  }
}

// Block: four waves, NR along the rows and 4 / NR along the columns, each
// with 128 rows x 32 columns: 4 blocks of v_mfma_i32_32x32x32_i8 x 3 digit
// places = 192 accumulator registers, so that two waves share a SIMD.  Per
// chunk of 64 variants a wave expands its rows' codes (2 K steps x 4 blocks x
// 15 instructions) for up to 48 MFMAs, and generates a quarter of the digits
// of the block's columns for the next chunk (28 instructions per strip).
// Codes and tables come to LDS by direct loads, two chunks ahead of their
// use (the accumulators leave no registers to hold them); the barrier of a
// chunk leaves the newest three loads of each wave in flight.
// kPlanes: the planes of the pass that are not zero.
//
// Bound: the matrix cores, busy 64% of the cycles at the 2.07 GHz the chip
// holds under this load (10,000 x 71,307); 4.6 other vector instructions per
// MFMA.  Steps on the way, at that size: codes and tables through registers
// 57.0 ms (the compiler moves the loads to their uses); direct loads to LDS
// and one table read for both columns 45.6; two chunks ahead, and the last
// round's tiles split, 41.9.  Raised wave priority around the MFMAs: no change.
template <int NR>
struct GiLds {
  static constexpr int kStrips = 4 / NR;
  uint32_t dig[2][kStrips][6][512];              // digits of the columns
  uint32_t rows[3][4][4 * kGiBlockWords];        // each wave's row codes
  // tables, then the columns' codes
  uint32_t stage[3][kGiTabWords + kStrips * kGiBlockWords];
};

// Lane l's 16 bytes at `src` to LDS `dst` + 16 l (dst uniform over the wave).
__device__ __forceinline__ void gi_to_lds(const uint32_t* src, uint32_t* dst) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)src,
      (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

// The first chunk from c on that has its bit in `fine` set, c_end if none.
__device__ __forceinline__ int gi_next(const uint32_t* __restrict__ fine, int c, int c_end) {
  while (c < c_end) {
    const uint32_t w = fine[c >> 5] >> (c & 31);
    if (w) {
      c += __builtin_ctz(w);
      break;
    }
    c = (c | 31) + 1;
  }
  return c < c_end ? c : c_end;
}

// Chunks [c_begin, c_end), or (kListed, fine not NULL) those of them with a bit
// in `fine`, at least one.
template <int NR, int kPlanes, bool kListed>
__device__ __forceinline__ void gi_pass(const uint32_t* __restrict__ G,
                                        const uint32_t* __restrict__ tab, int64_t nch, int64_t I,
                                        int64_t J, int c_begin, int c_end, GiLds<NR>& s,
                                        v16i_t (&acc)[3][4],
                                        const uint32_t* __restrict__ fine) {
  constexpr int kStrips = 4 / NR;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave % NR, ws = wave / NR;
  const int e = lane & 3, col16 = lane >> 2;
  // row blocks in pairs: 64 lanes x 16 bytes
  const uint32_t* rsrc = G + ((I * 4 * NR + wr * 4 + (lane >> 5)) * nch) * kGiBlockWords +
                         4 * (lane & 31);
  // staged per chunk: 320 words of tables and 128 per strip, 4 a lane, a
  // quarter of them by each wave
  constexpr int kStage = (kGiTabWords + kStrips * kGiBlockWords) / 16;
  const int at = wave * kStage + lane;
  const uint32_t* ssrc = tab + 4 * at;
  int64_t sstep = kGiTabWords;
  if (at >= kGiTabWords / 4) {
    const int q = at - kGiTabWords / 4;
    ssrc = G + ((J * kStrips + q / 32) * nch) * kGiBlockWords + 4 * (q % 32);
    sstep = kGiBlockWords;
  }
  auto load_rows = [&](int c, int buf) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
      gi_to_lds(rsrc + (2 * a * nch + c) * kGiBlockWords, &s.rows[buf][wave][256 * a]);
  };
  auto load_stage = [&](int c, int buf) {
    if (lane < kStage) gi_to_lds(ssrc + c * sstep, &s.stage[buf][4 * kStage * wave]);
  };
  // digits of word `wave` of the chunk for columns col16 and col16 + 16
  auto generate = [&](int buf, int dbuf) {
    uint4 t4[5];
    uint32_t w[kStrips][2];
#pragma unroll
    for (int k = 0; k < 5; ++k)
      t4[k] = reinterpret_cast<const uint4*>(&s.stage[buf][(wave * 4 + e) * kGiQuadWords])[k];
#pragma unroll
    for (int q = 0; q < kStrips; ++q)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        w[q][u] = s.stage[buf][kGiTabWords + q * kGiBlockWords + (wave >> 1) * 64 +
                               2 * (col16 + 16 * u) + (wave & 1)];
    const uint32_t t[18] = {t4[0].x, t4[0].y, t4[0].z, t4[0].w, t4[1].x, t4[1].y,
                            t4[1].z, t4[1].w, t4[2].x, t4[2].y, t4[2].z, t4[2].w,
                            t4[3].x, t4[3].y, t4[3].z, t4[3].w, t4[4].x, t4[4].y};
#pragma unroll
    for (int q = 0; q < kStrips; ++q)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t sel = (w[q][u] >> (2 * e)) & 0x03030303u;
        const uint32_t m0 = gi_perm(0x000000FFu, sel), m1 = gi_perm(0x00FF0000u, sel),
                       m2 = gi_perm(0xFF000000u, sel);
        uint32_t* out = &s.dig[dbuf][q][0][(wave & 1) * 256 + (wave >> 1) * 128 +
                                          (col16 + 16 * u) * 4 + e];
#pragma unroll
        for (int p = 0; p < 6; ++p)
          if (kPlanes >> p & 1)
            out[p * 512] = (t[3 * p] & m0) | (t[3 * p + 1] & m1) | (t[3 * p + 2] & m2);
      }
  };

  // the chunks after c, the last one again past the end
  auto after = [&](int c) {
    const int n = kListed && fine ? gi_next(fine, c + 1, c_end) : c + 1;
    return n < c_end ? n : c;
  };
  int c = kListed && fine ? gi_next(fine, c_begin, c_end) : c_begin;
  int c1 = after(c), c2 = after(c1);
  load_stage(c, 0);
  load_rows(c, 0);
  load_stage(c1, 1);
  load_stage(c2, 2);
  load_rows(c1, 1);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  generate(0, 0);
  __syncthreads();
  int b0 = 0, b1 = 1, b2 = 2;   // buffers of chunks c, c1, c2
  int buf = 0;
  while (true) {
    const int c3 = after(c2);
    load_rows(c2, b2);
    load_stage(c3, b0);   // chunk c's were used a chunk ago
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v4i_t dig[6];
#pragma unroll
      for (int p = 0; p < 6; ++p)
        if (kPlanes >> p & 1)
          dig[p] = *reinterpret_cast<const v4i_t*>(&s.dig[buf][ws][p][h * 256 + lane * 4]);
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const uint32_t w = s.rows[b0][wave][a * kGiBlockWords + 2 * lane + h];
        v4i_t x, m;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t sel = (w >> (2 * q)) & 0x03030303u;
          x[q] = (int)gi_perm(0x02010000u, sel);
          m[q] = (int)gi_perm(0x01010001u, sel);
        }
#pragma unroll
        for (int p = 0; p < 6; ++p)
          if (kPlanes >> p & 1)
            acc[p % 3][a] = __builtin_amdgcn_mfma_i32_32x32x32_i8(p < 3 ? x : m, dig[p],
                                                                  acc[p % 3][a], 0, 0, 0);
      }
    }
    generate(b1, buf ^ 1);
    // rows of the next chunk and tables of the one after have arrived
    asm volatile("s_waitcnt vmcnt(3) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const int b = b0;
    b0 = b1;
    b1 = b2;
    b2 = b;
    if (c1 == c) break;
    c = c1;
    c1 = c2;
    c2 = c3;
    buf ^= 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int NR>
__global__ __launch_bounds__(256, 2) void k_gi_pairs(const uint32_t* __restrict__ G,
                                                     const uint32_t* __restrict__ tab,
                                                     const GiPanel* __restrict__ panel,
                                                     const uint32_t* __restrict__ fine,
                                                     int64_t nch, GiOut o) {
  // the operands, or the sums on their way out (12 KB per wave)
  __shared__ __align__(16) union {
    GiLds<NR> in;
    uint4 out[4 * 768];
  } s;
  // each XCD takes a contiguous run of tiles: neighbours share their rows
  const int64_t item = blockIdx.x, tail_item = item - o.head;
  const bool whole = item < o.head;
  const int64_t tile = whole ? xcd_swizzle(item, o.head) : o.head + tail_item % o.tail;
  const int64_t split = whole ? 0 : tail_item / o.tail;
  int64_t I, J;
  gi_tile<NR>(tile, o.nj, I, J);
  const GiPlaces at = gi_places(*panel);
  const int c_begin = whole ? 0 : (int)(split * o.cps);
  const int c_end = whole || (split + 1) * o.cps > nch ? (int)nch : (int)((split + 1) * o.cps);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rb = (wave % NR) * 128 + 4 * (lane >> 5), cb = (wave / NR) * 32 + (lane & 31);
  // pass -1: the low places of the listed chunks
  const int t0 = at.low == 0 && gi_next(fine, c_begin, c_end) < c_end ? -1 : 0;
  for (int t = t0; t < at.passes; ++t) {
    v16i_t acc[3][4];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int a = 0; a < 4; ++a) acc[q][a] = (v16i_t){0};
    const uint32_t* tt = tab + (int64_t)(t < 0 ? kGiListedSlot : t) * nch * kGiTabWords;
    const bool end = t == at.passes - 1;
    // the last of the usual eight places (and of eleven): F1 and F2 at the first,
    // F1 at the second, the count at the third
    if (end && at.n1 % 3 == 2)
      gi_pass<NR, 0x2B, false>(G, tt, nch, I, J, c_begin, c_end, s.in, acc, nullptr);
    else
      gi_pass<NR, 0x3F, true>(G, tt, nch, I, J, c_begin, c_end, s.in, acc,
                              t < 0 ? fine : nullptr);
    // the places' sum is below 2^48 in magnitude: exact in double; the
    // passes before are read back from where they were parked
    const int count_at = at.n1 - 3 * t;
    const double scale =
        __longlong_as_double((int64_t)(1023 - 53 - 8 * at.low + 24 * t) << 52);
    const double s0 = count_at > 0 ? scale : 0.0, s1 = count_at > 1 ? 256.0 * scale : 0.0,
                 s2 = count_at > 2 ? 65536.0 * scale : 0.0;
    const int64_t park =
        whole || o.n_split == 1 ? -((int64_t)1 << 60) : tail_item * 16384 + cb;
    const int64_t j = J * (128 / NR) + cb;
    // each lane's sums go through LDS so that the code that stores them is a
    // loop (unrolled 64 times over registers it spills)
    __syncthreads();
    uint4* mine = s.out + wave * 768 + lane;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          mine[(q * 4 + g) * 64] =
              make_uint4((uint32_t)acc[q][a][4 * g], (uint32_t)acc[q][a][4 * g + 1],
                         (uint32_t)acc[q][a][4 * g + 2], (uint32_t)acc[q][a][4 * g + 3]);
#pragma unroll 1
      for (int g = 0; g < 4; ++g) {
        const uint4 v0 = mine[g * 64], v1 = mine[(4 + g) * 64], v2 = mine[(8 + g) * 64];
        const int x0[4] = {(int)v0.x, (int)v0.y, (int)v0.z, (int)v0.w};
        const int x1[4] = {(int)v1.x, (int)v1.y, (int)v1.z, (int)v1.w};
        const int x2[4] = {(int)v2.x, (int)v2.y, (int)v2.z, (int)v2.w};
        const int il = rb + a * 32 + 8 * g;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double S = s0 * (double)x0[r] + s1 * (double)x1[r] + s2 * (double)x2[r];
          const int n = count_at == 0 ? x0[r] : count_at == 1 ? x1[r] : x2[r];
          gi_put(o, t == t0, end, park + (int64_t)(il + r) * (128 / NR), I * 128 * NR + il + r, j,
                 S, (uint32_t)n);
        }
      }
    }
    __syncthreads();
  }
}

// Adds the ranges of every entry in order.
template <int NR>
__global__ __launch_bounds__(256) void k_gi_reduce(GiOut o) {
  const int64_t total = o.tail * 16384;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * 256) {
    int64_t I, J;
    gi_tile<NR>(o.head + (e >> 14), o.nj, I, J);
    const int in = (int)(e & 16383);
    const int64_t i = I * 128 * NR + in / (128 / NR), j = J * (128 / NR) + in % (128 / NR);
    if (j >= o.m || i > j) continue;
    double S = 0.0;
    uint32_t n = 0;
    for (int64_t k = 0; k < o.n_split; ++k) {
      S = __dadd_rn(S, o.part_s[k * total + e]);
      n += o.part_n[k * total + e];
    }
    gi_store(o, i, j, S, n);
  }
}

// ---- plan and launch ------------------------------------------------------------------
namespace {
constexpr int64_t kGiAlign = 256;

// Rows per tile: 512 (NR = 4) or 256 (2).  The larger tile generates its
// digits for twice the rows, but fills the diagonal worse: 1,000 samples take
// 0.80 ms with 256, 0.86 ms with 512.
int gi_shape(int64_t m) { return m > 1536 ? 4 : 2; }

int64_t gi_tile_count(int64_t m, int64_t& ni, int64_t& nj) {
  const int nr = gi_shape(m);
  return nr == 4 ? gi_tiles<4>(m, ni, nj) : gi_tiles<2>(m, ni, nj);
}

// 512 blocks run at once (two per CU).  Whole rounds of them take whole tiles;
// the tiles of the last, partial round are split into ranges of chunks, by
// the fewest rounds times chunks per range (3 more for a range's first
// loads, 0.025 per tile and range for adding it).
void gi_split(int64_t tiles, int64_t nch, int64_t& head, int64_t& n_split, int64_t& cps) {
  head = tiles / 512 * 512;
  const int64_t tail = tiles - head;
  n_split = 1;
  cps = nch;
  double best = (double)nch;
  for (int64_t want = 2; want <= 64 && tail > 0 && want * tail <= 4096; ++want) {
    const int64_t c = ceil_div(nch, want);
    if (c < 4) break;
    const int64_t n = ceil_div(nch, c);
    const double cost = (double)ceil_div(tail * n, 512) * (double)(c + 3) + 0.025 * tail * n;
    if (cost < 0.97 * best) {
      best = cost;
      n_split = n;
      cps = c;
    }
  }
}
}  // namespace

bool grm_int_plan(int64_t m, int64_t nv, int64_t rows_pad, int64_t wp, int64_t base,
                  GrmIntPlan& p) {
  // int32 sums: at most 384 per variant and digit place
  if (nv > (int64_t)4 << 20 || m > (int64_t)1 << 20) return false;
  const double work = (double)m * (double)m * (double)nv;
  if (work < kGrmIntMinWork && nv < kGrmIntLong &&
      !(m <= kGrmIntSmall && nv >= kGrmIntShortMin && nv <= kGrmIntShortMax))
    return false;
  int64_t ni, nj;
  p.nch = wp / 4;
  p.tiles = gi_tile_count(m, ni, nj);
  if (p.tiles >= (int64_t)1 << 30) return false;
  p.nj = nj;
  p.blocks32 = ni * 4 * gi_shape(m);
  gi_split(p.tiles, p.nch, p.head, p.n_split, p.cps);
  const int64_t parts = p.n_split > 1 ? p.n_split * (p.tiles - p.head) : 0;
  int64_t at = base;
  auto take = [&](int64_t bytes) {
    const int64_t o = at;
    at = round_up(at + bytes, kGiAlign);
    return o;
  };
  // column strips reach past the last row tile only within its rows
  p.off_G = take(p.blocks32 * p.nch * kGiBlockWords * 4);
  p.off_tab = take((kGiListedSlot + 1) * p.nch * kGiTabWords * 4);
  p.off_cnt = take(ceil_div(rows_pad, kGiSeg) * wp * 16 * 4);
  p.off_stat = take(wp * 16 * 8);
  p.off_marks = take(wp * 4);
  p.off_panel = take(sizeof(GiPanel));
  p.off_fine = take(ceil_div(p.nch, 32) * 4);
  p.off_part_s = take(parts * 16384 * 8);
  p.off_part_n = take(parts * 16384 * 4);
  p.bytes = at;
  return p.bytes - base <= kGrmIntMaxBytes &&
         p.bytes + nv * ceil_div(m, 4) + 12 * m * m <= kGrmIntMaxCall;
}

namespace {
template <int NR>
int gi_launch_pairs(const GrmIntPlan& p, char* ws, const GiOut& o, hipStream_t st) {
  hipLaunchKernelGGL((k_gi_pairs<NR>), dim3((unsigned)(o.head + o.tail * o.n_split)),
                     dim3(256), 0, st,
                     (const uint32_t*)(ws + p.off_G), (const uint32_t*)(ws + p.off_tab),
                     (const GiPanel*)(ws + p.off_panel), (const uint32_t*)(ws + p.off_fine),
                     p.nch, o);
  int rc = check_launch("grm_int_pairs");
  if (rc == PG_OK && p.n_split > 1) {
    const int64_t blocks = o.tail * 64;
    hipLaunchKernelGGL((k_gi_reduce<NR>), dim3((unsigned)(blocks < 65536 ? blocks : 65536)),
                       dim3(256), 0, st, o);
    rc = check_launch("grm_int_reduce");
  }
  return rc;
}
}  // namespace

int launch_grm_int(const GrmIntPlan& p, char* ws, const uint32_t* T, int64_t m, int64_t rows_pad,
                   int64_t wp, double* grm, uint32_t* n_used, int full, hipStream_t st) {
  uint32_t* cnt = (uint32_t*)(ws + p.off_cnt);
  uint2* stat = (uint2*)(ws + p.off_stat);
  uint32_t* marks = (uint32_t*)(ws + p.off_marks);
  GiPanel* panel = (GiPanel*)(ws + p.off_panel);
  uint32_t* fine = (uint32_t*)(ws + p.off_fine);
  const int64_t segs = rows_pad / kGiSeg, nv_pad = wp * 16;
  hipLaunchKernelGGL(k_gi_counts, dim3((unsigned)ceil_div(wp, 256), (unsigned)segs), dim3(256), 0,
                     st, T, wp, cnt, panel, fine);
  int rc = check_launch("grm_int_counts");
  if (rc != PG_OK) return rc;
  hipLaunchKernelGGL(k_gi_stats, dim3((unsigned)ceil_div(nv_pad, 256)), dim3(256), 0, st, cnt,
                     nv_pad, (int)segs, stat, marks, panel, fine);
  rc = check_launch("grm_int_stats");
  if (rc != PG_OK) return rc;
  hipLaunchKernelGGL(k_gi_tables, dim3((unsigned)ceil_div(nv_pad, 256), 6), dim3(256), 0, st, stat,
                     p.nch, panel, fine, (uint32_t*)(ws + p.off_tab));
  rc = check_launch("grm_int_tables");
  if (rc != PG_OK) return rc;
  hipLaunchKernelGGL(k_gi_operand, dim3((unsigned)ceil_div(wp, 64), (unsigned)p.blocks32),
                     dim3(256), 0, st, T, rows_pad, wp, marks, (uint32_t*)(ws + p.off_G));
  rc = check_launch("grm_int_operand");
  mark_stage(1, st);
  if (rc != PG_OK) return rc;
  const GiOut o{grm,    n_used, m, full, p.nj, p.head, p.tiles - p.head, p.n_split, p.cps,
                (double*)(ws + p.off_part_s), (uint32_t*)(ws + p.off_part_n)};
  const int nr = gi_shape(m);
  rc = nr == 4 ? gi_launch_pairs<4>(p, ws, o, st)
               : gi_launch_pairs<2>(p, ws, o, st);
  mark_stage(2, st);
  return rc;
}

}  // namespace pg
