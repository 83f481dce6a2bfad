// LD window sums with missing-call corrections (section "Bit population
// count": without missing calls the per-variant sums are fixed, and only
// sum x_a x_b has to be computed per pair).
//
// Per variant v over the selected samples: c_v missing calls (the list of
// their samples, in increasing order) and the totals over its non-missing
// calls, t_v = sum x and u_v = sum x^2.  With x_a[k] = 0 for a missing call,
// the sums of a pair (a, b) over the samples where neither call is missing
// are the totals minus what the other variant's missing calls remove:
//   n   = m - c_a - c_b + |miss(a) and miss(b)|
//   Sx  = t_a - sum over k in miss(b) of x_a[k],  Sxx = u_a - (same for x_a^2)
//   Sy  = t_b - sum over k in miss(a) of x_b[k],  Syy = u_b - (same for x_b^2)
// and Sxy is one Gram over all samples on the matrix cores (fp4, int8 for
// the largest cohorts).  Every sum
// stays an exact integer.
//
// A correction reads one word per missing call and 16 variants: a word of
// the sample-major operand T holds the codes of 16 consecutive variants at
// one sample, and their per-variant counts of homozygous A1, homozygous A2
// and missing codes grow as bytes, one byte-permute lookup per four variants.
// T is stored in strips of 64 variants (a tile's side), so one tile side at
// one sample is 16 contiguous bytes and the samples of a strip are adjacent:
// the missing calls of a tile read from two contiguous runs, and a line
// fetched for one sample holds the tile's codes at seven neighbouring ones.
//
// Tiles are the 64 x 64 variant tiles of the dense kernel.  A tile takes
// this path when all of its variants have at most `cap` missing calls (the
// length of a list slot) and its missing calls are few enough (at most
// `budget` over its two 64-variant groups) that the corrections cost less
// than the five dense Grams they replace; the dense kernel runs the other
// tiles and skips these.
//
// Launch order: the layout (partial counts per variant), k_ld_totals (counts
// and totals, group statistics, and whether enough groups qualify for the path
// to be on), k_ld_lists and k_ld_transpose (lists and T, only when it is on and
// has missing calls to correct), then the dense kernel and k_ld_sparse, each
// taking its own tiles (k_ld_complete those without any missing call).
#include "tiles.h"

namespace pg {

// A thread per variant sums the layout's partial counts; a wave is a group of
// 64 variants, so the group statistics are lane reductions.  Padding samples
// were counted as missing; padding variants get zero counts.  A group counts in
// groups_ok[0] when its diagonal tile qualifies (a tile (I, J) can qualify only
// if one of its groups has total <= budget / 2, whose diagonal tile then
// qualifies too), and in groups_ok[1] when it has missing calls that a tile the
// path takes could ask for, in groups_ok[2] when it has any.  Bound by the start
// of its few blocks (11 to 14 us);
// counting in the layout and skipping lists and T where there is nothing to
// correct took pruning 10,000 x 88,025 calls without missing ones from 1.10 to
// 0.85 ms (the operand was read twice more for counts, 72 us each, and T built
// for nothing, 117 us), and 5,000 x 500,000 at 1% from 5.95 to 5.85 ms.
constexpr int kTotThreads = 1024;

__global__ __launch_bounds__(kTotThreads) void k_ld_totals(
    const uint32_t* __restrict__ part, int64_t n_part, int64_t pad, int64_t m, int64_t nv,
    int64_t rows_pad, int2* __restrict__ stats, int4* __restrict__ vst, int cap, int64_t budget,
    int64_t* __restrict__ gsum, int* __restrict__ gmax, uint32_t* __restrict__ groups_ok) {
  __shared__ uint32_t s_ok[3];
  if (threadIdx.x < 3) s_ok[threadIdx.x] = 0;
  __syncthreads();
  const int64_t v = (int64_t)blockIdx.x * kTotThreads + threadIdx.x;
  if (v < rows_pad) {   // rows_pad: whole waves
    int n3 = 0, n0 = 0, c = 0;
    if (v < nv) {
      for (int64_t b = 0; b < n_part; ++b) {
        const uint32_t p = part[b * rows_pad + v];
        n3 += p & 1023u;
        n0 += (p >> 10) & 1023u;
        c += p >> 20;
      }
      c -= (int)pad;
    }
    if (stats && v < nv) stats[v] = allele_counts(n3, n0, m - c);
    if (vst) {
      vst[v] = make_int4(c, n3 - n0, n3 + n0, 0);
      int64_t sum = c;
      int mx = c;
      for (int d = 32; d > 0; d >>= 1) {
        sum += __shfl_xor(sum, d, 64);
        const int o = __shfl_xor(mx, d, 64);
        mx = o > mx ? o : mx;
      }
      if ((threadIdx.x & 63) == 0) {
        gsum[v / 64] = sum;
        gmax[v / 64] = mx;
        if (mx <= cap && sum <= budget / 2) atomicAdd(&s_ok[0], 1u);
        if (mx > 0 && mx <= cap && sum <= budget) atomicAdd(&s_ok[1], 1u);
        if (mx > 0) atomicAdd(&s_ok[2], 1u);
      }
    }
  }
  __syncthreads();
  if (vst && threadIdx.x < 3 && s_ok[threadIdx.x])
    atomicAdd(&groups_ok[threadIdx.x], s_ok[threadIdx.x]);
}

int launch_ld_totals(const LdCounts& cn, int64_t wn, int64_t m, int64_t nv, int64_t rows_pad,
                     int2* stats, const LdSparse* sp, hipStream_t st) {
  hipLaunchKernelGGL(k_ld_totals, dim3((unsigned)ceil_div(rows_pad, kTotThreads)),
                     dim3(kTotThreads), 0, st, cn.part, ceil_div(wn, kLdCountWords), 16 * wn - m, m,
                     nv, rows_pad, stats, sp ? sp->vst : nullptr, sp ? sp->cap : 0,
                     sp ? sp->budget : 0, sp ? sp->gsum : nullptr, sp ? sp->gmax : nullptr,
                     sp ? sp->groups_ok : nullptr);
  return check_launch("ld_totals");
}

// Whether the correction path is on and has calls to correct.
__device__ __forceinline__ bool ld_corrects(const uint32_t* groups_ok, uint32_t min_groups) {
  return groups_ok[0] >= min_groups && groups_ok[1] > 0;
}

// Per-variant missing-call lists (sample indices, increasing) of the groups
// that tiles of the path can use: one wave per variant row of the
// variant-major operand D (padding samples are
// not listed).
__global__ __launch_bounds__(256) void k_ld_lists(const uint32_t* __restrict__ D, int64_t wn,
                                                  int64_t m, int64_t nv, int cap, int64_t budget,
                                                  uint32_t* __restrict__ lists,
                                                  const int4* __restrict__ vst,
                                                  const int64_t* __restrict__ gsum,
                                                  const int* __restrict__ gmax,
                                                  const uint32_t* __restrict__ groups_ok,
                                                  uint32_t min_groups) {
  if (!ld_corrects(groups_ok, min_groups)) return;
  const int lane = threadIdx.x & 63;
  const int64_t waves = (int64_t)gridDim.x * 4;
  for (int64_t v = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); v < nv; v += waves) {
    if (vst[v].x == 0 || gmax[v / 64] > cap || gsum[v / 64] > budget) continue;
    const uint32_t* row = D + v * wn;
    uint32_t* list = lists + v * (int64_t)cap;
    int64_t c = 0;
    constexpr int kU = 8;   // 64-word slices loaded ahead of the scan
    for (int64_t w0 = 0; w0 < wn; w0 += 64 * kU) {
      uint32_t x[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int64_t w = w0 + 64 * u + lane;
        x[u] = w < wn ? row[w] : 0u;   // past the row: no missing calls
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int64_t w = w0 + 64 * u + lane;
        uint32_t miss = x[u] & ~(x[u] >> 1) & 0x55555555u;   // code 01
        const int64_t valid = m - 16 * w;   // selected samples in this word
        if (valid < 16) miss &= valid <= 0 ? 0u : ((1u << (2 * valid)) - 1u);
        if (__ballot(miss != 0) == 0) continue;   // (the same for the whole wave)
        // exclusive prefix sum of the per-lane counts (at most 16) over the
        // wave, one bit of the count at a time, with no cross-lane data moves
        const int k = __popc(miss);
        int excl = 0, total = 0;
#pragma unroll
        for (int b = 0; b < 5; ++b) {
          const uint64_t bb = __ballot((k >> b) & 1);
          excl += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bb >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)bb, 0u)) << b;
          total += __popcll(bb) << b;
        }
        int64_t pos = c + excl;
        while (miss) {
          const int bit = __ffs(miss) - 1;
          if (pos < cap) list[pos] = (uint32_t)(16 * w + (bit >> 1));
          ++pos;
          miss &= miss - 1;
        }
        c += total;
      }
    }
  }
}

constexpr int kSpS = 65;          // LDS row stride of the per-pair cells (words)
constexpr int kSpBatch = 8;       // missing calls per lane and batch
constexpr int kSpFlush = 248;     // missing calls between byte-counter flushes (< 256)

__device__ __forceinline__ uint32_t gather_word(const uint32_t* p) { return *p; }

// Walks one lane's missing-call list (cnt entries; the wave's longest list
// has cmax) in batches of kSpBatch and hands each batch of gathered words to
// consume(); the word of sample k is at base + 16 k + lane_bytes (one strip
// of T).  Lanes past their list get `idle`.  Two stages in flight: the
// entries of batch j + 2 and the words of batch j + 1 load while batch j is
// counted.  List slots hold a multiple of kSpBatch entries and cmax does not
// exceed the slot, so every list read stays inside the slot (entries past
// cnt are read but not used).
template <typename W, typename F>
__device__ __forceinline__ void gather_list(const uint32_t* __restrict__ list, int cnt, int cmax,
                                            const char* __restrict__ base, uint32_t lane_bytes,
                                            W idle, F&& consume) {
  const int nb = (cmax + kSpBatch - 1) / kSpBatch;
  if (nb == 0) return;
  uint32_t ks[kSpBatch];
  auto load_ks = [&](int j) {
    const uint4 a = *reinterpret_cast<const uint4*>(list + j * kSpBatch);
    const uint4 b = *reinterpret_cast<const uint4*>(list + j * kSpBatch + 4);
    ks[0] = a.x; ks[1] = a.y; ks[2] = a.z; ks[3] = a.w;
    ks[4] = b.x; ks[5] = b.y; ks[6] = b.z; ks[7] = b.w;
  };
  W w[kSpBatch];
  auto load_w = [&](int j) {
#pragma unroll
    for (int u = 0; u < kSpBatch; ++u) {
      const char* p = base + (((uint64_t)ks[u] << 4) + lane_bytes);
      w[u] = j * kSpBatch + u < cnt ? gather_word(reinterpret_cast<const W*>(p)) : idle;
    }
  };
  load_ks(0);
  load_w(0);
  if (nb > 1) load_ks(1);
  for (int j = 0; j < nb; ++j) {
    W cur[kSpBatch];
#pragma unroll
    for (int u = 0; u < kSpBatch; ++u) cur[u] = w[u];
    if (j + 1 < nb) load_w(j + 1);
    if (j + 2 < nb) load_ks(j + 2);
    consume(cur);
  }
}

// Byte c of each table is the count increment of code c: homA1 in the low
// nibble and homA2 in the high nibble of one byte, or missing.
constexpr uint32_t kNibHom = 0x10000001u;
constexpr uint32_t kCntMiss = 0x00000100u;

// Per-variant counters of one batch of 16-code words: counter dword d, byte
// e counts position 4e + d.  homA1 / homA2 grow as nibbles over the batch
// (at most kSpBatch < 16 per nibble) and are then added to the byte counters
// h1 / h2; missing codes (kMiss) go straight to the byte counters ms.
template <bool kMiss>
__device__ __forceinline__ void count_batch(const uint32_t (&words)[kSpBatch], uint32_t (&h1)[4],
                                            uint32_t (&h2)[4], uint32_t (&ms)[4]) {
  uint32_t nib[4] = {0, 0, 0, 0};
#pragma unroll
  for (int u = 0; u < kSpBatch; ++u) {
    uint32_t c[4];
    spread_codes(words[u], c);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      nib[d] += __builtin_amdgcn_perm(0u, kNibHom, c[d]);
      if constexpr (kMiss) ms[d] += __builtin_amdgcn_perm(0u, kCntMiss, c[d]);
    }
  }
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    h1[d] += nib[d] & 0x0F0F0F0Fu;
    h2[d] += (nib[d] >> 4) & 0x0F0F0F0Fu;
  }
}

// kFp4: Sxy from the nibbles of E.  A whole nibble is v = x + 0.5 for a call
// and 0 for a missing one, so one fp4 Gram without any expansion gives
// G = <v_a, v_b> = Sxy + (Sx + Sy) / 2 + n / 4 over the samples where neither
// is missing, exactly (kLdFp4MaxSamples); the cells hold 4 G.
template <bool kFp4>
__device__ __forceinline__ void ld_sparse_tile(
    const uint32_t* __restrict__ D, int64_t wn, const uint32_t* __restrict__ T, int64_t t_rows,
    const uint32_t* __restrict__ lists, const int4* __restrict__ vst, int cap, int64_t m,
    int64_t nv, int64_t I, int64_t J, int32_t window, double r2_min, const LdScratch& sc,
    pg_ld_pair* __restrict__ dbg, int64_t v0) {
  // per-pair cells: first the Sxy partial sums, then the b-side corrections
  // (row a, column b); the a-side corrections (row b, column a): homA1 |
  // homA2 << 16 and the shared missing calls
  __shared__ uint32_t s_cell[kLdTile * kSpS];
  __shared__ uint32_t s_acell[kLdTile * kSpS];
  __shared__ uint32_t s_mcell[kLdTile * kSpS];
  const int t = threadIdx.x, lane = t & 63;
  const int wid = __builtin_amdgcn_readfirstlane(t >> 6);
  const int g = lane >> 5, rl = lane & 31;
  const int qi = wid >> 1, qj = wid & 1;   // this wave's 32 x 32 quadrant
  for (int e = t; e < kLdTile * kSpS; e += 256) s_cell[e] = s_acell[e] = s_mcell[e] = 0;
  __syncthreads();

  // ---- Sxy: each wave takes a quarter of the samples for the whole tile
  // (2 x 2 blocks of 32 x 32); lane group g holds words 8q + 4g .. + 3 of its
  // rows, and A and B use the same word order, so K matches.
  if constexpr (kFp4) {
    // steps of 64 samples; a wave's load of 32 variants is two runs of 512
    // bytes.  Four register sets, rotating: loads three steps ahead.
    const int64_t nsteps = wn / 4;
    const uint32_t* pa = D + I * nsteps * 512 + g * 256 + 4 * rl;
    const uint32_t* pb = D + J * nsteps * 512 + g * 256 + 4 * rl;
    const int64_t q0 = nsteps * wid / 4, q1 = nsteps * (wid + 1) / 4;
    v16f acc00 = (v16f){0}, acc01 = (v16f){0}, acc10 = (v16f){0}, acc11 = (v16f){0};
    uint4 r[4][4];
    auto load = [&](uint4 (&x)[4], int64_t q) {
      q = q < q1 ? q : q1 - 1;
      x[0] = *reinterpret_cast<const uint4*>(pa + 512 * q);
      x[1] = *reinterpret_cast<const uint4*>(pa + 512 * q + 128);
      x[2] = *reinterpret_cast<const uint4*>(pb + 512 * q);
      x[3] = *reinterpret_cast<const uint4*>(pb + 512 * q + 128);
    };
    auto step = [&](const uint4 (&x)[4]) {
      const v8i a0 = nib_mask(x[0], ~0u), a1 = nib_mask(x[1], ~0u);
      const v8i c0 = nib_mask(x[2], ~0u), c1 = nib_mask(x[3], ~0u);
      acc00 = mfma_fp4(a0, c0, acc00);
      acc01 = mfma_fp4(a0, c1, acc01);
      acc10 = mfma_fp4(a1, c0, acc10);
      acc11 = mfma_fp4(a1, c1, acc11);
    };
    if (q0 < q1) {
#pragma unroll
      for (int u = 0; u < 3; ++u) load(r[u], q0 + u);
      for (int64_t q = q0; q < q1; q += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          load(r[(u + 3) & 3], q + u + 3);
          if (q + u < q1) step(r[u]);
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = 8 * (v >> 2) + 4 * g + (v & 3);
      atomicAdd(&s_cell[row * kSpS + rl], (uint32_t)(int)(4.0f * acc00[v]));
      atomicAdd(&s_cell[row * kSpS + 32 + rl], (uint32_t)(int)(4.0f * acc01[v]));
      atomicAdd(&s_cell[(32 + row) * kSpS + rl], (uint32_t)(int)(4.0f * acc10[v]));
      atomicAdd(&s_cell[(32 + row) * kSpS + 32 + rl], (uint32_t)(int)(4.0f * acc11[v]));
    }
  } else {
    const uint32_t* pa = D + (I * kLdTile + rl) * wn + 4 * g;
    const uint32_t* pb = D + (J * kLdTile + rl) * wn + 4 * g;
    const int64_t off1 = 32 * wn;
    const int64_t ngroups = wn / 8;
    const int64_t q0 = ngroups * wid / 4, q1 = ngroups * (wid + 1) / 4;
    v16i acc00 = (v16i){0}, acc01 = (v16i){0}, acc10 = (v16i){0}, acc11 = (v16i){0};
    // three register sets, rotating, so the prefetch (two groups ahead)
    // needs no copies
    uint4 r0[4], r1[4], r2[4];
    auto load = [&](uint4 (&r)[4], int64_t q) {
      r[0] = *reinterpret_cast<const uint4*>(pa + 8 * q);
      r[1] = *reinterpret_cast<const uint4*>(pa + off1 + 8 * q);
      r[2] = *reinterpret_cast<const uint4*>(pb + 8 * q);
      r[3] = *reinterpret_cast<const uint4*>(pb + off1 + 8 * q);
    };
    auto step = [&](const uint4 (&r)[4]) {
      const uint32_t wa0[4] = {r[0].x, r[0].y, r[0].z, r[0].w};
      const uint32_t wa1[4] = {r[1].x, r[1].y, r[1].z, r[1].w};
      const uint32_t wb0[4] = {r[2].x, r[2].y, r[2].z, r[2].w};
      const uint32_t wb1[4] = {r[3].x, r[3].y, r[3].z, r[3].w};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        uint32_t c[4];
        spread_codes(wa0[s], c);
        const v4i xa0 = ld_lookup(kLdLutX, c);
        spread_codes(wa1[s], c);
        const v4i xa1 = ld_lookup(kLdLutX, c);
        spread_codes(wb0[s], c);
        const v4i xb0 = ld_lookup(kLdLutX, c);
        spread_codes(wb1[s], c);
        const v4i xb1 = ld_lookup(kLdLutX, c);
        acc00 = __builtin_amdgcn_mfma_i32_32x32x32_i8(xa0, xb0, acc00, 0, 0, 0);
        acc01 = __builtin_amdgcn_mfma_i32_32x32x32_i8(xa0, xb1, acc01, 0, 0, 0);
        acc10 = __builtin_amdgcn_mfma_i32_32x32x32_i8(xa1, xb0, acc10, 0, 0, 0);
        acc11 = __builtin_amdgcn_mfma_i32_32x32x32_i8(xa1, xb1, acc11, 0, 0, 0);
      }
    };
    if (q0 < q1) load(r0, q0);
    if (q0 + 1 < q1) load(r1, q0 + 1);
    for (int64_t q = q0; q < q1; q += 3) {
      if (q + 2 < q1) load(r2, q + 2);
      step(r0);
      if (q + 3 < q1) load(r0, q + 3);
      if (q + 1 < q1) step(r1);
      if (q + 4 < q1) load(r1, q + 4);
      if (q + 2 < q1) step(r2);
    }
    // 32x32 accumulator layout: register v of lane l holds row
    // 8*(v/4) + 4*(l/32) + v%4 and column l%32.
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = 8 * (v >> 2) + 4 * g + (v & 3);
      atomicAdd(&s_cell[r * kSpS + rl], (uint32_t)acc00[v]);
      atomicAdd(&s_cell[r * kSpS + 32 + rl], (uint32_t)acc01[v]);
      atomicAdd(&s_cell[(32 + r) * kSpS + rl], (uint32_t)acc10[v]);
      atomicAdd(&s_cell[(32 + r) * kSpS + 32 + rl], (uint32_t)acc11[v]);
    }
  }
  __syncthreads();
  // this lane's 16 pairs of the quadrant: rows al(v) of tile I, column bl of J
  const int bl = 32 * qj + rl;
  int xy[16];
#pragma unroll
  for (int v = 0; v < 16; ++v)
    xy[v] = (int)s_cell[(32 * qi + 8 * (v >> 2) + 4 * g + (v & 3)) * kSpS + bl];
  __syncthreads();

  // ---- corrections.  Lane (16 * wave + lane / 4, q = lane % 4) owns
  // variant `own` of each tile side and the 16 variants of word q of the
  // other side.  b-side: at the missing calls of variant own of tile I, the
  // codes of word q of tile J, into s_cell; the first flush stores, so every
  // cell is written even for an empty list.  a-side: at the missing calls of
  // variant own of tile J, the codes of word q of tile I, into s_acell and
  // s_mcell.  The four lanes of one variant read one 16-byte piece.
  const int own = 16 * wid + (lane >> 2), q = lane & 3;
  uint32_t bh1[4] = {0, 0, 0, 0}, bh2[4] = {0, 0, 0, 0}, bms[4];
  uint32_t ah1[4] = {0, 0, 0, 0}, ah2[4] = {0, 0, 0, 0}, ams[4] = {0, 0, 0, 0};
  bool first = true;
  int since_b = 0, since_a = 0;
  auto flush_b = [&]() {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int idx = own * kSpS + 16 * q + 4 * e + d;
        const uint32_t val = ((bh1[d] >> (8 * e)) & 0xFFu) | (((bh2[d] >> (8 * e)) & 0xFFu) << 16);
        s_cell[idx] = first ? val : s_cell[idx] + val;
      }
      bh1[d] = bh2[d] = 0;
    }
    first = false;
  };
  auto flush_a = [&]() {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int idx = own * kSpS + 16 * q + 4 * e + d;
        s_acell[idx] += ((ah1[d] >> (8 * e)) & 0xFFu) | (((ah2[d] >> (8 * e)) & 0xFFu) << 16);
        s_mcell[idx] += (ams[d] >> (8 * e)) & 0xFFu;
      }
      ah1[d] = ah2[d] = ams[d] = 0;
    }
  };
  auto count_b = [&](const uint32_t (&w)[kSpBatch]) {
    count_batch<false>(w, bh1, bh2, bms);
    since_b += kSpBatch;
    if (since_b == kSpFlush) {
      flush_b();
      since_b = 0;
    }
  };
  auto count_a = [&](const uint32_t (&w)[kSpBatch]) {
    count_batch<true>(w, ah1, ah2, ams);
    since_a += kSpBatch;
    if (since_a == kSpFlush) {
      flush_a();
      since_a = 0;
    }
  };
  const uint32_t* stripI = T + I * t_rows * 4;
  const uint32_t* stripJ = T + J * t_rows * 4;
  {
    const int cnt = vst[I * kLdTile + own].x;
    int cmax = cnt;
    for (int d = 32; d > 0; d >>= 1) {
      const int o = __shfl_xor(cmax, d, 64);
      cmax = o > cmax ? o : cmax;
    }
    cmax = __builtin_amdgcn_readfirstlane(cmax);
    gather_list(lists + (I * kLdTile + own) * (int64_t)cap, cnt, cmax,
                reinterpret_cast<const char*>(stripJ), 4u * q, 0xAAAAAAAAu, count_b);
  }
  {
    const int cnt = vst[J * kLdTile + own].x;
    int cmax = cnt;
    for (int d = 32; d > 0; d >>= 1) {
      const int o = __shfl_xor(cmax, d, 64);
      cmax = o > cmax ? o : cmax;
    }
    cmax = __builtin_amdgcn_readfirstlane(cmax);
    gather_list(lists + (J * kLdTile + own) * (int64_t)cap, cnt, cmax,
                reinterpret_cast<const char*>(stripI), 4u * q, 0xAAAAAAAAu, count_a);
  }
  if (since_b || first) flush_b();
  if (since_a) flush_a();
  __syncthreads();

  // ---- pairs
  const int64_t b = J * kLdTile + bl;
  if (b >= nv) return;
  const int4 sb = vst[b];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int al = 32 * qi + 8 * (v >> 2) + 4 * g + (v & 3);
    const int64_t a = I * kLdTile + al;
    if (!(a < b && b - a <= window)) continue;
    const int4 sa = vst[a];
    const uint32_t pb = s_cell[al * kSpS + bl], pa = s_acell[bl * kSpS + al];
    const int64_t a1 = pa & 0xFFFFu, a2 = pa >> 16;
    const int64_t b1 = pb & 0xFFFFu, b2 = pb >> 16;
    const int64_t both = s_mcell[bl * kSpS + al];
    const int64_t n = m - sa.x - sb.x + both;
    const int64_t sx = sa.y - (a2 - a1), sy = sb.y - (b2 - b1);
    const int64_t sxx = sa.z - (a2 + a1), syy = sb.z - (b2 + b1);
    const int64_t sxy = kFp4 ? (xy[v] - 2 * (sx + sy) - n) / 4 : xy[v];
    if (dbg) {
      pg_ld_pair rec;
      rec.a = (int32_t)(v0 + a);
      rec.b = (int32_t)(v0 + b);
      rec.n = n; rec.sx = sx; rec.sy = sy; rec.sxx = sxx; rec.syy = syy; rec.sxy = sxy;
      rec.r2 = ld_r2(n, sx, sy, sxx, syy, sxy);
      dbg[a * window + (b - a - 1)] = rec;
    } else {
      ld_mark(sc, a, b, r2_min, n, sx, sy, sxx, syy, sxy);
    }
  }
}

// ---- tiles without missing calls ---------------------------------------------
// 128 x 128 variants whose four groups have no missing call: n, Sx, Sy, Sxx and
// Syy are the variants' totals, and Sxy follows from the Gram of the whole
// nibbles, 4 G = 4 Sxy + 2 (Sx + Sy) + m.  Four waves of 64 x 64; chunks of two
// 64-sample steps (16 KB) reach LDS by direct loads two chunks ahead, three
// buffers, three blocks a CU.  The 64 x 64 tiles of the correction kernel read
// 4 KB from L2 per 16 matrix instructions, a tile here 8 KB per 64.
// Bound: the latency of the operand loads (a chunk nearly always holds a line
// that comes from HBM): 10,000 x 88,025, distance 699: 413 us at 37% matrix-core
// occupancy, against 589 us for the 64 x 64 tiles.  Chunks of one step in six
// buffers 442 us, two blocks a CU with 64 KB 458 to 500, four with 32 to 40 KB
// 450 to 480.
constexpr int kCtChunk = 2;                        // steps of 64 samples
constexpr int kCtGroup = kCtChunk * 512;           // words of a group's chunk
constexpr int kCtBuf = 4 * kCtGroup;               // two groups a side

// Whether the 128 x 128 tile (I2, J2) is one of these (n_groups of 64).
__device__ __forceinline__ bool ld_tile_complete(const int* gmax, int64_t I2, int64_t J2,
                                                 int64_t n_groups) {
  const int64_t a = 2 * I2 + 1 < n_groups ? 2 * I2 + 1 : 2 * I2;
  const int64_t b = 2 * J2 + 1 < n_groups ? 2 * J2 + 1 : 2 * J2;
  return (gmax[2 * I2] | gmax[a] | gmax[2 * J2] | gmax[b]) == 0;
}

__device__ __forceinline__ void ld_complete_tile(const uint32_t* __restrict__ E, int64_t nsteps,
                                                 const int4* __restrict__ vst, int64_t m,
                                                 int64_t nv, int64_t n_groups, int64_t I2,
                                                 int64_t J2, int32_t window, double r2_min,
                                                 const LdScratch& sc, lds_t* smem) {
  const int t = threadIdx.x, lane = t & 63;
  const int wid = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wr = wid >> 1, wc = wid & 1;           // this wave's 64 x 64 quadrant
  const int64_t ga = 2 * I2 + wr, gb = 2 * J2 + wc;   // its groups
  const bool active = ga < n_groups && gb < n_groups && gb >= ga &&
                      64 * (gb - ga) - 63 <= (int64_t)window;
  // wave w stages group w of {2 I2, 2 I2 + 1, 2 J2, 2 J2 + 1} (the last one
  // again where the tile reaches past it)
  const int64_t gs = wid < 2 ? 2 * I2 + wid : 2 * J2 + (wid - 2);
  const uint32_t* src = E + (gs < n_groups ? gs : n_groups - 1) * nsteps * 512 + 4 * lane;
  const int64_t nch = nsteps / kCtChunk;
  auto fetch = [&](int64_t c, int buf) {
    const uint32_t* p = src + (c < nch ? c : nch - 1) * kCtGroup;
    lds_t* const d = smem + buf * kCtBuf + wid * kCtGroup;
#pragma unroll
    for (int h = 0; h < kCtGroup / 256; ++h) lds_from_global(p + 256 * h, d + 256 * h);
  };
  v16f acc[2][2] = {{(v16f){0}, (v16f){0}}, {(v16f){0}, (v16f){0}}};
  fetch(0, 0);
  fetch(1, 1);
  asm volatile("s_waitcnt vmcnt(4)\n\ts_barrier" ::: "memory");
  int b0 = 0, b1 = 1, b2 = 2;
  for (int64_t k = 0; k < nch; ++k) {
    fetch(k + 2, b2);   // chunk k - 1's buffer: every wave is past it
    if (active) {
      const lds_t* ra = smem + b0 * kCtBuf + wr * kCtGroup + (lane >> 5) * 256 + (lane & 31) * 4;
      const lds_t* rb = smem + b0 * kCtBuf + (2 + wc) * kCtGroup + (lane >> 5) * 256 +
                        (lane & 31) * 4;
#pragma unroll
      for (int s = 0; s < kCtChunk; ++s) {
        v8i a[2], b[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          a[h] = nib_mask(lds_ld4(ra + s * 512 + 128 * h), ~0u);
          b[h] = nib_mask(lds_ld4(rb + s * 512 + 128 * h), ~0u);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = mfma_fp4(a[i], b[j], acc[i][j]);
      }
    }
    // chunk k + 1 has arrived, chunk k is used up
    asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const int b = b0;
    b0 = b1;
    b1 = b2;
    b2 = b;
  }
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  // per row of the tile: Sx and r2_min Var_a (1 - 2^-16), as ld_r2_reaches
  // forms it (m times the variances; the order of its nine roundings differs)
  const bool narrow = m < (1 << 15) && r2_min > 0.0;
  auto var_of = [&](const int4& s) {
    return narrow ? (float)(__mul24((int)m, s.z) - __mul24(s.y, s.y)) : 0.0f;
  };
  if (t < 128) {
    const int64_t a = 128 * I2 + t;
    const int4 s = a < nv ? vst[a] : make_int4(0, 0, 0, 0);
    smem[2 * t] = (uint32_t)s.y;
    smem[2 * t + 1] =
        __builtin_bit_cast(uint32_t, (float)r2_min * (1.0f - 0x1p-16f) * var_of(s));
  }
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if (!active) return;   // nothing after this point synchronises
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int64_t b = 64 * gb + 32 * j + (lane & 31);
    const int4 sb = b < nv ? vst[b] : make_int4(0, 0, 0, 0);
    const float vb = var_of(sb);
    const unsigned lim = b < nv ? (unsigned)window : 0u;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r0 = 64 * wr + 32 * i + 4 * (lane >> 5);   // row of register 0 in the tile
      const int d0 = (int)(b - 128 * I2) - r0;             // b - a of register 0
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int ar = 8 * (v >> 2) + (v & 3);
        if ((unsigned)(d0 - ar - 1) >= lim) continue;
        const int sx = (int)smem[2 * (r0 + ar)];
        const int sxy = ((int)(4.0f * acc[i][j][v]) - 2 * (sx + sb.y) - (int)m) >> 2;
        if (narrow) {
          const float c = (float)(__mul24((int)m, sxy) - __mul24(sx, sb.y));
          if (c * c < __builtin_bit_cast(float, (uint32_t)smem[2 * (r0 + ar) + 1]) * vb) continue;
        }
        const int64_t a = 128 * I2 + r0 + ar;
        ld_mark(sc, a, b, r2_min, m, sx, sb.y, vst[a].z, sb.z, sxy);
      }
    }
  }
}

__global__ __launch_bounds__(256, 3) void k_ld_complete(
    const uint32_t* __restrict__ E, int64_t wn, const int4* __restrict__ vst,
    const int* __restrict__ gmax, const uint32_t* __restrict__ groups_ok, uint32_t min_groups,
    int64_t m, int64_t nv, int64_t n_groups, int64_t n_band, int32_t window, double r2_min,
    LdScratch sc) {
  __shared__ __attribute__((aligned(16))) uint32_t smem[3 * kCtBuf];
  if (*groups_ok < min_groups) return;
  const int64_t blk = xcd_swizzle(blockIdx.x, gridDim.x);
  const int64_t I2 = blk / n_band, J2 = I2 + blk % n_band;
  if (J2 >= ceil_div(n_groups, 2) || !ld_tile_complete(gmax, I2, J2, n_groups)) return;
  ld_complete_tile(E, wn / 4, vst, m, nv, n_groups, I2, J2, window, r2_min, sc, (lds_t*)smem);
}

// One tile per block, in the band's order: neighbours that run together share
// their strips in L2 (blocks that walked several tiles each, for fewer block
// starts where the path is off, took 12% longer at 5,000 x 300,000; starting
// 132,000 blocks that leave at once takes 29 us).
template <bool kFp4>
__global__ __launch_bounds__(256, 3) void k_ld_sparse(
    const uint32_t* __restrict__ D, int64_t wn, const uint32_t* __restrict__ T, int64_t t_rows,
    const uint32_t* __restrict__ lists, const int4* __restrict__ vst,
    const int64_t* __restrict__ gsum, const int* __restrict__ gmax,
    const uint32_t* __restrict__ groups_ok, uint32_t min_groups, int cap, int64_t budget,
    int64_t m, int64_t nv, int64_t n_row_tiles, int64_t n_band, int32_t window,
    double r2_min, LdScratch sc, pg_ld_pair* __restrict__ dbg, int64_t v0) {
  if (*groups_ok < min_groups) return;
  if (kFp4 && !dbg && groups_ok[2] == 0) return;   // every tile is k_ld_complete's
  const int64_t blk = xcd_swizzle(blockIdx.x, gridDim.x);
  const int64_t I = blk / n_band;
  const int64_t J = I + blk % n_band;
  if (J >= n_row_tiles || !ld_tile_sparse(gsum, gmax, groups_ok, min_groups, I, J, cap, budget))
    return;
  if (kFp4 && !dbg && ld_tile_complete(gmax, I >> 1, J >> 1, n_row_tiles)) return;
  ld_sparse_tile<kFp4>(D, wn, T, t_rows, lists, vst, cap, m, nv, I, J, window, r2_min, sc, dbg, v0);
}

constexpr int kTrW = 32;            // words per block side: 512 variants x 512 samples
constexpr int kTrS = kTrW + 1;      // LDS row stride (words)

// Sample-major operand T in strips of 64 variants from the variant-major D
// (rows_pad x wn words): word a (the codes of variants 16a..16a+15) at sample
// k is T[((a / 4) * t_rows + k) * 4 + a % 4].  A block takes 32 words of each
// side; lanes read consecutive words of a D row (full lines), the 16x16
// transposes land in LDS, and each half-wave writes one sample's 32 words as
// eight 16-byte pieces of eight strips (consecutive samples of a strip are
// adjacent, so a block fills whole lines).  Variants past rows_pad read as
// missing.  Does nothing unless ld_corrects.
__global__ __launch_bounds__(256) void k_ld_transpose(const uint32_t* __restrict__ D,
                                                      int64_t rows_pad, int64_t wn,
                                                      uint32_t* __restrict__ T, int64_t t_rows,
                                                      int64_t tw,
                                                      const uint32_t* __restrict__ groups_ok,
                                                      uint32_t min_groups) {
  if (!ld_corrects(groups_ok, min_groups)) return;
  __shared__ uint32_t s_out[16 * kTrW * kTrS];
  const int64_t nb_a = ceil_div(tw, kTrW);
  const int64_t a0 = ((int64_t)blockIdx.x % nb_a) * kTrW;   // T word (16 variants)
  const int64_t g0 = ((int64_t)blockIdx.x / nb_a) * kTrW;   // D word (16 samples)
  const int t = threadIdx.x;
  const int gl = t % kTrW;
#pragma unroll 1
  for (int i = 0; i < 4; ++i) {
    const int al = t / kTrW + 8 * i;
    const int64_t a = a0 + al, g = g0 + gl;
    uint32_t x[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t v = 16 * a + r;
      x[r] = (v < rows_pad && g < wn) ? D[v * wn + g] : kAllMissing16;
    }
    transpose16_2bit(x);
#pragma unroll
    for (int c = 0; c < 16; ++c) s_out[(c * kTrW + gl) * kTrS + al] = x[c];
  }
  __syncthreads();
  const int lane = t & 63, wave = t >> 6;
  for (int row = 2 * wave + (lane >> 5); row < 16 * kTrW; row += 8) {
    const int64_t k = 16 * g0 + row, a = a0 + (lane & 31);
    if (k < t_rows && a < tw)   // T row 16 gl + c is LDS row c * kTrW + gl
      T[((a >> 2) * t_rows + k) * 4 + (a & 3)] =
          s_out[((row & 15) * kTrW + (row >> 4)) * kTrS + (lane & 31)];
  }
}

int launch_ld_lists(const uint32_t* D, int64_t wn, int64_t m, int64_t nv, const LdSparse& sp,
                    hipStream_t st) {
  const int64_t blocks = ceil_div(nv, 4) < 8192 ? ceil_div(nv, 4) : 8192;
  hipLaunchKernelGGL(k_ld_lists, dim3((unsigned)blocks), dim3(256), 0, st, D, wn, m, nv, sp.cap,
                     sp.budget, sp.lists, sp.vst, sp.gsum, sp.gmax, sp.groups_ok, sp.min_groups);
  return check_launch("ld_lists");
}

int launch_ld_transpose(const uint32_t* D, int64_t rows_pad, int64_t wn, uint32_t* T,
                        int64_t t_rows, int64_t tw, const LdSparse& sp, hipStream_t st) {
  const int64_t blocks = ceil_div(tw, kTrW) * ceil_div(t_rows, 16 * kTrW);
  hipLaunchKernelGGL(k_ld_transpose, dim3((unsigned)blocks), dim3(256), 0, st, D, rows_pad, wn, T,
                     t_rows, tw, sp.groups_ok, sp.min_groups);
  return check_launch("ld_transpose");
}

int launch_ld_sparse(const uint32_t* D, const uint32_t* E, int64_t wn, const uint32_t* T,
                     int64_t t_rows, int64_t m,
                     int64_t nv, int64_t rows_pad, int32_t window, double r2_min,
                     const LdScratch& sc, const LdSparse& sp, hipStream_t st, pg_ld_pair* dbg,
                     int64_t v0) {
  int rc;
  // the dense kernel takes the tiles this path leaves
  if (!dbg) {
    rc = launch_ld_mfma(D, E, m < kFp4MaxVariants, wn, nv, rows_pad, window, r2_min, sc, st, &sp);
    if (rc != PG_OK) return rc;
  }
  const int64_t n_row_tiles = rows_pad / kLdTile;
  const int64_t n_band = ((int64_t)window + kLdTile - 1) / kLdTile + 1;
  if (E && !dbg) {
    const int64_t n_row2 = ceil_div(n_row_tiles, 2), n_band2 = ((int64_t)window + 127) / 128 + 1;
    hipLaunchKernelGGL(k_ld_complete, dim3((unsigned)(n_row2 * n_band2)), dim3(256), 0, st, E, wn,
                       sp.vst, sp.gmax, sp.groups_ok, sp.min_groups, m, nv, n_row_tiles, n_band2,
                       window, r2_min, sc);
    rc = check_launch("ld_complete");
    if (rc != PG_OK) return rc;
  }
  hipLaunchKernelGGL(E ? k_ld_sparse<true> : k_ld_sparse<false>,
                     dim3((unsigned)(n_row_tiles * n_band)), dim3(256), 0, st, E ? E : D, wn, T,
                     t_rows, sp.lists, sp.vst, sp.gsum, sp.gmax, sp.groups_ok, sp.min_groups,
                     sp.cap, sp.budget, m, nv, n_row_tiles, n_band, window, r2_min, sc, dbg, v0);
  rc = check_launch("ld_sparse");
  mark_stage(2, st);
  return rc;
}

}  // namespace pg
