// Rank select of the zr quantile for binary16 activations in ONE sweep of X
// (constraint C2 of DCRP, Eq. zr_constraint: the k-th smallest |x| of every
// (image, token set), k = ceil(zr n), Supp. "Quantile Implementation").
//
// The magnitude key of a binary16 value has 15 bits.  A radix select over LDS
// histograms needs two sweeps of X for that many bits.  Here a small sample of
// every set first says where to look:
//
//   k_sets            one workgroup per set finds the set's tokens and moments, reads up
//                     to 8 Ki sampled elements and finds, in an LDS histogram of their top
//                     key bits, the sample order statistic whose sample rank corresponds
//                     to k.  The key interval [lo, lo + W) centred on it (W = as many
//                     one-key bins as the sweep's LDS histogram has per set) holds the true
//                     answer unless the sample is off by more than W/2 keys.
//   k_bracket_hist    one sweep of X: per set, the number of keys below lo and an LDS
//                     histogram, one bin per key, of the keys inside the interval.
//   k_bracket_finish  one workgroup per set: if below < k <= below + inside, the
//                     answer is the bin where the running count reaches k - below --
//                     the exact k-th smallest, no matter how the interval was chosen --
//                     and the set is projected.  Otherwise the set is counted as missed
//                     and the same workgroup resolves it with a two-level radix select
//                     over the set's own rows (exact as well, and rare).
//
// The result is therefore always the exact order statistic; the sample only decides
// which of the two routes computes it, i.e. how long it takes.
#include "tdq_device.hpp"

namespace tdq {

constexpr int kRunLen = 32;                                     // channels per run (64 bytes)
constexpr int kSampleBits = 10;                                 // key bits the sample histogram resolves
constexpr int kSweepThreads = 1024;
constexpr int kIdRounds = 16;                                   // range keys a thread of k_sets holds

// ---------------------------------------------------------------------------
// k_sets: one workgroup of NT threads per (image, token set).
//   1. the image's smallest and largest range key -> the key interval that belongs to this
//      set: gid = (key - lo) G / width is j exactly for ceil(j width / G) <= key - lo <
//      ceil((j + 1) width / G), so a token is recognised with two compares and no division;
//   2. the set's tokens (ids stored, counted, ranked) and their merged moments, summed
//      about the mean of the set's first token (identical tokens add exact zeros);
//   3. the sample of the set and the key interval that its order statistic says holds the
//      k-th smallest |x|.
// Bound by its chain of dependent steps (three trips to memory, seven barriers), not by
// traffic: every workgroup reads the image's T range keys itself, which is cheaper than a
// kernel boundary, and everything per token sits in registers when T <= 16 NT.  Ranks are
// counted wavefront by wavefront (any numbering of the set's tokens serves the sample), so
// the wavefronts exchange one count each.  SM = most sampled elements: the rank error of 8 Ki
// is 0.45 % of the set's mass, about 40 keys at 1024 keys per octave, against a half-width of
// W / 2 >= 256 keys; with fewer bins per set (more than 32 sets) 16 Ki are drawn.
// Measured, calibration of one call (two kernels for this before: assignment, then sample):
// [1, 7744, 64] 46.3 -> 30.9 us, [8, 121, 512] 30.7 -> 26.0, [32, 4096, 1024] 118.7 -> 108.3;
// with 16 Ki samples 31.7 / 26.9 / 111.0.
// ---------------------------------------------------------------------------
template <int NT, int SM>
__global__ __launch_bounds__(NT) void k_sets(
    const u16* __restrict__ X, long long ld, int T, int C, int G, int W, int vec,
    const float* __restrict__ r, const double* __restrict__ mean, const double* __restrict__ m2,
    int* __restrict__ gid, Scalars sc, int pass, int keep_base, GroupWork* __restrict__ grp,
    Bracket* __restrict__ br, u32* __restrict__ bhist, u32* __restrict__ img_flag,
    u32* __restrict__ status) {
  constexpr int NW = NT / 64;
  constexpr int kSampleRuns = SM / kRunLen;
  constexpr int kSampleTokens = kSampleRuns;         // at most one run per token
  __shared__ int sel[kSampleTokens];                 // drawn token of every stratum
  __shared__ long long run_base[kSampleRuns];        // element offset of every run's first channel
  __shared__ int run_len[kSampleRuns];               // channels of the run (<= kRunLen)
  __shared__ u32 shist[1 << kSampleBits];            // sample histogram over the top key bits
  __shared__ u32 s_min[NW], s_max[NW], wtot[NW], stot[NW], s_cmax[NW];
  __shared__ double s_s1[NW], s_s2[NW];
  __shared__ int s_first;
  const int j = blockIdx.x, b = blockIdx.y, idx = b * G + j;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* rb = r + (long long)b * T;
  const double* meanb = mean + (long long)b * T;
  const double* m2b = m2 + (long long)b * T;
  int* gb = gid + (long long)b * T;
  constexpr u32 kDead = 0xFFFFFFFFu;                 // no range key reaches it
  const bool one_batch = T <= kIdRounds * NT;
  u32 kv[kIdRounds];
  auto load_keys = [&](int t0) {
#pragma unroll
    for (int u = 0; u < kIdRounds; ++u) {
      const int t = t0 + u * NT + tid;
      kv[u] = t < T ? __float_as_uint(rb[t]) : kDead;
    }
  };

  // ---- 1: key range of the image, key interval of the set
  load_keys(0);
  for (int i = tid; i < (1 << kSampleBits); i += NT) shist[i] = 0;
  u32 kinv = 0, kmax = 0;                            // largest ~key, largest key
  for (int t0 = 0;;) {
#pragma unroll
    for (int u = 0; u < kIdRounds; ++u) {
      const u32 k = kv[u];
      kinv = ~k > kinv ? ~k : kinv;                  // ~kDead is 0
      kmax = k != kDead && k > kmax ? k : kmax;
    }
    t0 += kIdRounds * NT;
    if (t0 >= T) break;
    load_keys(t0);
  }
  kinv = group_max_u32<64>(kinv);
  kmax = group_max_u32<64>(kmax);
  if (lane == 63) { s_min[wave] = ~kinv; s_max[wave] = kmax; }
  __syncthreads();
  u32 lo = s_min[0], hi = s_max[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    lo = s_min[w] < lo ? s_min[w] : lo;
    hi = s_max[w] > hi ? s_max[w] : hi;
  }
  {
    const u32 span = (u32)kOctaveFloor << 23;
    const u32 floor_key = hi > span ? hi - span : 0u;
    lo = lo > floor_key ? lo : floor_key;
  }
  if (tid == 0 && j == 0) {
    img_flag[b] = hi >= 0x7F800000u ? TDQ_DEV_NONFINITE : 0u;
    if (b == 0) {                         // counts of sets the sampled interval misses
      status[1 + pass] = 0u;
      if (!keep_base) status[1 + (pass ^ 1)] = 0u;
    }
  }
  // ceil(j width / G) = j q + ceil(j rem / G) with width = q G + rem; everything fits 32 bits
  const u32 width = hi - lo + 1u, wq = width / (u32)G, wr = width - wq * (u32)G;
  const u32 start = j == 0 ? 0u : lo + (u32)j * wq + ((u32)j * wr + (u32)G - 1u) / (u32)G;
  const u32 end = j == G - 1 ? hi + 1u : lo + (u32)(j + 1) * wq + ((u32)(j + 1) * wr + (u32)G - 1u) / (u32)G;
  auto in_set = [&](u32 k) { return k >= start && k < end; };

  // ---- 2: the set's tokens
  u32 wcount = 0;
  for (int t0 = 0; t0 < T; t0 += kIdRounds * NT) {
    if (!one_batch) load_keys(t0);
#pragma unroll
    for (int u = 0; u < kIdRounds; ++u) wcount += (u32)__popcll(__ballot(in_set(kv[u])));
  }
  if (lane == 0) wtot[wave] = wcount;
  __syncthreads();
  u32 tokens_u = 0, running = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const u32 v = wtot[w];
    running += w < wave ? v : 0u;
    tokens_u += v;
  }
  if (tokens_u == 0) {
    if (tid == 0) {
      GroupWork w;
      w.n = 0; w.k_rem = 0; w.prefix = 0; w.tokens = 0; w.c_base = 0.f; w.sigma = 0.f;
      grp[idx] = w;
      Bracket e;
      e.lo = 0; e.width = 0; e.below = 0; e.pad = 0;
      br[idx] = e;
    }
    return;
  }
  // the sweep adds into this set's histogram: clear it here
  for (int i = tid; i < W; i += NT) bhist[(size_t)idx * W + i] = 0;

  // Sample geometry.  The set's tokens are cut into strata of `stride` tokens (at most
  // kSampleTokens strata) and one token is drawn from each at a hashed position: a regular
  // stride would alias with any period the token sequence has (image rows).  Of each drawn
  // token `rpt` runs of kRunLen consecutive channels are read, the first at a hashed offset,
  // so that all channels are represented; a row that fits is read whole.
  const int tokens = (int)tokens_u;
  const int stride = (tokens + kSampleTokens - 1) / kSampleTokens;
  const int n_sel = (tokens + stride - 1) / stride;         // <= kSampleTokens
  const int row_runs = (C + kRunLen - 1) / kRunLen;
  int rpt = kSampleRuns / n_sel;                            // runs per drawn token, >= 1
  rpt = rpt < row_runs ? rpt : row_runs;
  const int cw = rpt == row_runs ? C : rpt * kRunLen;       // channels read per drawn token
  const int n_runs = n_sel * rpt;                           // <= kSampleRuns
  const long long m = (long long)n_sel * cw;                // sample size, <= SM

  for (int t0 = 0; t0 < T; t0 += kIdRounds * NT) {
    if (!one_batch) load_keys(t0);
#pragma unroll
    for (int u = 0; u < kIdRounds; ++u) {
      const bool mine = in_set(kv[u]);
      const unsigned long long mask = __ballot(mine);
      if (mask == 0) continue;                              // uniform over the wavefront
      if (mine) {
        const int t = t0 + u * NT + tid;
        const u32 rank = running + (u32)__popcll(mask & ((1ull << lane) - 1ull));
        gb[t] = j;
        if (rank == 0) s_first = t;
        if (stride == 1) {
          sel[rank] = t;
        } else {
          const u32 stratum = rank / (u32)stride, first = stratum * (u32)stride;
          const u32 len = (u32)tokens - first < (u32)stride ? (u32)tokens - first : (u32)stride;
          const u32 pick =
              first + (((stratum + 1u) * 2246822519u + (u32)idx * 3266489917u) >> 12) % len;
          if (rank == pick) sel[stratum] = t;
        }
      }
      running += (u32)__popcll(mask);
    }
  }
  __syncthreads();

  // Moments of the set about the mean of its first token (zero if that is not finite: the
  // image's results are then undefined anyway and its flag is raised).  The loads are in
  // flight while the run table is made.
  const int first_token = s_first;
  double piv = meanb[first_token];
  const double cn = (double)C;
  double a1 = 0.0, a2 = 0.0;
  u32 cmax = 0;
  // table of runs, so that the load loop below has no division in it
  for (int q = tid; q < kSampleRuns; q += NT) {
    long long rbase = 0;
    int rl = 0;
    if (q < n_runs) {
      const int slot = q / rpt, run = q - slot * rpt;
      const int t = sel[slot];
      // (whole 16-byte pieces when the rows allow 16-byte loads: C, cw and the offset are
      // then multiples of 8 channels)
      const u32 off = vec ? (((u32)t * 2654435761u >> 8) % (u32)((C - cw) / 8 + 1)) * 8u
                          : ((u32)t * 2654435761u >> 8) % (u32)(C - cw + 1);
      rbase = ((long long)b * T + t) * ld + off + run * kRunLen;
      rl = cw - run * kRunLen;
      rl = rl < kRunLen ? rl : kRunLen;
    } else {
      rbase = ((long long)b * T + sel[0]) * ld;       // a valid address; the key is discarded
    }
    run_base[q] = rbase;
    run_len[q] = rl;
  }
  piv = (piv - piv == 0.0) ? piv : 0.0;
  for (int t0 = 0; t0 < T; t0 += kIdRounds * NT) {
    if (!one_batch) load_keys(t0);
    // half of the rounds at a time, their loads issued together (a token of another set
    // reads the first token's entry, which is not added)
#pragma unroll
    for (int h = 0; h < kIdRounds; h += kIdRounds / 2) {
      double mv[kIdRounds / 2], qv[kIdRounds / 2];
#pragma unroll
      for (int u = 0; u < kIdRounds / 2; ++u) {
        const bool mine = in_set(kv[h + u]);
        mv[u] = piv;
        qv[u] = 0.0;
        if (__ballot(mine)) {                         // uniform over the wavefront
          const int t = mine ? t0 + (h + u) * NT + tid : first_token;
          mv[u] = meanb[t];
          qv[u] = m2b[t];
        }
      }
#pragma unroll
      for (int u = 0; u < kIdRounds / 2; ++u) {
        const u32 k = kv[h + u];
        const bool mine = in_set(k);
        const double dm = mv[u] - piv;
        const double d1 = cn * dm;
        a1 += mine ? d1 : 0.0;
        a2 += mine ? qv[u] + d1 * dm : 0.0;
        cmax = mine && k > cmax ? k : cmax;
      }
    }
  }
  a1 = group_sum_f64<64>(a1);                         // totals in lane 63
  a2 = group_sum_f64<64>(a2);
  cmax = group_max_u32<64>(cmax);
  if (lane == 63) { s_s1[wave] = a1; s_s2[wave] = a2; s_cmax[wave] = cmax; }
  __syncthreads();

  // ---- 3: the sample.  Every live key adds one to an LDS histogram of its top kSampleBits
  // bits.  Loads are issued unconditionally (from a clamped, valid address) so that they
  // overlap.
  if (vec) {
    // 16-byte pieces of 8 channels: piece p = NT e + tid is part p % 4 of run p / 4, so a
    // wavefront's load instruction fetches 16 whole runs of 64 bytes; a run's pieces are
    // all live or (runs past the end of the table) all dead.
    constexpr int kPieces = SM / 8 / NT;
    uint4 v[kPieces];
    bool live[kPieces];
#pragma unroll
    for (int e = 0; e < kPieces; ++e) {
      const int p = e * NT + tid;
      const int q = p >> 2, part = p & 3;
      live[e] = part * 8 < run_len[q];
      v[e] = *reinterpret_cast<const uint4*>(X + run_base[q] + (live[e] ? part * 8 : 0));
    }
#pragma unroll
    for (int e = 0; e < kPieces; ++e) {
      if (live[e]) {
        const u32 wd[4] = {v[e].x, v[e].y, v[e].z, v[e].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          atomicAdd(&shist[(wd[i] & 0x7FFFu) >> (15 - kSampleBits)], 1u);
          atomicAdd(&shist[((wd[i] >> 16) & 0x7FFFu) >> (15 - kSampleBits)], 1u);
        }
      }
    }
  } else {
    // element e of lane l of wavefront w is channel l % 32 of run 2 NW e + 2 w + l / 32
    constexpr int kPerThread = SM / NT;
    u32 key[kPerThread];
    const int half = lane >> 5, cl = lane & 31;
#pragma unroll
    for (int e = 0; e < kPerThread; ++e) {
      const int q = e * (2 * NW) + 2 * wave + half;
      const int rl = run_len[q];
      const int ch = cl < rl ? cl : (rl > 0 ? rl - 1 : 0);
      const u32 x = X[run_base[q] + ch];
      key[e] = cl < rl ? (x & 0x7FFFu) : 0xFFFFu;
    }
#pragma unroll
    for (int e = 0; e < kPerThread; ++e)
      if (key[e] != 0xFFFFu) atomicAdd(&shist[key[e] >> (15 - kSampleBits)], 1u);
  }

  // the set's working record: n, base radius, sigma, rank of this pass (binary64)
  GroupWork w;
  w.tokens = tokens_u;
  w.n = (long long)tokens * (long long)C;
  w.prefix = 0;
  const double n = (double)w.n;
  w.k_rem = (long long)ceil((pass == kPassBase ? sc.base_pct : sc.zr) * n);
  w.k_rem = w.k_rem < 1 ? 1 : (w.k_rem > w.n ? w.n : w.k_rem);
  if (tid == 0) {
    double S1 = s_s1[0], S2 = s_s2[0];
    u32 km = s_cmax[0];
    for (int i = 1; i < NW; ++i) {
      S1 += s_s1[i];
      S2 += s_s2[i];
      km = s_cmax[i] > km ? s_cmax[i] : km;
    }
    const double mu = S1 / n;
    double var = S2 / n - mu * mu;
    var = var > 0.0 ? var : 0.0;
    w.sigma = (float)(sqrt(var) + sc.eps_std);
    // (the base-radius pass left its radius in the record)
    w.c_base = keep_base ? grp[idx].c_base : __uint_as_float(km);
    grp[idx] = w;
  }
  __syncthreads();

  // Sample rank that corresponds to rank k of the set, and the histogram bin that
  // holds that order statistic (the low key bits do not matter to the interval).
  long long rk = (long long)((double)w.k_rem / n * (double)m + 0.5);
  rk = rk < 1 ? 1 : (rk > m ? m : rk);
  constexpr int kBinsPerThread = (1 << kSampleBits) / NT;
  u32 c[kBinsPerThread], mine = 0;
#pragma unroll
  for (int i = 0; i < kBinsPerThread; ++i) {
    c[i] = shist[tid * kBinsPerThread + i];
    mine += c[i];
  }
  u32 incl = mine;                           // inclusive scan over the wavefront
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const u32 o = (u32)__shfl_up((int)incl, d, 64);
    if (lane >= d) incl += o;
  }
  if (lane == 63) stot[wave] = incl;
  __syncthreads();
#pragma unroll
  for (int w2 = 0; w2 < NW; ++w2) incl += w2 < wave ? stot[w2] : 0u;
  if ((long long)(incl - mine) < rk && rk <= (long long)incl) {     // exactly one thread
    u32 cum = incl - mine;
    int i = 0;
    for (; i < kBinsPerThread - 1; ++i) {
      if ((long long)(cum + c[i]) >= rk) break;
      cum += c[i];
    }
    const u32 v = (u32)(tid * kBinsPerThread + i) << (15 - kSampleBits);
    // v <= estimate < v + 2^(15 - kSampleBits): centre the interval on the middle
    const u32 mid = v + (1u << (14 - kSampleBits));
    Bracket e;
    e.below = 0; e.pad = 0;
    e.lo = mid > (u32)W / 2 ? mid - (u32)W / 2 : 0u;
    e.width = (u32)W;
    br[idx] = e;
  }
}

hipError_t launch_sets(const void* X, int B, int T, int C, long long ld, int G, int W, const float* r,
                       const double* mean, const double* m2, int* gid, const Scalars& sc, int pass,
                       bool keep_base, GroupWork* grp, Bracket* br, unsigned* bhist,
                       unsigned* img_flag, unsigned* status, hipStream_t st) {
  // 16-byte sample loads need rows of whole, aligned 16-byte pieces
  const int vec = ((reinterpret_cast<uintptr_t>(X) & 15) == 0 && ld % 8 == 0 && C % 8 == 0) ? 1 : 0;
#define TDQ_SETS_SM(NT, SM)                                                                        \
  hipLaunchKernelGGL((k_sets<NT, SM>), dim3(G, B), dim3(NT), 0, st, static_cast<const u16*>(X), ld, \
                     T, C, G, W, vec, r, mean, m2, gid, sc, pass, keep_base ? 1 : 0, grp, br, bhist, \
                     img_flag, status)
#define TDQ_SETS(NT)                                        \
  do {                                                      \
    if (W >= 512) TDQ_SETS_SM(NT, 8192); else TDQ_SETS_SM(NT, 16384); \
  } while (0)
  // as few threads as hold the image's range keys in registers: [32, 4096, 1024] calibrates
  // in 111 / 117 / 145 us with 256 / 512 / 1024 threads per set
  if (T <= kIdRounds * 256)
    TDQ_SETS(256);
  else if (T <= kIdRounds * 512)
    TDQ_SETS(512);
  else
    TDQ_SETS(1024);
#undef TDQ_SETS
#undef TDQ_SETS_SM
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// k_bracket_hist: the one sweep
// ---------------------------------------------------------------------------
typedef short s2v __attribute__((ext_vector_type(2)));

// A group of L lanes takes R rows at a time and P pieces of 16 bytes of each: the set ids
// and all R P = 4 pieces are loaded before the first is looked at, so a wavefront has four
// kilobytes in flight whatever the row length -- what bounds this sweep otherwise is the
// chain set id -> interval -> piece of one row after another.  Measured, this kernel alone:
// [8, 7744, 512] 25.6 -> 17.1 us, [32, 4096, 1024] 52.1 -> 46.5 (5.8 TB/s), [16, 484, 320]
// 13.4 -> 6.1, [5, 1369, 333] (rows at odd addresses, read element by element before) 20.7 ->
// 7.5; without the in-loop histogram additions it takes the same time, without the final
// global additions 13.2 and 44.6 us on the first two.
template <int L, int P>
__global__ __launch_bounds__(kSweepThreads) void k_bracket_hist(
    const u16* __restrict__ X, long long ld, int T_, int C, int G, int W,
    const int* __restrict__ gid, Bracket* __restrict__ br, u32* __restrict__ bhist,
    int rows_per_block) {
  constexpr int R = 4 / P;
  extern __shared__ u32 lds[];                    // [G][W] bins, then per set: below, lo, width
  // walks X backwards: it runs right after the forward statistics sweep, so the end of
  // X is what the last-level cache still holds
  const int b = (int)(gridDim.y - 1 - blockIdx.y);
  const int chunk = (int)(gridDim.x - 1 - blockIdx.x);
  const int tid = threadIdx.x;
  const int nwords = G * W;
  u32* s_below = lds + nwords;
  u32* s_lo = s_below + G;
  u32* s_width = s_lo + G;
  for (int i = tid; i < nwords + G; i += kSweepThreads) lds[i] = 0;
  for (int g = tid; g < G; g += kSweepThreads) {
    const Bracket e = br[(long long)b * G + g];
    s_lo[g] = e.lo;
    s_width[g] = e.width;
  }
  __syncthreads();

  const int row0 = chunk * rows_per_block;
  int nrows = T_ - row0;
  nrows = nrows < rows_per_block ? nrows : rows_per_block;
  constexpr int SLOTS = kSweepThreads / L;
  const int slot = tid / L, lr = tid % L;
  const int nvec = C / 8;
  const long long first = (long long)b * T_ + row0;
  for (int rr = slot; rr < nrows; rr += SLOTS * R) {
    const u16* xp[R];
    int g[R];
    u32 below[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {                 // rows past the end: the last one, not counted
      const int ri = rr + SLOTS * i;
      const long long row = first + (ri < nrows ? ri : nrows - 1);
      xp[i] = X + row * ld;
      g[i] = gid[row];
      below[i] = 0;
    }
    for (int v0 = lr; v0 < nvec; v0 += P * L) {
      uint4 q[R][P];
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int k = 0; k < P; ++k) {
          const int v = v0 + k * L;
          q[i][k] = load16(xp[i] + (long long)(v < nvec ? v : v0) * 8);
        }
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const u32 lo = s_lo[g[i]], width = s_width[g[i]];
        const u32 lo2 = lo | (lo << 16);
        u32* h = lds + g[i] * W;
        if (rr + SLOTS * i < nrows) {
#pragma unroll
          for (int k = 0; k < P; ++k) {
            if (k > 0 && v0 + k * L >= nvec) break;
            const u32 wd[4] = {q[i][k].x, q[i][k].y, q[i][k].z, q[i][k].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              // both halves at once: keys and lo are below 2^15, so the 16-bit differences
              // cannot overflow and their sign bits say "key < lo"
              const s2v d = __builtin_bit_cast(s2v, wd[e] & 0x7FFF7FFFu) - __builtin_bit_cast(s2v, lo2);
              const u32 d2 = __builtin_bit_cast(u32, d);
              below[i] += (u32)__builtin_popcount(d2 & 0x80008000u);
              const u32 dl = d2 & 0xFFFFu, dh = d2 >> 16;     // negative ones are >= 2^15 > width
              if (dl < width) atomicAdd(&h[dl], 1u);
              if (dh < width) atomicAdd(&h[dh], 1u);
            }
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (rr + SLOTS * i < nrows) {
        const u32 lo = s_lo[g[i]], width = s_width[g[i]];
        for (int c = nvec * 8 + lr; c < C; c += L) {          // fewer than 8 elements
          const u32 k = xp[i][c] & 0x7FFFu;
          below[i] += k < lo ? 1u : 0u;
          const u32 d = k - lo;
          if (k >= lo && d < width) atomicAdd(&lds[g[i] * W + d], 1u);
        }
      }
      const u32 total = group_sum_u32<L>(below[i]);           // in the row's last lane
      if (lr == L - 1 && total) atomicAdd(&s_below[g[i]], total);
    }
  }
  __syncthreads();
  u32* gh = bhist + (size_t)b * G * W;
  for (int i = tid; i < nwords; i += kSweepThreads) {
    const u32 v = lds[i];
    if (v) atomicAdd(&gh[i], v);
  }
  for (int g = tid; g < G; g += kSweepThreads) {
    const u32 v = s_below[g];
    if (v) atomicAdd(&br[(long long)b * G + g].below, v);
  }
}

hipError_t launch_bracket_hist(const void* Xv, int B, int T_, int C, long long ld, int G, int W,
                               const int* gid, Bracket* br, unsigned* bhist, hipStream_t st) {
  const u16* X = static_cast<const u16*>(Xv);
  const int nvec = C / 8;
  const int L = sweep_lanes_per_row(C, 8);
  const int P = nvec > 2 * L ? 4 : nvec > L ? 2 : 1;
  // Two workgroups per CU where that leaves each 128 Ki elements, one otherwise, and at
  // least 32 Ki elements each: every workgroup clears G W bins and adds the non-zero ones to
  // the image's with global atomics, which is what more workgroups cost.  Calibration of
  // [8, 7744, 512] with 512 / 256 workgroups 47.3 / 44.5 us, of [32, 4096, 1024] 106.6 /
  // 107.5; of [8, 1936, 320] with at least 32 / 16 / 8 Ki elements 40.5 / 41.9 / 44.1 us, of
  // [8, 121, 512] 19.3 / 18.9 / 19.0 (64 Ki: 21.5).
  const long long total = (long long)B * T_ * C;
  const long long rows_min = (32768 + C - 1) / C;
  long long target_blocks = (total >= 512ll * 131072 ? 512 : 256) / B;
  if (target_blocks < 1) target_blocks = 1;
  long long rpb = (T_ + target_blocks - 1) / target_blocks;
  if (rpb < rows_min) rpb = rows_min;
  if (rpb > T_) rpb = T_;
  const unsigned chunks = (unsigned)((T_ + rpb - 1) / rpb);
  const size_t lds_bytes = ((size_t)G * W + 3 * (size_t)G) * sizeof(u32);
#define TDQ_BH(LL, PP)                                                                          \
  if (L == LL && P == PP) {                                                                     \
    if (lds_bytes > 65536)                                                                      \
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bracket_hist<LL, PP>),         \
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);    \
    hipLaunchKernelGGL((k_bracket_hist<LL, PP>), dim3(chunks, B), dim3(kSweepThreads), lds_bytes, \
                       st, X, ld, T_, C, G, W, gid, br, bhist, (int)rpb);                       \
  }
  TDQ_BH(1, 1) TDQ_BH(2, 1) TDQ_BH(4, 1) TDQ_BH(8, 1) TDQ_BH(8, 2) TDQ_BH(8, 4) TDQ_BH(16, 2)
  TDQ_BH(16, 4) TDQ_BH(32, 2) TDQ_BH(32, 4) TDQ_BH(64, 2) TDQ_BH(64, 4)
#undef TDQ_BH
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// k_bracket_finish: one workgroup per set.  Its first wavefront verifies the interval
// and, on a hit, finishes the set; on a miss the whole workgroup runs the exact
// two-level radix select (8 + 7 key bits, LDS histogram) over the set's own rows.
// ---------------------------------------------------------------------------
constexpr int kFinishThreads = 256;

__global__ __launch_bounds__(kFinishThreads) void k_bracket_finish(
    const u16* __restrict__ X, long long ld, int T, int C, int G, int vec_ok,
    const int* __restrict__ gid, const u32* __restrict__ bhist, int W, int force_miss, Scalars sc,
    int pass, GroupWork* __restrict__ grp, const Bracket* __restrict__ br,
    float* __restrict__ clip, float* __restrict__ scale, tdq_group_stats* __restrict__ stats,
    const u32* __restrict__ img_flag, int B, u32* __restrict__ status) {
  __shared__ u32 h[256];
  __shared__ int list[kFinishThreads];
  __shared__ u32 wtot[kFinishThreads / 64];
  __shared__ u32 s_ok, s_digit;
  __shared__ unsigned long long s_rem;
  const int idx = blockIdx.x;
  const int b = idx / G, j = idx - b * G;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (idx == 0 && wave == 0 && pass == kPassZr) {   // fold the per-image flags into the status word
    u32 f = 0;
    for (int bb = lane; bb < B; bb += 64) f |= img_flag[bb];
    const unsigned long long any = __ballot(f != 0);
    if (lane == 0) status[0] = any ? TDQ_DEV_NONFINITE : 0u;
  }
  const GroupWork w = grp[idx];
  if (w.tokens == 0) {
    if (tid == 0 && pass == kPassZr) project_store(idx, w, 0u, true, sc, clip, scale, stats);
    return;
  }
  if (wave == 0) {
    bool ok = false;
    unsigned long long need = 0, mine = 0, incl = 0;
    const u32* hb = bhist + (size_t)idx * W;
    const int per = W / 64;                     // W is a multiple of 64
    const int first = lane * per;
    Bracket e;
    e.lo = 0; e.width = 0; e.below = 0; e.pad = 0;
    if (!force_miss) {
      e = br[idx];
      const unsigned long long k = (unsigned long long)w.k_rem;
      for (int i = 0; i < per; ++i) mine += hb[first + i];
      incl = mine;                              // inclusive scan over lanes
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
      }
      const unsigned long long inside = __shfl(incl, 63, 64);
      ok = k > e.below && k - e.below <= inside;
      need = k - e.below;
    }
    if (ok) {                                   // wavefront-uniform
      const unsigned long long hit = __ballot(incl >= need);
      const int src = __ffsll((long long)hit) - 1;        // hit != 0 because need <= inside
      if (lane == src) {
        unsigned long long cum = incl - mine;
        int i = 0;
        for (; i < per - 1; ++i) {
          const unsigned long long c = hb[first + i];
          if (cum + c >= need) break;
          cum += c;
        }
        const u32 key = e.lo + (u32)(first + i);
        if (pass == kPassBase)
          grp[idx].c_base = h2f(key);            // the set's base radius Q_p(|x|)
        else
          project_store(idx, w, key, true, sc, clip, scale, stats);
      }
    }
    if (lane == 0) s_ok = ok ? 1u : 0u;
  }
  __syncthreads();
  if (s_ok) return;

  // The interval missed rank k (or the validation switch asked for this route).
  if (tid == 0) atomicAdd(&status[1 + pass], 1u);
  const int* gb = gid + (long long)b * T;
  unsigned long long k = (unsigned long long)w.k_rem;
  u32 prefix = 0;
  const int nvec = vec_ok ? C / 8 : 0;
  for (int level = 0; level < 2; ++level) {
    const int shift = level == 0 ? 7 : 0;
    const u32 mask = level == 0 ? 255u : 127u;
    h[tid] = 0;                                 // kFinishThreads == 256 bins
    __syncthreads();
    for (int t0 = 0; t0 < T; t0 += kFinishThreads) {
      // the set's tokens among t0 .. t0 + 255, compacted into `list`
      const int t = t0 + tid;
      const bool match = t < T && gb[t] == j;
      const unsigned long long m = __ballot(match);
      if (lane == 0) wtot[wave] = (u32)__popcll(m);
      __syncthreads();
      u32 before = 0, n_list = 0;
#pragma unroll
      for (int w2 = 0; w2 < kFinishThreads / 64; ++w2) {
        before += w2 < wave ? wtot[w2] : 0u;
        n_list += wtot[w2];
      }
      if (match) list[before + (u32)__popcll(m & ((1ull << lane) - 1ull))] = t;
      __syncthreads();
      for (u32 i = wave; i < n_list; i += kFinishThreads / 64) {     // one wavefront per row
        const u16* xp = X + ((long long)b * T + list[i]) * ld;
        for (int v = lane; v < nvec; v += 64) {
          const uint4 q = *reinterpret_cast<const uint4*>(xp + (long long)v * 8);
          const u32 wd[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const u32 k0 = wd[c] & 0x7FFFu, k1 = (wd[c] >> 16) & 0x7FFFu;
            if (level == 0 || (k0 >> 7) == prefix) atomicAdd(&h[(k0 >> shift) & mask], 1u);
            if (level == 0 || (k1 >> 7) == prefix) atomicAdd(&h[(k1 >> shift) & mask], 1u);
          }
        }
        for (int c = nvec * 8 + lane; c < C; c += 64) {
          const u32 k0 = xp[c] & 0x7FFFu;
          if (level == 0 || (k0 >> 7) == prefix) atomicAdd(&h[(k0 >> shift) & mask], 1u);
        }
      }
      __syncthreads();                          // `list` and `wtot` are reused
    }
    if (tid == 0) {
      unsigned long long cum = 0;
      const int nb = level == 0 ? 256 : 128;
      int bin = 0;
      for (; bin < nb - 1; ++bin) {
        if (cum + h[bin] >= k) break;
        cum += h[bin];
      }
      s_digit = (u32)bin;
      s_rem = k - cum;
    }
    __syncthreads();
    prefix = level == 0 ? s_digit : ((prefix << 7) | s_digit);
    k = s_rem;
    __syncthreads();
  }
  if (tid == 0) {
    if (pass == kPassBase)
      grp[idx].c_base = h2f(prefix);
    else
      project_store(idx, w, prefix, true, sc, clip, scale, stats);
  }
}

hipError_t launch_bracket_finish(const void* Xv, int B, int T, int C, long long ld, int G, int W,
                                 const int* gid, const unsigned* bhist, bool force_miss,
                                 const Scalars& sc, int pass, GroupWork* grp, const Bracket* br,
                                 float* clip, float* scale, tdq_group_stats* stats,
                                 const unsigned* img_flag, unsigned* status, hipStream_t st) {
  const u16* X = static_cast<const u16*>(Xv);
  const int vec_ok = ((reinterpret_cast<uintptr_t>(X) & 15) == 0 && ld % 8 == 0) ? 1 : 0;
  hipLaunchKernelGGL(k_bracket_finish, dim3(B * G), dim3(kFinishThreads), 0, st, X, ld, T, C, G,
                     vec_ok, gid, bhist, W, force_miss ? 1 : 0, sc, pass, grp, br, clip, scale, stats,
                     img_flag, B, status);
  return hipGetLastError();
}

}  // namespace tdq
