// C ABI of libtdq: argument validation on the host, workspace layout, and the
// launch sequence of each entry point.  Nothing here computes on the data.
#include <math.h>
#include <atomic>
#include <stdlib.h>
#include <string.h>

#include "tdq_device.hpp"

namespace tdq {

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

LevelPlan make_level_plan(tdq_dtype dt, int G) {
  LevelPlan lp;
  memset(&lp, 0, sizeof(lp));
  lp.key_bits = dt == TDQ_F16 ? 15 : 31;
  int max_bits = 0;
  while ((G << (max_bits + 1)) <= kHistLdsWords && max_bits + 1 <= kMaxLevelBits) ++max_bits;
  if (max_bits < 1) max_bits = 1;
  int n = (lp.key_bits + max_bits - 1) / max_bits;
  static_assert(31 <= 5 * kMaxLevels && ((TDQ_MAX_GROUPS << 5) <= kHistLdsWords),
                "the level arrays must hold the plan of the largest set count");
  lp.n_levels = n;
  int left = lp.key_bits;
  for (int l = 0; l < n; ++l) {
    const int levels_left = n - l;
    int b = (left + levels_left - 1) / levels_left;     // spread the bits evenly
    lp.bits[l] = b;
    left -= b;
    lp.shift[l] = left;
  }
  return lp;
}

int bracket_bins(int G) {
  int w = 2048;
  while (w >= kBracketMinBins && (long long)G * w > kBracketLdsWords) w >>= 1;
  return w >= kBracketMinBins ? w : 0;
}

int bracket_bins_zr(int G) {
  const int most = bracket_bins(G);
  int w = 2048;
  while (w > 512 && G * w > kBracketLdsWords / 2) w >>= 1;
  return w < most ? w : most;
}

WorkspaceLayout make_layout(int B, int T, int G, const LevelPlan& lp) {
  WorkspaceLayout w;
  memset(&w, 0, sizeof(w));
  const size_t M = (size_t)B * T, BG = (size_t)B * G;
  size_t off = 0;
  w.status = off;   off = align256(off + 64 * sizeof(unsigned));
  w.img_flag = off; off = align256(off + (size_t)B * sizeof(unsigned));
  w.r = off;        off = align256(off + M * sizeof(float));
  w.mean = off;     off = align256(off + M * sizeof(double));
  w.m2 = off;       off = align256(off + M * sizeof(double));
  w.part = off;     off = align256(off + assign_partial_bytes(B, G));
  w.grp = off;      off = align256(off + BG * sizeof(GroupWork));
  w.hist = off;
  for (int l = 0; l < lp.n_levels; ++l) {
    w.hist_level[l] = off;
    off += BG * ((size_t)1 << lp.bits[l]) * sizeof(unsigned);   // levels are contiguous
  }
  off = align256(off);
  w.br = off;       off = align256(off + BG * sizeof(Bracket));
  w.bhist = off;    off = align256(off + BG * (size_t)bracket_bins(G) * sizeof(unsigned));
  w.total = align256(off);
  return w;
}

// blocks = false: the token-set entry points (chan_group must be 0); true: the
// per-(token, 32-channel block) entry points (chan_group must be 32).
static int check_params(const tdq_params* p, bool blocks = false) {
  if (!p) return TDQ_ERR_NULL;
  if (p->n_groups < 1 || p->n_groups > TDQ_MAX_GROUPS) return TDQ_ERR_PARAM;
  if (p->act_bits != 4) return p->act_bits == 8 ? TDQ_ERR_UNSUPPORTED : TDQ_ERR_PARAM;
  if (p->flags & ~(TDQ_FLAG_C1 | TDQ_FLAG_C2 | TDQ_FLAG_EXACT_SELECT)) return TDQ_ERR_PARAM;
  if (!(p->tau > 0.0) || !isfinite(p->tau)) return TDQ_ERR_PARAM;
  if (!(p->zr > 0.0 && p->zr < 1.0)) return TDQ_ERR_PARAM;
  if (!(p->eps_scale > 0.f) || !(p->eps_std >= 0.f)) return TDQ_ERR_PARAM;
  if (p->chan_group < 0) return TDQ_ERR_PARAM;
  if (p->chan_group != (blocks ? TDQ_BLOCK : 0)) return TDQ_ERR_UNSUPPORTED;
  if (!(p->base_pct >= 0.0 && p->base_pct <= 1.0)) return TDQ_ERR_PARAM;
  return TDQ_OK;
}

static int check_shape(int32_t B, int32_t T, int32_t C, int64_t ld_x) {
  if (B < 1 || T < 1 || C < 1 || B > TDQ_MAX_IMAGES) return TDQ_ERR_SHAPE;
  if (ld_x < C) return TDQ_ERR_SHAPE;
  if ((int64_t)B * T > (int64_t)1 << 30) return TDQ_ERR_SHAPE;
  return TDQ_OK;
}

// Rank ceil(frac g) among the g values of a block, padding zeros included (binary64, as
// everywhere).
static int block_rank(double frac) {
  long long k = (long long)ceil(frac * (double)TDQ_BLOCK);
  return (int)(k < 1 ? 1 : (k > TDQ_BLOCK ? TDQ_BLOCK : k));
}

static Scalars make_scalars(const tdq_params* p) {
  Scalars s;
  s.qmax = (float)kQMax;
  s.qmax_tau = (float)kQMax * (float)p->tau;   // binary32 product, as in the definition
  s.two_qmax = 2.0f * (float)kQMax;
  s.eps_scale = p->eps_scale;
  s.eps_std = (double)p->eps_std;
  s.zr = p->zr;
  s.base_pct = (p->base_pct > 0.0 && p->base_pct < 1.0) ? p->base_pct : 0.0;
  s.flags = p->flags;
  s.inv_groups = 1.0 / (double)p->n_groups;
  return s;
}

// Whether the image takes the radix levels (a sweep per eight to five key bits, whatever the data)
// because of its sets.  The sampled route's first and last kernels have a workgroup per set, and in the
// first each reads the image's T ranges; figures below are us, sampled against levels.
//   * Thousands of sets of no more than 4096 elements: [256, 64, 768] with 16 sets, binary32 102 and
//     93, binary16 56 and 49; [256, 1024, 8] 88 and 60, 57 and 39; [512, 49, 768] with 64 sets, binary16,
//     247 and 147; [2048, 49, 96] 808 and 265.  Of 8192 elements a set the sampled route is faster
//     everywhere, and up to 4096 sets it is with few sets an image ([1024, 64, 128] with 4, binary32:
//     107 and 133) or many ([64, 256, 768] with 64: 101 and 115, 58 and 75).
//   * More tokens to look at than elements, and more workgroups than run at once: [64, 16384, 8] with 32
//     sets, binary32 202 and 130, binary16 141 and 91; [256, 16384, 8] 728 and 356, 553 and 253; but
//     [16, 65536, 8] with 16 sets 124 and 148, 97 and 113.
static bool many_small_sets(int B, int T, int C, int G) {
  const long long sets = (long long)B * G;
  if (sets > (G >= 8 && G <= 32 ? 2048 : 4096) && (long long)T * C <= 4096ll * G) return true;
  return sets > 512 && sets * T >= 1ll << 23 && C <= G;
}

// Whether a binary32 image may sample (two sweeps of X).
//   * A bin that collects more keys than a list holds, or an interval that misses, costs a search
//     of the set's rows by one workgroup: 50 us for 0.2 M elements, 200 for 1 M, against 50 to 70 for
//     all radix levels of such an image.  So images stay below 1 Mi elements, 0.6 Mi with more
//     than 32 sets, whose lists are short.
//   * A set of many tokens is one workgroup's chain of T / 1024 steps, which a small image's levels
//     undercut: [1, 400000, 1], one set: 239 us by levels, 473 sampled; 16 sets 467 and 470;
//     [1, 100000, 8], 5 sets: 117 and 159; 16 sets 166 and 130; [1, 16385, 33], one set: 69 and 57.
static bool sampled_f32(int T, int C, int G) {
  if (T > 32768 && T > 16384ll * G) return false;
  return (long long)T * C < (G <= 32 ? 1ll << 20 : 638976ll);
}

// Whether a calibration samples; the validation switch searches every set of a binary16 image and
// takes the radix levels for a binary32 one.
static bool samples_rank(tdq_dtype dt, int B, int T, int C, int G, bool exact_only) {
  if (bracket_bins(G) == 0) return false;              // too many sets for the interval histogram
  if (dt == TDQ_F16 && (long long)T * C >= 1ll << 32) return false;
  if (dt == TDQ_F16 && exact_only) return true;
  return !exact_only && !many_small_sets(B, T, C, G) && (dt == TDQ_F16 || sampled_f32(T, C, G));
}

// Whether one kernel does assignment and rank select together (k_sets with WHOLE), and if so with how many workgroups per
// image beyond one per set (-1 = no).  Every limit has its reason beside it.  Figures are us of one calibration (binary16
// with few elements: of the layer), in the order that the text names; "the chain" is what takes the call otherwise, three or
// four kernels after the statistics, five with binary32, ten with the radix levels.

// binary16: a workgroup counts its share of a set's rows and leaves, the last to arrive picks.
static int whole_extra_f16(int B, int T, int C, int G, bool two_ranks) {
  const long long e = (long long)T * C;
  // Three workgroups fit a CU, so these take two turns on the chip at most.  One kernel and chain: [49, 74, 832] with 32
  // sets (1568) 31.0 / 29.8, [58, 20, 9] with 32 42.8 / 36.6, [64, 322, 56] with 64 55.7 / 45.6; of 94 calls of 1024 to
  // 1536 sets none is slower.
  if ((long long)B * G > 1536) return -1;
  // One for every 8 Ki elements, 512 in all (two per CU): with one for 64 / 16 / 8 Ki [8, 121, 512] with 16 sets
  // 22.1 / 22.0 / 21.1, [16, 484, 320] 35.8 / 34.2 / 33.2.
  long long extra = e / 8192;
  const long long most = 512 / B - G;
  if (extra > most) extra = most > 0 ? most : 0;
  // Every workgroup of a set repeats the search for its tokens and its interval, so a large batch is better off with one
  // sweep over all sets.  Elements for each, no more than this.
  long long share;
  if (two_ranks) {
    // Two ranks share the set's words of the workspace if several meet in them: 512 bins each are the least.
    if (extra > 0 && bracket_bins(G) < 1024) return -1;
    share = 65536;                                     // (two sweeps by the chain; [14, 5850, 160], 29 Ki, 97.9 / 122.3)
  } else {
    // Fewer than 64 beyond the first for a set, which all meet in the same words: [3, 2125, 1669] with one set, 169 of
    // them, 39.0 / 33.6, [2, 5545, 419] with two 36.8 / 30.3; with 32 to 64 of them 41 calls 1.22 times as fast.
    if (extra >= 64 * G) return -1;
    // More than 8 Ki each: at least a quarter of the rows that its lanes take at a time ([2, 457, 6172] with 16 sets, two
    // rows for eight wavefronts, 43.8 / 39.5).
    const int slots = 512 / sweep_lanes_per_row(C, 8);
    if (e > 8192 * (extra + 1) && 4ll * T < slots * (extra + 1)) return -1;
    // One or two sets of many tokens, each read by every workgroup: 16 Ki ([58, 6152, 44] 52.7 / 47.8).
    if (G <= 2 && T > 4096 && e > 16384 * (extra + 1)) return -1;
    // With three to a set on average 80 Ki, about where the two are even.  Calls over 7 laws of an encoder's activations
    // (as they are, clamped, after a rectifier or a GELU), in the geometric mean 0.98 times the chain's time from 40 to 64 Ki
    // (606 calls, 38 of them more than 5 % slower), 1.00 to 80 (205, 26), 1.02 to 96, 1.03 to 128; over 19 other laws (ties,
    // grids, gaps, constants) 0.89 to 64 Ki (824, 85), 0.88 to 80 (317, 40).  [8, 7744, 512] with 16 sets, 79 Ki, 40.8 / 42.9,
    // [4, 8000, 1024] 40.7 / 46.2; after a rectifier 1.04 times the chain's time throughout, [15, 4450, 216] 35.3 / 30.6, [2,
    // 4808, 3283] with 24 87.4 / 73.4.  Sets that miss their interval have one workgroup search their rows alone, in the
    // chain too: 170 such calls 0.73, but one set of [4, 8079, 812] 850 / 631, 31 of [3, 2506, 2922] 623 / 398.
    // With fewer one set may hold nearly all rows: 40 Ki.  From there to 80 Ki such calls are even on an encoder's laws (589
    // calls, 1.01), but one in seven takes 1.1 times the chain's time or more: [27, 2800, 79] with 16 sets, two beyond one
    // each, 49.0 / 35.3, [27, 166, 1095] 36.1 / 26.8.
    share = extra >= 2 * G ? 81920 : 40960;
  }
  return e <= share * (extra + 1) ? (int)extra : -1;
}

// binary32: one workgroup to a set, or several that wait for each other.
static int whole_extra_f32(int B, int T, int C, int G, bool two_ranks) {
  const long long e = (long long)T * C;
  // Two turns on the chip, as above, but two workgroups a CU, and with two ranks one: [42, 3, 2424] with 32 sets (1344)
  // 48.2 / 41.9; percentile [52, 25, 8] with 16 (832) 72.4 / 60.4, [120, 13, 3821] with 5 (600) 137 / 117, but [292, 187,
  // 8] with 2 (584) 43.0 / 79.8.
  if ((long long)B * G > (two_ranks ? 512 : 1024)) return -1;
  // One workgroup sees all of a set ([2, 1400, 32], 45 Ki elements, 38.6 / 44.7); an image that is one set by itself 40 Ki
  // ([2, 576, 74], 42 Ki, 45.0 / 34.1).
  if (e <= (G == 1 ? 40960 : 57344)) return 0;
  // Beyond that several share a set: with one rank, and 2 to 32 sets (256 bins and 256 keys of a set have room then).  Each
  // keeps its slot of a CU while it waits.  [2, 484, 320] with 8 sets 20.8 / 33.4, [24, 300, 300] with 16 29.3 / 41.7, [16,
  // 1024, 1024] 65 / 103, [1, 8192, 1024] with 8 60 / 73.  Over an encoder's laws 800 calls take 0.62 times the chain's time,
  // over 19 laws of data (Laplace, rectified, masked, clamped, with ties, on a grid, constant, ...; T from 2, C up to 256 Ki)
  // 760 calls 0.61.  More than 5 % slower are, of 716 calls of two to four sets, where a second round reads many rows again,
  // 18: values on a grid [7, 905, 864] with two 61.4 / 47.8, [3, 3676, 356] with three 90 / 68; two groups of values [6, 179,
  // 3932] with three 52.5 / 45.7; 19 % zeros [2, 440, 2208] with two 46 / 40; of the calls of more sets those of one
  // value, [17, 61, 4268] 80.4 / 66.5.
  if (two_ranks || G == 1 || G > 32) return -1;
  // One for every 8 Ki elements, of as many as the chip holds 64 Ki for each, 256 of them to an image ([1, 8192, 1024] with 8
  // sets 97 with 496 of them, 74 with 240).
  long long extra = e / 8192;
  if (extra > 512 / B - G) extra = 512 / B - G;
  if (extra > 256) extra = 256;
  if (e > 65536 * (extra + 1)) return -1;
  // One slot in 32 stays free, for kernels of calls on other streams, which costs a call alone nothing: [8, 1024, 768] with 16
  // sets on one and on eight streams, a call, by the chain 46.8 and 21.5, by 512 workgroups 33.0 and 29.0, by 496 32.8 and
  // 27.4, by 480 33.8 and 26.4; [4, 4096, 768] 90.4 and 46.8, 54.5 and 53.2, 52.8 and 51.5, 53.2 and 49.9.
  if (extra > 496 / B - G) extra = 496 / B - G;
  // No more than 64 beyond the first for a set, which all meet in the same words and each read all of its tokens' ranges: with
  // two sets and up to 256, 128 of them, and by the chain [2, 6434, 487] 122 / 72 / 88, [2, 2170, 1624] 79 / 52 / 61, [3,
  // 2342, 1165] on a grid 96 / 83 / 85, [1, 3828, 2193] 92 / 97 / 90.
  if (extra > 64 * G) extra = 64 * G;
  if (extra <= 0) return -1;
  // An image that the chain samples and that has fewer than three workgroups to a set on average: no more than 24 Ki for
  // each, if it has 128 tokens or more.  The chain's sweeps run at the chip's bandwidth then, while one set may hold nearly
  // all rows: [15, 5890, 87] with 24 sets 72.6 / 60.7, [23, 296, 1169] with 16 73.0 / 60.7, with ties [15, 2780, 292] 88.5 / 68.3.
  if (extra < 2 * G && e > 24576 * (extra + 1) && T >= 128 && sampled_f32(T, C, G)) return -1;
  return (int)extra;
}

static int whole_extra(tdq_dtype dt, int B, int T, int C, int G, bool two_ranks) {
  if (T > kWholeTokens) return -1;                     // (the list of its tokens is in LDS)
  return dt == TDQ_F16 ? whole_extra_f16(B, T, C, G, two_ranks) : whole_extra_f32(B, T, C, G, two_ranks);
}

// (not part of the ABI: the tests ask whether the chain of kernels samples their images or takes the radix levels; images
// for which tdq_whole_extra is not -1 take neither)
extern "C" int tdq_samples_rank(int32_t dt, int32_t B, int32_t T, int32_t C, int32_t G) {
  return samples_rank(static_cast<tdq_dtype>(dt), B, T, C, G, false) ? 1 : 0;
}

static int calibration_extra(tdq_dtype dt, int B, int T, int C, const tdq_params* p) {
  const bool exact_only = (p->flags & TDQ_FLAG_EXACT_SELECT) != 0;
  // (the limits of sampled_f32 are those of its chain of kernels)
  if (exact_only || bracket_bins(p->n_groups) == 0 || many_small_sets(B, T, C, p->n_groups)) return -1;
  return whole_extra(dt, B, T, C, p->n_groups, p->base_pct > 0.0 && p->base_pct < 1.0);
}

// What the statistics kernel clears for the rank select.
static SelectClear select_clear(tdq_dtype dt, int B, int T, int C, const tdq_params* p, void* workspace,
                                const WorkspaceLayout& wl) {
  SelectClear c;
  memset(&c, 0, sizeof(c));
  const int extra = calibration_extra(dt, B, T, C, p);
  if (extra < 0) return c;
  char* ws = static_cast<char*>(workspace);
  c.status = reinterpret_cast<unsigned*>(ws + wl.status);
  if (extra == 0) return c;
  c.ctl = reinterpret_cast<unsigned*>(ws + wl.part);
  c.n_ctl = (unsigned)(B * p->n_groups * kSetCtl);
  c.hist = reinterpret_cast<unsigned*>(ws + wl.bhist);
  c.n_hist = (unsigned)(B * p->n_groups * bracket_bins(p->n_groups));
  return c;
}

// (not part of the ABI: the tests ask which images take the one kernel)
extern "C" int tdq_whole_extra(int32_t dt, int32_t B, int32_t T, int32_t C, int32_t G, double base_pct) {
  tdq_params p;
  tdq_default_params(&p);
  p.n_groups = G;
  p.base_pct = base_pct;
  return calibration_extra(static_cast<tdq_dtype>(dt), B, T, C, &p);
}

// Everything of tdq_calibrate_groups after the per-token statistics (which are in the
// workspace): assignment, rank select(s), projection.  X is token-major.
static int calibrate_after_stats(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C,
                                 int64_t ld_x, const tdq_params* p, int32_t* group_id, float* clip,
                                 float* scale, tdq_group_stats* stats, void* workspace,
                                 const LevelPlan& lp, const WorkspaceLayout& wl, const Waits& waits,
                                 hipStream_t st) {
  const int G = p->n_groups;
  char* ws = static_cast<char*>(workspace);
  unsigned* status = reinterpret_cast<unsigned*>(ws + wl.status);
  unsigned* img_flag = reinterpret_cast<unsigned*>(ws + wl.img_flag);
  float* r = reinterpret_cast<float*>(ws + wl.r);
  double* mean = reinterpret_cast<double*>(ws + wl.mean);
  double* m2 = reinterpret_cast<double*>(ws + wl.m2);
  GroupWork* grp = reinterpret_cast<GroupWork*>(ws + wl.grp);
  unsigned* hist = reinterpret_cast<unsigned*>(ws + wl.hist);
  const Scalars sc = make_scalars(p);

  // One rank select per rank wanted of every set: first the base radius Q_p(|x|) when a
  // percentile is asked for (Eq. DSTG_clip), then Q_zr(|x|) with the projection.
  // One sweep (binary16 input) or two (binary32) around a sampled interval resolve the rank of
  // (nearly) every set exactly, and the kernel that verifies it resolves the others.  Too many
  // sets for the interval histogram, or binary32 images too large for the lists of collected
  // keys: radix levels.
  const int Wmax = bracket_bins(G);
  const bool exact_only = (p->flags & TDQ_FLAG_EXACT_SELECT) != 0;
  // words per set of the radix levels' histograms, which the sampled route of binary32 input
  // uses for the head, the cells and the collected keys of a set
  int cap = 0;
  for (int l = 0; l < lp.n_levels; ++l) cap += 1 << lp.bits[l];
  cap = cap > kListMax ? kListMax : cap;
  const bool f16 = dt == TDQ_F16;
  const bool sampled = samples_rank(dt, B, T, C, G, exact_only);
  Bracket* br = reinterpret_cast<Bracket*>(ws + wl.br);
  unsigned* bhist = reinterpret_cast<unsigned*>(ws + wl.bhist);
  const bool two_passes = sc.base_pct > 0.0;
  void* part = ws + wl.part;
  const int extra = calibration_extra(dt, B, T, C, p);
  if (extra >= 0) {
    if (launch_sets_whole(X, dt, B, T, C, ld_x, G, two_passes ? 2 : 1, extra, bracket_bins_zr(G), Wmax, r, mean, m2,
                          group_id, sc, bhist, part, img_flag, status, clip, scale, stats, waits,
                          st) != hipSuccess)
      return TDQ_ERR_HIP;
    return TDQ_OK;
  }
  if (!sampled || exact_only) {          // (the sampled route's own first kernel assigns the sets)
    if (launch_assign(r, mean, m2, B, T, C, G, group_id, part, img_flag, status, st) != hipSuccess)
      return TDQ_ERR_HIP;
  }
  for (int pass = two_passes ? kPassBase : kPassZr; pass >= kPassZr; --pass) {
    const bool keep_base = two_passes && pass == kPassZr;
    // binary32: a bin is as wide as the interval needs, 512 of them (256) are enough
    // binary16: few bins where the interval fits them, else all that there is room for
    const int W = f16 ? Wmax : G <= 32 ? 512 : 256;
    const int Wfew = f16 && pass == kPassZr ? bracket_bins_zr(G) : W;
    const int cells = f16 ? 0 : G <= 32 ? 64 : 32;
    if (sampled) {
      if (!exact_only) {
        if (launch_sets(X, dt, B, T, C, ld_x, G, Wfew, W, cells, r, mean, m2, group_id, sc, pass, keep_base, grp,
                        br, bhist, hist, cap, img_flag, status, st) != hipSuccess)
          return TDQ_ERR_HIP;
        if (launch_bracket_hist(X, dt, B, T, C, ld_x, G, Wfew, W, cells, hist, cap, group_id, br, bhist, st) != hipSuccess)
          return TDQ_ERR_HIP;
        if (!f16 && launch_bracket_gather(X, B, T, C, ld_x, G, W, cells, group_id, br, bhist, grp, hist, cap,
                                          st) != hipSuccess)
          return TDQ_ERR_HIP;
      } else if (launch_finalize_groups(part, B, T, C, G, sc, pass, keep_base, grp, hist, lp, st) !=
                 hipSuccess) {
        return TDQ_ERR_HIP;
      }
      if (launch_bracket_finish(X, dt, B, T, C, ld_x, G, Wfew, W, cells, group_id, bhist, hist, cap, exact_only, sc,
                                pass, grp, br, clip, scale, stats, img_flag, status, st) != hipSuccess)
        return TDQ_ERR_HIP;
      continue;
    }
    if (launch_finalize_groups(part, B, T, C, G, sc, pass, keep_base, grp, hist, lp, st) !=
        hipSuccess)
      return TDQ_ERR_HIP;
    for (int l = 0; l < lp.n_levels; ++l) {
      unsigned* hl = reinterpret_cast<unsigned*>(ws + wl.hist_level[l]);
      if (launch_hist(X, dt, B, T, C, ld_x, G, group_id, grp, hl, lp.shift[l], lp.bits[l], st) !=
          hipSuccess)
        return TDQ_ERR_HIP;
      if (launch_select(hl, B, G, lp.shift[l], lp.bits[l], l == lp.n_levels - 1, dt, sc, grp, clip,
                        scale, stats, img_flag, status, pass, st) != hipSuccess)
        return TDQ_ERR_HIP;
    }
  }
  return TDQ_OK;
}

static int calibrate_groups(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C,
                            int64_t ld_x, const tdq_params* p, int32_t* group_id, float* clip,
                            float* scale, tdq_group_stats* stats, void* workspace,
                            size_t workspace_bytes, const Waits& waits, void* stream) {
  if (!X || !p || !group_id || !clip || !scale || !workspace) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  int rc = check_params(p);
  if (rc != TDQ_OK) return rc;
  rc = check_shape(B, T, C, ld_x);
  if (rc != TDQ_OK) return rc;
  const int G = p->n_groups;
  const LevelPlan lp = make_level_plan(dt, G);
  const WorkspaceLayout wl = make_layout(B, T, G, lp);
  if (workspace_bytes < wl.total) return TDQ_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) & 255) return TDQ_ERR_WORKSPACE;
  const size_t esz = dt == TDQ_F16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(X) % esz) return TDQ_ERR_ALIGN;

  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  if (launch_token_stats(X, dt, B * T, C, ld_x, reinterpret_cast<float*>(ws + wl.r),
                         reinterpret_cast<double*>(ws + wl.mean),
                         reinterpret_cast<double*>(ws + wl.m2), select_clear(dt, B, T, C, p, ws, wl), st) != hipSuccess)
    return TDQ_ERR_HIP;
  return calibrate_after_stats(X, dt, B, T, C, ld_x, p, group_id, clip, scale, stats, workspace, lp,
                               wl, waits, st);
}

// ---------------------------------------------------------------------------
// Library-owned calibration scratch for tdq_calibrate_groups_static.  In host code the
// array's name is only a handle for hipGetSymbolAddress; the device address is looked up
// once per device (each GPU has its own copy at its own address) and that pointer is what
// the kernels get.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[TDQ_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on the current device, or nullptr (with *rc set).
static void* scratch_of_current_device(int* rc) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    *rc = TDQ_ERR_HIP;
    return nullptr;
  }
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    // two threads racing here look up the same address; either store is the right one
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      *rc = TDQ_ERR_HIP;
      return nullptr;
    }
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);
  }
  *rc = TDQ_OK;
  return ptr;
}

// The status area of the scratch, handed to the caller's buffer (a kernel, not a copy
// call: a caller may be capturing a graph).
__global__ void k_export_status(const unsigned* __restrict__ status, unsigned* __restrict__ out) {
  const int i = threadIdx.x;
  if (i < 4) out[i] = i < 3 ? status[i] : 0u;
}

}  // namespace tdq

using namespace tdq;

extern "C" {

int tdq_version(void) { return TDQ_VERSION; }

const char* tdq_status_string(int status) {
  switch (status) {
    case TDQ_OK: return "ok";
    case TDQ_ERR_NULL: return "null pointer";
    case TDQ_ERR_SHAPE: return "invalid shape or leading dimension";
    case TDQ_ERR_PARAM: return "parameter out of range";
    case TDQ_ERR_WORKSPACE: return "workspace too small or misaligned";
    case TDQ_ERR_DTYPE: return "unknown dtype";
    case TDQ_ERR_HIP: return "HIP call failed";
    case TDQ_ERR_UNSUPPORTED: return "not implemented in this build";
    case TDQ_ERR_ALIGN: return "pointer or leading dimension misaligned";
    default: return "unknown status";
  }
}

void tdq_default_params(tdq_params* p) {
  if (!p) return;
  p->n_groups = 8;
  p->chan_group = 0;
  p->act_bits = 4;
  p->flags = TDQ_FLAG_C1 | TDQ_FLAG_C2;
  p->tau = 1.0;
  p->zr = 0.2;
  p->base_pct = 0.0;
  p->eps_scale = 1e-8f;
  p->eps_std = 1e-12f;
}

size_t tdq_workspace_bytes(int32_t B, int32_t T, int32_t C, tdq_dtype dt, const tdq_params* p) {
  if (check_params(p) != TDQ_OK) return 0;
  if (check_shape(B, T, C, C) != TDQ_OK) return 0;
  if (dt != TDQ_F16 && dt != TDQ_F32) return 0;
  const LevelPlan lp = make_level_plan(dt, p->n_groups);
  return make_layout(B, T, p->n_groups, lp).total;
}

int tdq_calibrate_groups(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C,
                         int64_t ld_x, const tdq_params* p, int32_t* group_id, float* clip,
                         float* scale, tdq_group_stats* stats, void* workspace,
                         size_t workspace_bytes, void* stream) {
  return calibrate_groups(X, dt, B, T, C, ld_x, p, group_id, clip, scale, stats, workspace, workspace_bytes, kWaits,
                          stream);
}

// (not part of the ABI: the tests hurry the workgroups that wait for each other, and look at their words of the
// workspace afterwards, kSetCtl for each set from byte *set_words on)
int tdq_calibrate_groups_waits(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C, int64_t ld_x,
                               const tdq_params* p, int32_t* group_id, float* clip, float* scale,
                               tdq_group_stats* stats, void* workspace, size_t workspace_bytes, uint32_t patience,
                               uint32_t limit, size_t* set_words, void* stream) {
  const int rc = calibrate_groups(X, dt, B, T, C, ld_x, p, group_id, clip, scale, stats, workspace, workspace_bytes,
                                  Waits{patience, limit}, stream);
  if (rc == TDQ_OK) *set_words = make_layout(B, T, p->n_groups, make_level_plan(dt, p->n_groups)).part;
  return rc;
}

int tdq_calibrate_groups_static(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C,
                                int64_t ld_x, const tdq_params* p, int32_t* group_id, float* clip,
                                float* scale, tdq_group_stats* stats, uint32_t* status,
                                void* stream) {
  if (!X || !p || !group_id || !clip || !scale) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  int rc = check_params(p);
  if (rc != TDQ_OK) return rc;
  rc = check_shape(B, T, C, ld_x);
  if (rc != TDQ_OK) return rc;
  if (reinterpret_cast<uintptr_t>(status) & 3) return TDQ_ERR_ALIGN;
  const LevelPlan lp = make_level_plan(dt, p->n_groups);
  const WorkspaceLayout wl = make_layout(B, T, p->n_groups, lp);
  if (wl.total > (size_t)TDQ_STATIC_SCRATCH_BYTES) return TDQ_ERR_WORKSPACE;
  void* ws = scratch_of_current_device(&rc);
  if (!ws) return rc;
  // the kernels of tdq_calibrate_groups clear every part of the workspace they add into
  // (set records, histograms, counters), so what the last call left behind does not matter
  rc = tdq_calibrate_groups(X, dt, B, T, C, ld_x, p, group_id, clip, scale, stats, ws,
                            TDQ_STATIC_SCRATCH_BYTES, stream);
  if (rc != TDQ_OK) return rc;
  if (status) {
    hipLaunchKernelGGL(k_export_status, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream),
                       reinterpret_cast<const unsigned*>(static_cast<char*>(ws) + wl.status), status);
    if (hipGetLastError() != hipSuccess) return TDQ_ERR_HIP;
  }
  return TDQ_OK;
}

int tdq_calibrate_groups_chw(const void* X, tdq_dtype dt, int32_t B, int32_t C, int32_t T,
                             int64_t ld_c, int64_t ld_b, const tdq_params* p, void* Xt,
                             int64_t ld_xt, int32_t* group_id, float* clip, float* scale,
                             tdq_group_stats* stats, void* workspace, size_t workspace_bytes,
                             void* stream) {
  if (!X || !Xt || !p || !group_id || !clip || !scale || !workspace) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  int rc = check_params(p);
  if (rc != TDQ_OK) return rc;
  rc = check_shape(B, T, C, ld_xt);
  if (rc != TDQ_OK) return rc;
  if (B > TDQ_MAX_IMAGES) return TDQ_ERR_SHAPE;
  if (ld_c < T || ld_b < (int64_t)(C - 1) * ld_c + T) return TDQ_ERR_SHAPE;
  const int G = p->n_groups;
  const LevelPlan lp = make_level_plan(dt, G);
  const WorkspaceLayout wl = make_layout(B, T, G, lp);
  if (workspace_bytes < wl.total) return TDQ_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) & 255) return TDQ_ERR_WORKSPACE;
  const size_t esz = dt == TDQ_F16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(X) % esz || reinterpret_cast<uintptr_t>(Xt) % esz)
    return TDQ_ERR_ALIGN;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  if (launch_tokenize_stats_chw(X, dt, B, C, T, ld_c, ld_b, Xt, ld_xt,
                                reinterpret_cast<float*>(ws + wl.r),
                                reinterpret_cast<double*>(ws + wl.mean),
                                reinterpret_cast<double*>(ws + wl.m2), select_clear(dt, B, T, C, p, ws, wl),
                                st) != hipSuccess)
    return TDQ_ERR_HIP;
  return calibrate_after_stats(Xt, dt, B, T, C, ld_xt, p, group_id, clip, scale, stats, workspace,
                               lp, wl, kWaits, st);
}

int tdq_quantize_act(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C, int64_t ld_x,
                     const tdq_params* p, const int32_t* group_id, const float* clip,
                     const float* scale, uint8_t* Qx, int64_t ld_q, void* stream) {
  if (!X || !p || !clip || !scale || !Qx) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  int rc = check_params(p);
  if (rc != TDQ_OK) return rc;
  rc = check_shape(B, T, C, ld_x);
  if (rc != TDQ_OK) return rc;
  if (!group_id && p->n_groups != 1) return TDQ_ERR_NULL;
  if (ld_q < (C + 1) / 2) return TDQ_ERR_SHAPE;
  const size_t esz = dt == TDQ_F16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(X) % esz) return TDQ_ERR_ALIGN;
  if (launch_quantize(X, dt, B, T, C, ld_x, p->n_groups, group_id, clip, scale, Qx, ld_q,
                      static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_calibrate_quantize_fused(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C,
                                 int64_t ld_x, const tdq_params* p, int32_t* group_id, float* clip,
                                 float* scale, tdq_group_stats* stats, uint32_t* image_flags,
                                 uint8_t* Qx, int64_t ld_q, void* workspace, size_t workspace_bytes,
                                 void* stream) {
  if (!X || !p || !group_id || !clip || !scale || !Qx || !workspace) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  int rc = check_params(p);
  if (rc != TDQ_OK) return rc;
  rc = check_shape(B, T, C, ld_x);
  if (rc != TDQ_OK) return rc;
  const int G = p->n_groups;
  if (G > TDQ_FUSED_MAX_GROUPS) return TDQ_ERR_UNSUPPORTED;
  if (ld_q < (C + 1) / 2) return TDQ_ERR_SHAPE;
  const WorkspaceLayout wl = make_layout(B, T, G, make_level_plan(dt, G));
  if (workspace_bytes < wl.total) return TDQ_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) & 255) return TDQ_ERR_WORKSPACE;
  const size_t esz = dt == TDQ_F16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(X) % esz) return TDQ_ERR_ALIGN;
  if (reinterpret_cast<uintptr_t>(image_flags) & 3) return TDQ_ERR_ALIGN;
  char* ws = static_cast<char*>(workspace);
  if (launch_fused_small(X, dt, B, T, C, ld_x, G, make_scalars(p),
                         reinterpret_cast<float*>(ws + wl.r), reinterpret_cast<double*>(ws + wl.mean),
                         reinterpret_cast<double*>(ws + wl.m2), group_id, clip, scale, stats,
                         image_flags, Qx, ld_q, static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_range_disparity(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C, int64_t ld_x,
                        float* token_median, float* token_max, float* disparity, float* max_abs,
                        void* stream) {
  if (!X || !token_median || !token_max || !disparity || !max_abs) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  const int rc = check_shape(B, T, C, ld_x);
  if (rc != TDQ_OK) return rc;
  const size_t esz = dt == TDQ_F16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(X) % esz) return TDQ_ERR_ALIGN;
  if ((reinterpret_cast<uintptr_t>(token_median) | reinterpret_cast<uintptr_t>(token_max) |
       reinterpret_cast<uintptr_t>(disparity) | reinterpret_cast<uintptr_t>(max_abs)) & 3)
    return TDQ_ERR_ALIGN;
  if (launch_range_disparity(X, dt, B, T, C, ld_x, token_median, token_max, disparity, max_abs,
                             static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_tokenize_chw(const void* X, tdq_dtype dt, int32_t B, int32_t C, int32_t T, int64_t ld_c,
                     int64_t ld_b, void* Xt, int64_t ld_xt, void* stream) {
  if (!X || !Xt) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  if (B < 1 || T < 1 || C < 1 || B > TDQ_MAX_IMAGES) return TDQ_ERR_SHAPE;
  if ((int64_t)B * T > (int64_t)1 << 30) return TDQ_ERR_SHAPE;
  if (ld_c < T || ld_b < (int64_t)(C - 1) * ld_c + T || ld_xt < C) return TDQ_ERR_SHAPE;
  const size_t esz = dt == TDQ_F16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(X) % esz || reinterpret_cast<uintptr_t>(Xt) % esz)
    return TDQ_ERR_ALIGN;
  if (launch_tokenize_chw(X, dt, B, C, T, ld_c, ld_b, Xt, ld_xt,
                          static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_quantize_act_blocks(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C,
                            int64_t ld_x, const tdq_params* p, uint8_t* Qx, int64_t ld_q,
                            float* block_scale, float* block_clip, int64_t ld_s, void* stream) {
  if (!X || !p || !Qx || !block_scale) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  int rc = check_params(p, true);
  if (rc != TDQ_OK) return rc;
  rc = check_shape(B, T, C, ld_x);
  if (rc != TDQ_OK) return rc;
  const int64_t KB = ((int64_t)C + TDQ_BLOCK - 1) / TDQ_BLOCK;
  if (ld_q < (C + 1) / 2 || ld_s < KB) return TDQ_ERR_SHAPE;
  if ((int64_t)B * T * KB >= (int64_t)1 << 31) return TDQ_ERR_SHAPE;
  const size_t esz = dt == TDQ_F16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(X) % esz) return TDQ_ERR_ALIGN;
  if ((reinterpret_cast<uintptr_t>(block_scale) | reinterpret_cast<uintptr_t>(block_clip)) & 3)
    return TDQ_ERR_ALIGN;
  const int kq = block_rank(p->zr);
  const int kp = (p->base_pct > 0.0 && p->base_pct < 1.0) ? block_rank(p->base_pct) : TDQ_BLOCK;
  if (launch_quantize_blocks(X, dt, (long long)B * T, C, ld_x, kq, kp, make_scalars(p), Qx, ld_q,
                             block_scale, block_clip, ld_s,
                             static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_quantize_act_blocks_f6(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C,
                               int64_t ld_x, const tdq_params* p, uint8_t* Qx6, float* block_scale,
                               float* block_clip, int64_t ld_s, void* stream) {
  if (!X || !p || !Qx6 || !block_scale) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  int rc = check_params(p, true);
  if (rc != TDQ_OK) return rc;
  rc = check_shape(B, T, C, ld_x);
  if (rc != TDQ_OK) return rc;
  const int64_t KB = ((int64_t)C + TDQ_BLOCK - 1) / TDQ_BLOCK;
  if (ld_s < KB) return TDQ_ERR_SHAPE;
  if ((int64_t)B * T * KB >= (int64_t)1 << 31) return TDQ_ERR_SHAPE;
  const size_t esz = dt == TDQ_F16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(X) % esz) return TDQ_ERR_ALIGN;
  if (reinterpret_cast<uintptr_t>(Qx6) & 15) return TDQ_ERR_ALIGN;
  if ((reinterpret_cast<uintptr_t>(block_scale) | reinterpret_cast<uintptr_t>(block_clip)) & 3)
    return TDQ_ERR_ALIGN;
  const int kq = block_rank(p->zr);
  const int kp = (p->base_pct > 0.0 && p->base_pct < 1.0) ? block_rank(p->base_pct) : TDQ_BLOCK;
  if (launch_quantize_blocks_f6(X, dt, (long long)B * T, C, ld_x, kq, kp, make_scalars(p), Qx6,
                                block_scale, block_clip, ld_s,
                                static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_quantize_act_blocks_chw(const void* X, tdq_dtype dt, int32_t B, int32_t C, int32_t T,
                                int64_t ld_c, int64_t ld_b, const tdq_params* p, uint8_t* Qx,
                                int64_t ld_q, float* block_scale, float* block_clip, int64_t ld_s,
                                void* stream) {
  if (!X || !p || !Qx || !block_scale) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  int rc = check_params(p, true);
  if (rc != TDQ_OK) return rc;
  if (B < 1 || T < 1 || C < 1 || B > TDQ_MAX_IMAGES) return TDQ_ERR_SHAPE;
  if ((int64_t)B * T > (int64_t)1 << 30) return TDQ_ERR_SHAPE;
  if (ld_c < T || ld_b < (int64_t)(C - 1) * ld_c + T) return TDQ_ERR_SHAPE;
  const int64_t KB = ((int64_t)C + TDQ_BLOCK - 1) / TDQ_BLOCK;
  if (ld_q < (C + 1) / 2 || ld_s < KB) return TDQ_ERR_SHAPE;
  const size_t esz = dt == TDQ_F16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(X) % esz) return TDQ_ERR_ALIGN;
  if ((reinterpret_cast<uintptr_t>(block_scale) | reinterpret_cast<uintptr_t>(block_clip)) & 3)
    return TDQ_ERR_ALIGN;
  const int kq = block_rank(p->zr);
  const int kp = (p->base_pct > 0.0 && p->base_pct < 1.0) ? block_rank(p->base_pct) : TDQ_BLOCK;
  if (launch_quantize_blocks_chw(X, dt, B, C, T, ld_c, ld_b, kq, kp, make_scalars(p), Qx, ld_q,
                                 block_scale, block_clip, ld_s,
                                 static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_group_diagnostics(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C, int64_t ld_x,
                          const tdq_params* p, const int32_t* group_id, const float* clip,
                          const float* scale, uint64_t* zero_count, uint64_t* clipped_count,
                          void* stream) {
  if (!X || !p || !clip || !scale || !zero_count || !clipped_count) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  int rc = check_params(p);
  if (rc != TDQ_OK) return rc;
  rc = check_shape(B, T, C, ld_x);
  if (rc != TDQ_OK) return rc;
  if (!group_id && p->n_groups != 1) return TDQ_ERR_NULL;
  const size_t esz = dt == TDQ_F16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(X) % esz) return TDQ_ERR_ALIGN;
  if ((reinterpret_cast<uintptr_t>(zero_count) | reinterpret_cast<uintptr_t>(clipped_count)) & 7)
    return TDQ_ERR_ALIGN;
  if (launch_group_diag(X, dt, B, T, C, ld_x, p->n_groups, group_id, clip, scale,
                        reinterpret_cast<unsigned long long*>(zero_count),
                        reinterpret_cast<unsigned long long*>(clipped_count),
                        static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_w4a4_linear(const uint8_t* Qx, int64_t ld_q, const int32_t* group_id, const float* scale,
                    int32_t B, int32_t T, int32_t K, int32_t N, int32_t G, const uint8_t* Qw,
                    int64_t ld_w, const float* w_scale, const float* bias, void* Y,
                    tdq_dtype y_dt, int64_t ld_y, int32_t* acc_dump, void* stream) {
  if (!Qx || !scale || !Qw || !w_scale || !Y) return TDQ_ERR_NULL;
  if (y_dt != TDQ_F16 && y_dt != TDQ_F32) return TDQ_ERR_DTYPE;
  if (B < 1 || T < 1 || K < 1 || N < 1) return TDQ_ERR_SHAPE;
  if ((int64_t)B * T > (int64_t)1 << 30) return TDQ_ERR_SHAPE;
  if (K > TDQ_MAX_K) return TDQ_ERR_SHAPE;  // 256 * 64 * K must stay below 2^31
  if (G < 1 || G > TDQ_MAX_GROUPS) return TDQ_ERR_PARAM;
  if (!group_id && G != 1) return TDQ_ERR_NULL;
  const int64_t row_bytes = 16 * (((int64_t)K + 31) / 32);
  if (ld_q < row_bytes || ld_w < row_bytes || ld_y < N) return TDQ_ERR_SHAPE;
  if (ld_q % 16 || ld_w % 16) return TDQ_ERR_ALIGN;
  if ((reinterpret_cast<uintptr_t>(Qx) & 15) || (reinterpret_cast<uintptr_t>(Qw) & 15))
    return TDQ_ERR_ALIGN;
  if (reinterpret_cast<uintptr_t>(Y) % (y_dt == TDQ_F16 ? 2 : 4)) return TDQ_ERR_ALIGN;
  if (launch_w4a4_gemm(Qx, ld_q, group_id, scale, B * T, T, K, N, G, Qw, ld_w, w_scale, bias, Y,
                       y_dt, ld_y, acc_dump, static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_w4a4_linear_blocks(const uint8_t* Qx, int64_t ld_q, const float* block_scale, int64_t ld_s,
                           int64_t M, int32_t K, int32_t N, const uint8_t* Qw, int64_t ld_w,
                           const float* w_scale, const float* bias, void* Y, tdq_dtype y_dt,
                           int64_t ld_y, void* stream) {
  if (!Qx || !block_scale || !Qw || !w_scale || !Y) return TDQ_ERR_NULL;
  if (y_dt != TDQ_F16 && y_dt != TDQ_F32) return TDQ_ERR_DTYPE;
  if (M < 1 || K < 1 || N < 1) return TDQ_ERR_SHAPE;
  if (M > (int64_t)1 << 30 || K > 131072) return TDQ_ERR_SHAPE;
  const int64_t KB = ((int64_t)K + TDQ_BLOCK - 1) / TDQ_BLOCK;
  const int64_t row_bytes = 16 * KB;
  if (ld_q < row_bytes || ld_w < row_bytes || ld_y < N || ld_s < KB) return TDQ_ERR_SHAPE;
  if (ld_q % 16 || ld_w % 16) return TDQ_ERR_ALIGN;
  if ((reinterpret_cast<uintptr_t>(Qx) & 15) || (reinterpret_cast<uintptr_t>(Qw) & 15))
    return TDQ_ERR_ALIGN;
  if (reinterpret_cast<uintptr_t>(block_scale) & 3) return TDQ_ERR_ALIGN;
  if (reinterpret_cast<uintptr_t>(Y) % (y_dt == TDQ_F16 ? 2 : 4)) return TDQ_ERR_ALIGN;
  if (launch_w4a4_gemm_blocks(Qx, ld_q, block_scale, ld_s, (int)M, K, N, Qw, ld_w, w_scale, bias, Y,
                              y_dt, ld_y, static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_quantize_act_f6(const void* X, tdq_dtype dt, int32_t B, int32_t T, int32_t C, int64_t ld_x,
                        const tdq_params* p, const int32_t* group_id, const float* clip,
                        const float* scale, uint8_t* Qx6, void* stream) {
  if (!X || !p || !clip || !scale || !Qx6) return TDQ_ERR_NULL;
  if (dt != TDQ_F16 && dt != TDQ_F32) return TDQ_ERR_DTYPE;
  int rc = check_params(p);
  if (rc != TDQ_OK) return rc;
  rc = check_shape(B, T, C, ld_x);
  if (rc != TDQ_OK) return rc;
  if (C > 131072) return TDQ_ERR_SHAPE;
  if (!group_id && p->n_groups != 1) return TDQ_ERR_NULL;
  const size_t esz = dt == TDQ_F16 ? 2 : 4;
  if (reinterpret_cast<uintptr_t>(X) % esz) return TDQ_ERR_ALIGN;
  if (reinterpret_cast<uintptr_t>(Qx6) & 15) return TDQ_ERR_ALIGN;
  if (launch_quantize_f6(X, dt, B, T, C, ld_x, p->n_groups, group_id, clip, scale, Qx6,
                         static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

size_t tdq_f6_bytes(int64_t rows, int32_t K) {
  if (rows < 1 || K < 1) return 0;
  const int64_t KB = 2 * (((int64_t)K + 127) / 128);
  return (size_t)(((rows + 31) / 32) * KB * 1536);
}

int tdq_pack_codes_f6(const uint8_t* Q, int64_t ld, int64_t rows, int32_t K, uint8_t* F, void* stream) {
  if (!Q || !F) return TDQ_ERR_NULL;
  if (rows < 1 || rows > (int64_t)1 << 30 || K < 1 || K > 131072 || ld < (K + 1) / 2) return TDQ_ERR_SHAPE;
  if (reinterpret_cast<uintptr_t>(F) & 15) return TDQ_ERR_ALIGN;
  if (launch_pack_f6(Q, ld, (int)rows, K, F, static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_w4a4_linear_f6(const uint8_t* Qx6, const int32_t* group_id, const float* scale, int32_t B,
                       int32_t T, int32_t K, int32_t N, int32_t G, const uint8_t* Qw6,
                       const float* w_scale, const float* bias, void* Y, tdq_dtype y_dt, int64_t ld_y,
                       int32_t* acc_dump, void* stream) {
  if (!Qx6 || !scale || !Qw6 || !w_scale || !Y) return TDQ_ERR_NULL;
  if (y_dt != TDQ_F16 && y_dt != TDQ_F32) return TDQ_ERR_DTYPE;
  if (B < 1 || T < 1 || K < 1 || N < 1) return TDQ_ERR_SHAPE;
  if ((int64_t)B * T > (int64_t)1 << 30 || K > 131072 || ld_y < N) return TDQ_ERR_SHAPE;
  if (G < 1 || G > TDQ_MAX_GROUPS) return TDQ_ERR_PARAM;
  if (!group_id && G != 1) return TDQ_ERR_NULL;
  if ((reinterpret_cast<uintptr_t>(Qx6) & 15) || (reinterpret_cast<uintptr_t>(Qw6) & 15))
    return TDQ_ERR_ALIGN;
  if (reinterpret_cast<uintptr_t>(Y) % (y_dt == TDQ_F16 ? 2 : 4)) return TDQ_ERR_ALIGN;
  if (launch_w4a4_gemm_f6(Qx6, Qw6, K, group_id, scale, B * T, T, N, G, w_scale, bias, Y, y_dt, ld_y,
                          acc_dump, static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_w4a4_linear_blocks_f6(const uint8_t* Qx6, const float* block_scale, int64_t ld_s, int64_t M,
                              int32_t K, int32_t N, const uint8_t* Qw6, const float* w_scale,
                              const float* bias, void* Y, tdq_dtype y_dt, int64_t ld_y, void* stream) {
  if (!Qx6 || !block_scale || !Qw6 || !w_scale || !Y) return TDQ_ERR_NULL;
  if (y_dt != TDQ_F16 && y_dt != TDQ_F32) return TDQ_ERR_DTYPE;
  if (M < 1 || K < 1 || N < 1 || M > (int64_t)1 << 30 || K > 131072) return TDQ_ERR_SHAPE;
  const int64_t KB = ((int64_t)K + TDQ_BLOCK - 1) / TDQ_BLOCK;
  if (ld_y < N || ld_s < KB) return TDQ_ERR_SHAPE;
  if (ld_s > ((int64_t)1 << 22)) return TDQ_ERR_SHAPE;     // 128 rows of scales within 32-bit offsets
  if ((reinterpret_cast<uintptr_t>(Qx6) & 15) || (reinterpret_cast<uintptr_t>(Qw6) & 15))
    return TDQ_ERR_ALIGN;
  if (reinterpret_cast<uintptr_t>(block_scale) & 3) return TDQ_ERR_ALIGN;
  if (reinterpret_cast<uintptr_t>(Y) % (y_dt == TDQ_F16 ? 2 : 4)) return TDQ_ERR_ALIGN;
  if (launch_w4a4_gemm_blocks_f6(Qx6, Qw6, block_scale, ld_s, (int)M, K, N, w_scale, bias, Y, y_dt,
                                 ld_y, static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

int tdq_quantize_weight(const float* W, int32_t N, int32_t K, int64_t ld_w_in, uint8_t* Qw,
                        int64_t ld_w, float* w_scale, void* stream) {
  if (!W || !Qw || !w_scale) return TDQ_ERR_NULL;
  if (N < 1 || K < 1 || ld_w_in < K || ld_w < (K + 1) / 2) return TDQ_ERR_SHAPE;
  if (reinterpret_cast<uintptr_t>(W) & 3) return TDQ_ERR_ALIGN;
  if (launch_quantize_weight(W, N, K, ld_w_in, Qw, ld_w, w_scale,
                             static_cast<hipStream_t>(stream)) != hipSuccess)
    return TDQ_ERR_HIP;
  return TDQ_OK;
}

}  // extern "C"
