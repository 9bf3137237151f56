// Rank select of the zr quantile guided by a sample: one sweep of X for binary16 activations,
// two for binary32 (constraint C2 of DCRP, Eq. zr_constraint: the k-th smallest |x| of every
// (image, token set), k = ceil(zr n), Supp. "Quantile Implementation").
//
// The magnitude key of a binary16 value has 15 bits, that of a binary32 value 31.  A radix
// select over LDS histograms needs two (four) sweeps of X for that many bits.  Here a small
// sample of every set first says where to look:
//
//   k_sets            one workgroup per set finds the set's tokens and moments, reads 8 or
//                     16 Ki sampled elements and takes the key interval between two sample order
//                     statistics on either side of the one that corresponds to k: one-key bins
//                     (binary16), or bins of about equal mass (binary32).  It holds the true
//                     answer unless the sample is off by more than that.
//   k_bracket_hist    one sweep of X: per set, the number of keys below the interval and an
//                     LDS histogram of the keys inside it.
//   k_bracket_gather  binary32: a second sweep collects the keys of every set that fall into
//                     the bin where the running count reaches k.
//   k_bracket_finish  one workgroup per set: if below < k <= below + inside, the answer is the
//                     bin where the running count reaches k - below -- or, of the keys
//                     collected from it, the one of the remaining rank: the exact k-th
//                     smallest, no matter how the interval was chosen -- and the set is
//                     projected.  Otherwise the set is counted as missed and the same
//                     workgroup finds the key in the set's own rows, on the side of the
//                     interval where it must be (exact as well, and rare).
//
// Images of ordinary size take one kernel instead of these (k_sets with WHOLE): the workgroups that find a
// set's tokens and place its interval then read the set's own rows, several sharing a set, and the last of
// them to finish verifies, picks and projects (binary32: they wait for each other's counts and pick the bin's key
// together, shared_rank).  Nothing but the statistics has to be complete before it.
//
// The result is therefore always the exact order statistic; the sample only decides
// which of the two routes computes it, i.e. how long it takes.
//
// Zeros are never inside an interval (it starts at key 1 at the lowest): where it starts there,
// "below" counts exactly the zeros, and a rank among them is answered by that count.  A fifth
// of an activation behind a rectifier is zeros, which would all meet in one word of LDS.
#include <type_traits>

#include "tdq_device.hpp"
#include "tdq_workgroup.hpp"

namespace tdq {

typedef short s2v __attribute__((ext_vector_type(2)));
typedef unsigned long long u64;

constexpr int kRunLen = 32;                                     // channels per run (64 bytes)
constexpr int kSampleBits = 10;                                 // key bits the sample histogram resolves
constexpr int kSweepThreads = 1024;
constexpr int kIdRounds = 16;                                   // most range keys a thread of k_sets holds

// Words of a set's control block: shares (binary16: workgroups) that have arrived, elements below the interval
// (binary16, two ranks: the next word for the second); binary32: keys handed over, what the words have been
// cleared for, claims of a share, whether one workgroup did it alone in the end.
enum { kCtlArrived = 0, kCtlBelow = 1, kCtlListed = 2, kCtlReady = 3, kCtlClaimed = 4, kCtlAlone = 5 };

// Arguments of a k_sets that sees a set through to its radius.
struct WholeArgs {
  int extra;                  // workgroups per image beyond one per set
  int L;                      // lanes per row
  u32* ctl;                   // per set kSetCtl words, cleared before: parts that have arrived, counts below
  float* clip;
  float* scale;
  tdq_group_stats* stats;
  Waits waits;
};

// binary32: what a set's `lists` area of cap words holds.  First a head: the largest ~key and the
// largest key collected; a key that the sample holds often, or kNoKey, how often the set holds it,
// and its bin.  Then, if the interval has cells (kCells in Bracket::shift), these: at most 64, each
// its first bin | number of bins << 16.  Then the collected keys.
constexpr int kListHead = 8;
enum { kHeadMin = 0, kHeadMax, kHeadTie, kHeadTies, kHeadTieBin };
constexpr u32 kNoKey = 0xFFFFFFFFu;
constexpr u32 kCells = 0x100u;

// Bin of a key d past the interval's start: cell d >> shift is cut into equal parts (1 <= shift).
__device__ __forceinline__ u32 bin_of(u32 d, u32 shift, u32 cell) {
  return (cell & 0xFFFFu) + __umulhi(d << (32u - shift), cell >> 16);
}

// The bin of a set's interval histogram (W = 256 to 2048 words) that holds its k-th smallest
// key, by one wavefront; the same in every lane.  ok = the interval does hold it.  (binary32:
// `ties` more elements lie in bin tie_bin than its word says.)  A set has fewer than 2^32 elements.
struct BinPick {
  bool ok;
  u32 bin, need;              // rank wanted among the bin's elements (1-based)
  u32 count;                  // elements of the bin's histogram word
  u32 inside;                 // elements inside the interval
};
template <bool TIES>
__device__ __forceinline__ BinPick pick_bin(const u32* __restrict__ hb, int W, u32 below, u32 k,
                                            u32 tie_bin = kNoKey, u32 ties = 0) {
  const int lane = threadIdx.x & 63;
  const int quads = W / 256;                    // 1 to 8 groups of four bins per lane
  const uint4* mine_bins = reinterpret_cast<const uint4*>(hb) + lane * quads;
  uint4 c[2];                                   // two groups stay in registers
  u32 sum[8];
#pragma unroll
  for (int i = 0; i < 2; ++i) c[i] = mine_bins[i < quads ? i : 0];
#pragma unroll
  for (int i = 0; i < 8; ++i) sum[i] = i < 2 && i < quads ? c[i].x + c[i].y + c[i].z + c[i].w : 0u;
  if (quads > 2) {                              // uniform; the loads issued together
    uint4 t[6];
#pragma unroll
    for (int i = 2; i < 8; ++i) t[i - 2] = mine_bins[i < quads ? i : 0];
#pragma unroll
    for (int i = 2; i < 8; ++i)
      sum[i] = i < quads ? t[i - 2].x + t[i - 2].y + t[i - 2].z + t[i - 2].w : 0u;
  }
  if (TIES && ties != 0) {                      // uniform
    const int at = (int)(tie_bin >> 2) - lane * quads;         // of this lane's groups, if any
#pragma unroll
    for (int i = 0; i < 8; ++i) sum[i] += i == at && i < quads ? ties : 0u;
  }
  u32 mine = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) mine += sum[i];
  const u32 incl = wave_scan_u32(mine);
  BinPick r;
  r.inside = (u32)__builtin_amdgcn_readlane((int)incl, 63);
  r.ok = k > below && k - below <= r.inside;
  const u32 need = k - below;
  const unsigned long long hit = __ballot(incl >= need);
  const int src = r.ok ? __ffsll((long long)hit) - 1 : 0;       // hit != 0 because need <= inside
  u32 cum = incl - mine;
  int group = 0;                                // the group of four ...
  bool found = false;
  if (quads > 1) {
#pragma unroll
    for (int i = 0; i < 7; ++i) {
      found = found || i >= quads - 1 || cum + sum[i] >= need;
      if (!found) {
        cum += sum[i];
        ++group;
      }
    }
  }
  // (member by member: a choice between the two of c would put them into scratch memory)
  uint4 q = make_uint4(group == 0 ? c[0].x : c[1].x, group == 0 ? c[0].y : c[1].y, group == 0 ? c[0].z : c[1].z,
                       group == 0 ? c[0].w : c[1].w);
  if (quads > 2) q = mine_bins[group];
  u32 bin = (u32)(4 * (lane * quads + group));
  const u32 v[4] = {q.x, q.y, q.z, q.w};        // ... and the bin in it
  u32 count = v[0];
  found = false;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const u32 all = v[i] + (TIES && bin == tie_bin ? ties : 0u);
    found = found || cum + all >= need;
    if (!found) {
      cum += all;
      ++bin;
      count = v[i + 1];
    }
  }
  r.bin = (u32)__builtin_amdgcn_readlane((int)bin, src);
  r.need = need - (u32)__builtin_amdgcn_readlane((int)cum, src);
  r.count = (u32)__builtin_amdgcn_readlane((int)count, src);
  return r;
}

// ---------------------------------------------------------------------------
// Search of a set's rows by one workgroup.
// ---------------------------------------------------------------------------
constexpr int kFinishBits = 11;                 // key bits a pass resolves
constexpr int kFinishTokens = 2048;             // tokens looked at together
constexpr int kWindow = 1 << kFinishBits;       // keys of a pass that looks at them one by one

// LDS of the search
template <int NT, bool LISTED>
struct FinishLds {
  __attribute__((aligned(16))) u32 h[1 << kFinishBits];
  unsigned short list[LISTED ? 1 : kFinishTokens];    // the set's tokens among those looked at together
  u32 wtot[NT / 64], digit;
  unsigned long long wsum[NT / 64], rest;
};

// Rows list[0 .. n - 1] (offsets from row Xb), read by a workgroup of NT threads: groups of L lanes take R rows
// and P 16-byte pieces of each at a time, R P = Q and P by the row length, and (AHEAD) load the next Q while
// the caller's piece(uint4) looks at these; single(element) gets what no whole piece holds.  (The search loads
// nothing ahead: with 1024 threads the registers cost it more, [3, 11324, 171] with 31 missed sets 200 us, 190 so.)
template <typename TX, int NT, int Q, bool AHEAD>
struct RowVisitor {
  static constexpr int V = Elem<TX>::V;
  const TX* Xb;
  long long ld;
  int C, L, n, nvec, P, R, lr, slots, row, v0;
  const unsigned short* list;
  uint4 q[Q];
  // starts with the loads of the first pieces
  __device__ __forceinline__ RowVisitor(const TX* Xb_, long long ld_, int C_, int L_, const unsigned short* list_,
                                        int n_)
      : Xb(Xb_), ld(ld_), C(C_), L(L_), n(n_), list(list_) {
    nvec = C / V;
    P = nvec <= L ? 1 : nvec <= 2 * L ? 2 : 4;
    R = Q / P;
    lr = threadIdx.x & (L - 1);
    const int shift = 31 - __clz(L);
    row = threadIdx.x >> shift;
    slots = NT >> shift;
    v0 = lr;
    if (AHEAD && n > 0) load();
  }
  __device__ __forceinline__ void load() {
#pragma unroll
    for (int i = 0; i < Q; ++i) {               // past the end: the last row, piece v0; not looked at
      const int at = row + slots * (P == 1 ? i : P == 2 ? i >> 1 : i >> 2), v = v0 + (i & (P - 1)) * L;
      const TX* xp = Xb + (long long)list[at < n ? at : n - 1] * ld;
      if (nvec > 0) q[i] = load16(xp + (long long)(v < nvec ? v : lr < nvec ? lr : 0) * V);
    }
  }
  template <typename FP, typename FS>
  __device__ __forceinline__ void visit(FP&& piece, FS&& single) {
    const int row_first = row;
    if (lr < nvec) {
      while (row < n) {
        uint4 c[Q];
        bool ok[Q];
        if (!AHEAD) load();
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          const int at = row + slots * (P == 1 ? i : P == 2 ? i >> 1 : i >> 2), v = v0 + (i & (P - 1)) * L;
          ok[i] = at < n && v < nvec;
          c[i] = q[i];
        }
        v0 += P * L;
        if (v0 >= nvec) {
          v0 = lr;
          row += slots * R;
        }
        if (AHEAD && row < n) load();
#pragma unroll
        for (int i = 0; i < Q; ++i)
          if (ok[i]) piece(c[i]);
      }
    }
    if (__builtin_expect(nvec * V < C, 0))
      for (int at = row_first; at < n; at += 4 * slots)
        for (int c = nvec * V + lr; c < C; c += L) {
          TX x[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int ri = at + i * slots;
            x[i] = Xb[(long long)list[ri < n ? ri : n - 1] * ld + c];
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (at + i * slots < n) single(x[i]);
        }
  }
};

// One pass of the search over rows list[0 .. n - 1]: the histogram of digits (key - k0 >> shift) - off.
// Digit 0 takes all that is below as well and is counted in a register (the result), the last digit takes all
// that is above and is not counted (what the others do not hold): either may be most of the set, and would meet in
// one word of LDS.  binary32: of the keys in [k0, k0 + span).  binary16: of all keys of the set, so that those below
// need no second compare, both halves of a word at once as in k_bracket_hist.
template <typename TX, int NT, int Q, bool AHEAD>
__device__ __forceinline__ u32 count_rows(const TX* __restrict__ Xb, long long ld, int C, int L,
                                           const unsigned short* list, int n, u32 k0, u32 span, int shift,
                                           int off, u32* h) {
  constexpr int kBins = 1 << kFinishBits;
  u32 low = 0;
  RowVisitor<TX, NT, Q, AHEAD> rows(Xb, ld, C, L, list, n);
  if constexpr (sizeof(TX) == 2) {
    const u32 first = k0 + (u32)off + (1u << shift);           // the first key of digit 1 (off: shift is 0)
    // keys of digits 1 to kBins - 2, no further than the range (what lies past it may be many ties)
    const u32 most = (u32)(kBins - 2) << shift, left = k0 + span - first, counted = left < most ? left : most;
    const u32 first2 = first | (first << 16);
    rows.visit([&](const uint4& q) {
      const u32 wd[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const u32 d2 = __builtin_bit_cast(u32, __builtin_bit_cast(s2v, wd[c] & 0x7FFF7FFFu) -
                                                   __builtin_bit_cast(s2v, first2));
        low += (u32)__builtin_popcount(d2 & 0x80008000u);
        const u32 dl = d2 & 0xFFFFu, dh = d2 >> 16;
        if (dl < counted) atomicAdd(&h[1 + (dl >> shift)], 1u);
        if (dh < counted) atomicAdd(&h[1 + (dh >> shift)], 1u);
      }
    },
               [&](TX x) {
                 const u32 k = Elem<TX>::key(x);
                 low += k < first ? 1u : 0u;
                 if (k >= first && k - first < counted) atomicAdd(&h[1 + ((k - first) >> shift)], 1u);
               });
  } else {
    auto count = [&](TX x) {
      const u32 d = Elem<TX>::key(x) - k0;
      const int digit = d < span ? (int)(d >> shift) - off : kBins;
      low += digit <= 0 ? 1u : 0u;
      if (digit > 0 && digit < kBins - 1) atomicAdd(&h[digit], 1u);
    };
    rows.visit([&](const uint4& q) {
      TX x[Elem<TX>::V];
      Elem<TX>::unpack(q, x);
#pragma unroll
      for (int c = 0; c < Elem<TX>::V; ++c) count(x[c]);
    },
               count);
  }
  return low;
}

// binary16: which window of `span` keys from k0 to look at, where the set has `from` keys below k0 and `to` below
// k0 + span, and the one of rank k lies between; cum = sampled keys before every 32nd, m in all.  Half of the
// window is below the sampled key that as large a share of the sampled ones in the range precede, because a set
// has keys closer to a gap than its sample.  The same in every wavefront.
__device__ __forceinline__ int place_window(const u32* cum, u32 m, u32 k0, u32 span, u32 from, u32 to, u32 k) {
  const u32 s_from = cum[k0 >> 5], s_to = k0 + span < 1u << 15 ? cum[(k0 + span) >> 5] : m;
  const u32 at = s_from + (u32)((float)(s_to - s_from) * ((float)(k - 1u - from) * __builtin_amdgcn_rcpf((float)(to - from))));
  int cell = -1;                                 // (cum[0] is 0)
#pragma unroll
  for (int i = 0; i < 1024 / 64; ++i)
    cell += (int)__popcll(__ballot(cum[i * 64 + (threadIdx.x & 63)] <= at));
  const int start = cell * 32 + 16 - kWindow / 2 - (int)k0, most = (int)span - kWindow;
  return start < 0 ? 0 : start > most ? most : start;
}

// The key in [k0, k0 + span) of rank `need` (1-based; binary32: among the set's keys in that range, binary16:
// among all of the set's), by the whole workgroup.  LISTED: the set's tokens are list[0 .. T - 1], otherwise
// those of T with gb[t] == j.  Every pass divides span by 2^kFinishBits, so two passes at most (binary32: three);
// window >= 0: one more before them that looks at the 2046 keys of the range from the window-th on one by one;
// cum != nullptr (see place_window, `from` and `to` as there): up to two such.  A pass reads all rows of the set,
// by one workgroup whose instructions set the pace (0.95 M elements 100 us), so what counts is how many passes
// there are.  Calibration by k_sets<WHOLE> where a fifth of the values is far below the others and the rank between,
// three passes with the window next to the interval, and now: [2, 4844, 586] with 16 sets, 14 missed, 410 and 120
// us; [10, 4349, 272] with 8, 9 missed, 339 and 104.  (With one window at the sample's place the first took 127.)
template <typename TX, int NT, bool LISTED>
__device__ __forceinline__ u32 search_rows(const TX* __restrict__ Xb, long long ld, int T, int C, int L,
                           const int* __restrict__ gb, int j, const unsigned short* list, u32 k0, u32 span,
                           unsigned long long need, int window, FinishLds<NT, LISTED>& s,
                           const u32* cum = nullptr, u32 m = 0, u32 from = 0, u32 to = 0) {
  constexpr int kBins = 1 << kFinishBits, NW = NT / 64, kPer = kBins / NT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int tries = cum ? 2 : 0;
  while (span > 1) {
    int shift = 32 - __clz(span - 1) - kFinishBits, off = 0;
    shift = shift > 0 ? shift : 0;
    if (LISTED && sizeof(TX) == 2 && tries > 0 && span > (u32)kBins) {
      window = place_window(cum, m, k0, span, from, to, (u32)need);
      --tries;
    }
    if (window >= 0 && span > (u32)kBins) {
      shift = 0;
      off = window;
    }
    window = -1;
    __syncthreads();
    for (int i = tid; i < kBins; i += NT) s.h[i] = 0;
    if (tid == 0) s.digit = kBins - 1;
    u32 low = 0;
    if constexpr (LISTED) {
      __syncthreads();
      low = count_rows<TX, NT, 8, false>(Xb, ld, C, L, list, T, k0, span, shift, off, s.h);
    } else {
      for (int t0 = 0; t0 < T; t0 += kFinishTokens) {
        constexpr int kIds = kFinishTokens / NT;
        bool mine[kIds];
        u32 count = 0;
#pragma unroll
        for (int u = 0; u < kIds; ++u) {
          const int t = t0 + u * NT + tid;
          mine[u] = t < T && gb[t] == j;
        }
#pragma unroll
        for (int u = 0; u < kIds; ++u) count += (u32)__popcll(__ballot(mine[u]));
        if (lane == 0) s.wtot[wave] = count;
        __syncthreads();
        u32 at = 0, n = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          at += w < wave ? s.wtot[w] : 0u;
          n += s.wtot[w];
        }
#pragma unroll
        for (int u = 0; u < kIds; ++u) {
          const unsigned long long m = __ballot(mine[u]);
          if (mine[u])
            s.list[at + (u32)__popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)(u * NT + tid);
          at += (u32)__popcll(m);
        }
        __syncthreads();
        low += count_rows<TX, NT, 4, false>(Xb + (long long)t0 * ld, ld, C, L, s.list, (int)n, k0, span, shift, off,
                                            s.h);
        __syncthreads();                        // `list` and `wtot` are reused
      }
    }
    // (one addition a wavefront: they all go to one word; by every thread, after every look at 2048 tokens, [38,
    // 37536, 8] with 4 sets, one missed, took 178 us and not 125)
    low = group_sum_u32<64>(low);
    if (lane == 63 && low) atomicAdd(&s.h[0], low);
    __syncthreads();
    // the bin where the running count reaches `need`
    unsigned long long mine = 0;
    u32 c[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      c[i] = s.h[tid * kPer + i];
      mine += c[i];
    }
    unsigned long long incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const unsigned long long o = __shfl_up(incl, d, 64);
      if (lane >= d) incl += o;
    }
    if (lane == 63) s.wsum[wave] = incl;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) incl += w < wave ? s.wsum[w] : 0ull;
    if (tid == NT - 1 && incl < need) s.rest = need - incl;       // the last digit
    if (incl - mine < need && need <= incl) {   // at most one thread
      unsigned long long cum = incl - mine;
      int i = 0;
      bool found = false;                       // (a break would put c into scratch memory)
#pragma unroll
      for (int k = 0; k < kPer - 1; ++k) {
        found = found || cum + c[k] >= need;
        cum += found ? 0u : c[k];
        i += found ? 0 : 1;
      }
      s.digit = (u32)(tid * kPer + i);
      s.rest = need - cum;
    }
    __syncthreads();
    const u32 digit = s.digit, first = digit == 0 ? 0u : (digit + (u32)off) << shift;
    const u32 next = digit == kBins - 1 ? span : (digit + (u32)off + 1u) << shift;
    k0 += first;
    span = (next < span ? next : span) - first;
    if (sizeof(TX) == 4) need = s.rest;
    if (LISTED && sizeof(TX) == 2) {                // (the counts around it are known only after a window)
      if (digit == 0) to = s.h[0];
      if (digit == kBins - 1) from = (u32)(need - s.rest);
    }
  }
  return k0;
}

// ---------------------------------------------------------------------------
// k_sets: one workgroup of NT threads per (image, token set).
//   1. the image's smallest and largest range key -> the key interval that belongs to this
//      set: gid = (key - lo) G / width is j exactly for ceil(j width / G) <= key - lo <
//      ceil((j + 1) width / G), so a token is recognised with two compares and no division;
//   2. the set's tokens (ids stored, counted, ranked) and their merged moments, summed
//      about the mean of the set's first token (identical tokens add exact zeros);
//   3. the sample of the set and the key interval that its order statistic says holds the
//      k-th smallest |x|.
// Bound by its chain of dependent steps (two trips to memory, six barriers), not by
// traffic: every workgroup reads the image's T range keys itself, which is cheaper than a
// kernel boundary, and everything per token sits in registers when T <= 16 NT.  Ranks are
// counted wavefront by wavefront (any numbering of the set's tokens serves the sample), so
// the wavefronts exchange one count each.  SM = most sampled elements: the rank error of 8 Ki
// is 0.45 % of the set's mass, about 40 keys at 1024 keys per octave where keys are dense, against
// a half-width of Wfew / 2 >= 256 keys; where they are not, W bins are used.  16 Ki are drawn with
// fewer bins per set (more than 32 sets), for the percentile base radius, with fewer than 8
// sets, whose tokens differ more, and for large sets that have no W bins to turn to.  A set smaller than the sample is read with as many loads as it
// has pieces (2048 images of [49, 96], 64 sets: 920 -> 640 us).
// Measured, calibration of one call (two kernels for this before: assignment, then sample):
// [1, 7744, 64] 46.3 -> 30.9 us, [8, 121, 512] 30.7 -> 26.0, [32, 4096, 1024] 118.7 -> 108.3;
// with 16 Ki samples 31.7 / 26.9 / 111.0.  Then, this kernel alone: the sample's loads issued
// before those of the moments, and the tokens listed by rank in LDS, so that only the drawn
// ones cost divisions (T <= kListTokens; the list of a larger image would not leave LDS for
// several workgroups): 24.8 -> 20.3 us at [32, 4096, 1024] (25.4 with 16 Ki samples), 14.4 -> 11.9 at
// [1, 7744, 64].
// ---------------------------------------------------------------------------
// WHOLE = 1 or 2 (ranks wanted: 2 with a percentile base radius): the kernel sees the set through to its
// radius.  G + extra workgroups an image are shared out to the sets by the sizes that one round of keys
// suggests, so that a large set's rows are read by many; each finds the set's tokens and interval itself,
// the same as the others, and then counts its share of the rows in LDS.
//
// Bound by instruction issue on few wavefronts: a dependent vector instruction takes 4 cycles, and a SIMD
// issues one in 4 cycles to all its wavefronts together, so everything that is done once per set costs
// (instructions) x 1.7 ns x (wavefronts per SIMD), and everything per element its instructions shared out.
// Hence 512 threads (256: too few loads in flight, [8, 1936, 320] 52.1 us the layer instead of 45.6; 1024:
// [1, 7744, 64] 27.1 instead of 26.4), exact small quotients in binary32 instead of integer divisions, scans
// by DPP, rounds of keys as a template parameter; and a taken branch into code that is not in the
// instruction cache costs 55 to 85 ns, so what rarely runs is out of the way.  The rows' first loads are
// issued before the sample is counted.
// Measured against the chain k_sets, k_bracket_hist, k_bracket_finish (each kernel boundary costs 1.4 us and
// 0.9 until the first loads are back), layer of [8, 121, 512] 25.7 -> 21.1 us, [1, 7744, 64] 30.5 -> 26.2,
// [16, 484, 320] 36.0 -> 33.2, [5, 1369, 333] with a percentile, where one sweep serves both ranks,
// 62.8 -> 39.2.  Every workgroup of a set adds the same 16 Ki sampled keys to its LDS, so binary16 images of few
// different values, which meet in few words, were slower than by the chain until the sample's histogram and
// such an interval's got copies; calibration, us by the chain, without and with copies: one value [19, 167, 2056]
// with 12 sets 51, 85, 35 and [2, 7625, 920] with 64 87, 113, 47; values within 1e-4 of 1 [29, 128, 1080] with 12 52,
// 89, 34; Laplace [16, 484, 320] 21.6, 17.7, 17.2.  80 registers (forced: 2 more are spilled) leave three workgroups
// on a CU, 768 sets at once; with 86 and two, calls of 1024 to 1536 sets took turns three times and many were
// slower than by the chain: [40, 100, 64] with 32 sets 23.1, 24.7, 20.3, [60, 37, 88] with 24 24.2, 26.0, 21.2.
// A rank k of a set of n elements as seen by a sample of m of them from n_sel tokens.
struct SampleRank {
  u32 rk;                     // the rank of the sample that corresponds to k
  float dev;                  // its standard deviation as that of a sample of independent elements
                              // (none if the sample is the set) ...
  float dev_tokens;           // ... and of a sample of whole tokens, as if all elements of a token
                              // lay on one side
};
// (where to look, not what is found there: one instruction each for reciprocal and root)
__device__ __forceinline__ SampleRank sample_rank(u32 k, u32 n, u32 m, int n_sel) {
  SampleRank s;
  const float mf = (float)m, share = mf * __builtin_amdgcn_rcpf((float)n);
  s.rk = (u32)((float)k * share + 0.5f);
  s.rk = s.rk < 1u ? 1u : (s.rk > m ? m : s.rk);
  const float pq = (float)s.rk * __builtin_amdgcn_rcpf(mf);
  const float var = n > m ? pq * (1.f - pq) * (1.f - share) * mf : 0.f;
  s.dev = __builtin_amdgcn_sqrtf(var > 0.f ? var : 0.f);
  s.dev_tokens = s.dev * __builtin_amdgcn_sqrtf(mf * __builtin_amdgcn_rcpf((float)n_sel));
  return s;
}

// binary16: whether W one-key bins centred on the middle of the bin bm of the sample's histogram that holds sampled
// rank s reach two and a half standard deviations to either side (cum as in place_bins).
__device__ __forceinline__ bool bins_reach(const u32* cum, int bm, const SampleRank& s, u32 m, int W) {
  constexpr int kCell = 1 << (15 - kSampleBits);
  const int reach = (int)(2.5f * s.dev) + 1, rk = (int)s.rk;
  auto below_bin = [&](int c) { return c <= 0 ? 0 : c >= 1024 ? (int)m : (int)cum[c]; };
  const int under = below_bin(bm - W / 2 / kCell + 1), upto = below_bin(bm + W / 2 / kCell);
  return (under == 0 || rk - under >= reach) && (upto == (int)m || upto - rk >= reach);
}

// binary16: the one-key bins around sampled rank s, which lies in bin bm of the sample's histogram of 1024
// bins (the low key bits do not matter to the interval), cum = sampled elements before every bin.  Wfew of
// them centred on the middle of that bin, if they reach far enough.  Else the rank lies where keys are sparse
// (just above the zeros of a rectified activation, between the values of a coarse grid): the W bins that leave
// equally many sampled keys on either side of it.  By one wavefront.
__device__ __forceinline__ void place_bins(const u32* cum, int bm, const SampleRank& s, u32 m, int Wfew,
                                           int W, u32& first, u32& width) {
  constexpr int kCell = 1 << (15 - kSampleBits);
  const int lane = threadIdx.x & 63, rk = (int)s.rk;
  auto below_bin = [&](int c) { return c <= 0 ? 0 : c >= 1024 ? (int)m : (int)cum[c]; };
  int lo = bm * kCell + kCell / 2 - Wfew / 2;
  width = (u32)Wfew;
  if (!bins_reach(cum, bm, s, m, Wfew)) {
    width = (u32)W;
    const int nb = W / kCell;                        // 8 to 64 candidates, one per lane
    const int c0 = bm - nb + 1 + lane;
    u32 score = 0;
    if (lane < nb && c0 >= 0) {                      // (the last one, c0 = bm, always is)
      const int left = rk - below_bin(c0), right = below_bin(c0 + nb) - rk;
      score = ((u32)(left < right ? left : right) << 6) | (u32)lane;
    }
    if (lane == nb - 1) score |= (u32)lane;
    score = (u32)__builtin_amdgcn_readlane((int)group_max_u32<64>(score), 63);
    lo = (bm - nb + 1 + (int)(score & 63u)) * kCell;
  }
  first = lo > 1 ? (u32)lo : 1u;                     // zeros are counted below
}

// Where a rank k of n lies that an interval does not hold: among `span` keys from k0, as their `rank`-th
// (binary16: the set's); `from` of the set's keys are smaller than these, from and these together `to`; binary16:
// probably in the window that starts at key k0 + window, next to the interval.  above = first key after the interval.
struct Lost {
  u32 k0, span, from, to;
  int window;
  unsigned long long rank;
};
template <bool F16>
__device__ __forceinline__ Lost lost_rank(u32 k, u32 n, u32 below, u32 inside, u32 lo, u32 above) {
  constexpr u32 kKeysAll = F16 ? 1u << 15 : 1u << 31;
  Lost l;
  l.window = F16 ? 0 : -1;
  if (k <= below) {                                  // (span 1: there are only zeros)
    l.k0 = 0;
    l.span = lo;
    l.from = 0;
    l.to = below;
    if (F16 && lo > (u32)kWindow) l.window = (int)lo - kWindow;
  } else {
    l.k0 = above < kKeysAll ? above : kKeysAll - 1u;
    l.span = kKeysAll - l.k0;
    l.from = below + inside;
    l.to = n;
  }
  l.rank = F16 ? k : (u64)(k - l.from);
  return l;
}

// MEET: binary32 sets that several workgroups share.  (A kernel of its own: the sets of one workgroup each, calls of 13 to 40 us,
// lost 0.3 to 1.4 us to the code and the registers, 126 instead of 84, of a way that they never take.)
template <typename TX, int NT, int RD, int SM, int WHOLE, bool MEET = false>
__global__ __launch_bounds__(NT, (MEET ? 4 : WHOLE == 1 && sizeof(TX) == 2 && RD <= 8 ? 6 : 1)) void k_sets(
    const TX* __restrict__ X, long long ld, int T, int C, int G, int Wfew, int W, int cells, int aligned,
    const float* __restrict__ r, const double* __restrict__ mean, const double* __restrict__ m2,
    int* __restrict__ gid, Scalars sc, int pass, int keep_base, GroupWork* __restrict__ grp,
    Bracket* __restrict__ br, u32* __restrict__ bhist, u32* __restrict__ lists, int cap,
    u32* __restrict__ img_flag, u32* __restrict__ status, WholeArgs wa) {
  constexpr int NW = NT / 64;
  constexpr bool F16 = sizeof(TX) == 2;
  constexpr int V = Elem<TX>::V;
  constexpr int kHalf = RD > 1 ? RD / 2 : 1;
  constexpr int kSampleRuns = SM / kRunLen;
  constexpr int kSampleTokens = kSampleRuns;         // at most one run per token
  // binary32 values of one magnitude share their top bits, and binary16 ones may be few and the same: four
  // copies of the first histogram keep the lanes of a wavefront from all adding to one word
  constexpr int kCopies = F16 && !WHOLE ? 1 : 4;
  extern __shared__ unsigned short order[];          // the set's tokens by rank (T <= kListTokens)
  __shared__ int sel[WHOLE ? 1 : kSampleTokens];     // more tokens: the one drawn of every stratum
  __shared__ __attribute__((aligned(16))) u32 shist[kCopies << kSampleBits];   // sample histogram
                                                     // over the top key bits
  __shared__ u32 snext[F16 ? 1 : 2][F16 ? 1 : 1 << kSampleBits];   // binary32: two over the next ones
  __shared__ u32 s_cell[F16 ? 1 : 66], s_mode, s_tie;   // binary32: sampled keys per cell, one more at each end
  __shared__ __attribute__((aligned(16))) u32 cum[F16 ? 1024 : 4];                // binary16: sampled elements before every bin
  __shared__ u32 s_bin[4], s_before[4];
  __shared__ u32 s_min[NW], s_max[NW], wtot[NW], stot[3][NW], s_cmax[NW];
  __shared__ double s_s1[NW], s_s2[NW];
  __shared__ float s_sigma, s_cbase;
  __shared__ int s_first;
  // (whole)
  __shared__ __attribute__((aligned(16))) u32 hist[WHOLE ? (F16 ? WHOLE : 1) : 1][WHOLE ? 2048 : 4];
  __shared__ u32 s_lo[2], s_width[2], s_below[2], s_copies[2], s_last;
  __shared__ u32 s_share[64];                        // sampled tokens of every set
  __shared__ Lost s_lost[2];
  __shared__ FinishLds<WHOLE ? NT : 64, true> s_search;
  __shared__ unsigned s_known;                       // of known_to_all alone
  __shared__ unsigned short s_parts[MEET ? NT + 1 : 1];     // shares of the set's rows claimed by this workgroup
  // (whole: the set, and which of the S workgroups that share it this is, follow from the sets' sizes)
  int S = 1, part = 0, j = (int)blockIdx.x;
  const int b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* rb = r + (long long)b * T;
  const double* meanb = mean + (long long)b * T;
  const double* m2b = m2 + (long long)b * T;
  int* gb = gid + (long long)b * T;
  constexpr u32 kDead = 0xFFFFFFFFu;                 // no range key reaches it
  const bool one_batch = WHOLE || T <= RD * NT;
  u32 kv[RD];
  auto load_keys = [&](int t0) {
#pragma unroll
    for (int u = 0; u < RD; ++u) {
      const int t = t0 + u * NT + tid;
      kv[u] = t < T ? __float_as_uint(rb[t]) : kDead;
    }
  };
  // (the rounds of a batch that hold tokens; the same for every thread)
  auto in_use = [&](int t0, int u) { return u == 0 || t0 + u * NT < T; };

  // ---- 1: key range of the image, key interval of the set
  load_keys(0);
  for (int i = tid; i < (kCopies << kSampleBits) / 4; i += NT)
    reinterpret_cast<uint4*>(shist)[i] = make_uint4(0, 0, 0, 0);
  if (WHOLE && tid < 64) s_share[tid] = 0;
  if (!F16) {
    for (int i = tid; i < (int)(sizeof(snext) / sizeof(u32)); i += NT) (&snext[0][0])[i] = 0;
    if (tid < 66) s_cell[tid] = 0;
    if (tid == 0) s_mode = 0;
  }
  u32 kinv = 0, kmax = 0;                            // largest ~key, largest key
  for (int t0 = 0;;) {
#pragma unroll
    for (int u = 0; u < RD; ++u) {
      const u32 k = kv[u];
      kinv = ~k > kinv ? ~k : kinv;                  // ~kDead is 0
      kmax = k != kDead && k > kmax ? k : kmax;
    }
    t0 += RD * NT;
    if (one_batch || t0 >= T) break;
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
  if (tid == 0 && blockIdx.x == 0) {
    const u32 flag = hi >= 0x7F800000u ? TDQ_DEV_NONFINITE : 0u;
    img_flag[b] = flag;
    if (WHOLE) {                          // (cleared by the statistics kernel, like the counts)
      if (flag) atomicOr(&status[0], flag);
    } else if (b == 0) {                         // counts of sets the sampled interval misses
      status[1 + pass] = 0u;
      if (!keep_base) status[1 + (pass ^ 1)] = 0u;
    }
  }
  // ceil(j width / G) = j q + ceil(j rem / G) with width = q G + rem; everything fits 32 bits
  const u32 width = hi - lo + 1u;
  // x / G: (x + 1/2) / G is at least 1 / 128 from any integer, so the rounded reciprocal does
  auto div_g = [&](u32 x) { return (u32)(((double)x + 0.5) * sc.inv_groups); };
  const u32 wq = div_g(width), wr = width - wq * (u32)G;
  auto start_of = [&](int g) {
    return g == 0 ? 0u : g >= G ? hi + 1u : lo + (u32)g * wq + div_g((u32)g * wr + (u32)G - 1u);
  };
  if constexpr (WHOLE != 0) {
    // How many workgroups a set gets: one, and its share of the others by the keys that one round of the
    // image's tokens, spread over all of them, holds (about: no integer division, every workgroup alike).
    const int pick = tid & (RD - 1);                 // (a power of two; some threads have none)
    u32 k = kDead;
#pragma unroll
    for (int u = 0; u < RD; ++u) k = u == pick ? kv[u] : k;
    if (k != kDead) {
      const int g = (int)((float)(k > lo ? k - lo : 0u) * ((float)G / (float)width));
      atomicAdd(&s_share[g < G ? g : G - 1], 1u);
    }
    __syncthreads();
    const u32 drawn = s_share[lane], all = xor_reduce_sum<64, u32>(drawn);
    // (a little less than its share, so that rounding never makes it more than G + extra together)
    const float per = (float)wa.extra / (float)all * (1.f - 1e-6f);
    const u32 its = lane < G ? 1u + (u32)((float)drawn * per) : 0u, incl = wave_scan_u32(its);
    const u32 at = turned(blockIdx.x, gridDim.x, blockIdx.y);
    const unsigned long long later = __ballot(incl > at);
    if (__builtin_expect(later == 0, 0)) return;     // the same for every thread
    j = __ffsll((long long)later) - 1;
    S = F16 || MEET ? __builtin_amdgcn_readlane((int)its, j) : 1;
    part = !F16 && !MEET ? 0 : (int)at - (__builtin_amdgcn_readlane((int)incl, j) - S);
    // (binary32; there is time until it is looked at)
    if (MEET && S > 1 && tid == 0)
      s_parts[0] = (unsigned short)min(atomicAdd(&wa.ctl[(size_t)(b * G + j) * kSetCtl + kCtlClaimed], 1u), 0xFFFFu);
  }
  const u32 start = start_of(j), end = start_of(j + 1);
  auto in_set = [&](u32 k) { return k >= start && k < end; };

  // ---- 2: the set's tokens
  u32 wcount = 0;
  for (int t0 = 0; WHOLE ? t0 == 0 : t0 < T; t0 += RD * NT) {
    if (!one_batch) load_keys(t0);
#pragma unroll
    for (int u = 0; u < RD; ++u) {
      if (!in_use(t0, u)) break;
      wcount += (u32)__popcll(__ballot(in_set(kv[u])));
    }
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
  const int idx = b * G + j;
  if (__builtin_expect(tokens_u == 0, 0)) {
    if (tid == 0) {
      GroupWork w;
      w.n = 0; w.k_rem = 0; w.prefix = 0; w.tokens = 0; w.c_base = 0.f; w.sigma = 0.f;
      if (WHOLE) {
        if (part == 0) project_store(idx, w, 0u, F16, sc, wa.clip, wa.scale, wa.stats);
        return;
      }
      grp[idx] = w;
      Bracket e;
      e.lo = 0; e.width = 0; e.below = 0; e.shift = 0;
      br[idx] = e;
    }
    return;
  }

  // the sweep adds into this set's histogram: clear it here (more of it below if more is used)
  if (!WHOLE)
    for (int i = tid; i < Wfew; i += NT) bhist[(size_t)idx * W + i] = 0;

  // Sample geometry.  The set's tokens are cut into strata of `stride` tokens (at most
  // kSampleTokens strata) and one token is drawn from each at a hashed position: a regular
  // stride would alias with any period the token sequence has (image rows).  Of each drawn
  // token `rpt` runs of kRunLen consecutive channels are read, the first at a hashed offset,
  // so that all channels are represented; a row that fits is read whole, up to the last
  // V - 1 channels of a row that is not made of whole 16-byte pieces.
  const int tokens = (int)tokens_u;
  const int stride = (tokens + kSampleTokens - 1) / kSampleTokens;
  const int n_sel = (tokens + stride - 1) / stride;         // <= kSampleTokens
  const int Cv = C >= V ? C - C % V : C;                    // channels in whole pieces
  const int row_runs = (Cv + kRunLen - 1) / kRunLen;
  int rpt = kSampleRuns / n_sel;                            // runs per drawn token, >= 1
  rpt = rpt < row_runs ? rpt : row_runs;
  const int cw = rpt == row_runs ? Cv : rpt * kRunLen;      // channels read per drawn token
  const int n_runs = n_sel * rpt;                           // <= kSampleRuns
  const u32 m = (u32)(n_sel * cw);                          // sample size, <= SM
  const bool listed = WHOLE || T <= kListTokens;
  auto pick_of = [&](u32 stratum) {                         // rank of the token drawn from a stratum
    const u32 first = stratum * (u32)stride;
    const u32 len = (u32)tokens - first < (u32)stride ? (u32)tokens - first : (u32)stride;
    return first + mod24(((stratum + 1u) * 2246822519u + (u32)idx * 3266489917u) >> 12, len);
  };

  for (int t0 = 0; WHOLE ? t0 == 0 : t0 < T; t0 += RD * NT) {
    if (!one_batch) load_keys(t0);
#pragma unroll
    for (int u = 0; u < RD; ++u) {
      if (!in_use(t0, u)) break;
      const bool mine = in_set(kv[u]);
      const unsigned long long mask = __ballot(mine);
      if (RD > 4 && mask == 0) continue;                    // uniform over the wavefront
      if (mine) {
        const int t = t0 + u * NT + tid;
        const u32 rank = running + (u32)__popcll(mask & ((1ull << lane) - 1ull));
        if (part == 0) gb[t] = j;
        if (listed) {
          order[rank] = (unsigned short)t;
        } else {
          if (rank == 0) s_first = t;
          const u32 stratum = rank / (u32)stride;
          if (!WHOLE && rank == pick_of(stratum)) sel[WHOLE ? 0 : stratum] = t;
        }
      }
      running += (u32)__popcll(mask);
    }
  }
  __syncthreads();
  if constexpr (MEET) {
    if (S > 1 && (int)s_parts[0] >= S) return;       // nothing of the set is left (the same for every thread)
  }

  // The sample's loads first, in flight together with those of the moments.  Pieces of V
  // channels: piece p = NT e + tid is part p % PPR of run p / PPR, so a wavefront's load
  // instruction fetches whole runs of 64 (128) bytes; they are issued unconditionally, from a
  // valid address where there is no piece.
  constexpr int kKeyBits = F16 ? 15 : 31;
  constexpr int kKeys = SM / NT;                       // sampled keys per thread
  constexpr int kPieces = kKeys / V, PPR = kRunLen / V;
  uint4 v[kPieces];
  bool live[kPieces];
  const int steps = (n_runs * PPR + NT - 1) / NT;      // small sets need fewer than kPieces
  // offsets in steps of whole pieces where the rows consist of aligned ones
  const u32 step = aligned ? (u32)V : 1u, offsets = (u32)(C - cw) / step + 1u;
  const float per_token = 1.f / (float)rpt;
  auto load_piece = [&](int e) {
    const u32 p = (u32)(e * NT + tid), q = p / PPR, part = p % PPR;
    const u32 slot = (u32)(((float)q + 0.5f) * per_token), run = q - slot * (u32)rpt;      // q / rpt (q < 2^10)
    const int at = (int)(run * kRunLen + part * V);    // channel inside the part of the row read
    live[e] = q < (u32)n_runs && at < cw;
    const u32 sl = live[e] ? slot : 0u;
    const int t = !listed ? sel[WHOLE ? 0 : sl] : order[stride == 1 ? sl : pick_of(sl)];
    const u32 off = mod24((u32)t * 2654435761u >> 8, offsets) * step;
    const TX* src = X + ((long long)b * T + t) * ld + (live[e] ? (int)off + at : 0);
    if (__builtin_expect(C >= V, 1)) {
      v[e] = load16(src);
    } else {                                           // rows shorter than a piece
      TX x[V];
#pragma unroll
      for (int i = 0; i < V; ++i) x[i] = src[i < C ? i : 0];
      v[e] = *reinterpret_cast<const uint4*>(x);
    }
  };
#pragma unroll
  for (int e = 0; e < kPieces; ++e)
    if (e < steps) load_piece(e);                      // uniform

  // (whole, binary16: the first loads of this workgroup's share of the rows as well)
  const int share = WHOLE && F16 ? (tokens + S - 1) / S : 0, share_from = part * share;
  const int share_rows = tokens - share_from < share ? tokens - share_from : share;     // (none if negative)
  RowVisitor<TX, NT, 4, true> own(X + (long long)b * T * ld, ld, C, WHOLE && F16 ? wa.L : 1,
                         order + (share_rows > 0 ? share_from : 0), WHOLE && F16 ? share_rows : 0);

  // (of workgroups that share a binary32 set the first to claim a share projects, or does everything alone)
  bool sums = true;
  if constexpr (MEET) sums = S == 1 || s_parts[0] == 0;
  // Moments of the set about the mean of its first token (zero if that is not finite: the
  // image's results are then undefined anyway and its flag is raised).
  const int first_token = listed ? order[0] : s_first;
  double piv = meanb[first_token];
  const double cn = (double)C;
  double a1 = 0.0, a2 = 0.0;
  u32 cmax = 0;
  piv = (piv - piv == 0.0) ? piv : 0.0;
  for (int t0 = 0; WHOLE ? t0 == 0 && sums : t0 < T; t0 += RD * NT) {
    if (!one_batch) load_keys(t0);
    // half of the rounds at a time, their loads issued together (a token of another set
    // reads the first token's entry, which is not added)
#pragma unroll
    for (int h = 0; h < RD; h += kHalf) {
      if (!in_use(t0, h)) break;
      double mv[kHalf], qv[kHalf];
#pragma unroll
      for (int u = 0; u < kHalf; ++u) {
        const bool mine = in_set(kv[h + u]);
        mv[u] = piv;
        qv[u] = 0.0;
        if (RD <= 4 || __ballot(mine)) {              // uniform over the wavefront
          const int t = mine ? t0 + (h + u) * NT + tid : first_token;
          mv[u] = meanb[t];
          qv[u] = m2b[t];
        }
      }
#pragma unroll
      for (int u = 0; u < kHalf; ++u) {
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

  // ---- 3: the sample.  Every live key adds one to an LDS histogram of its top kSampleBits
  // bits; zeros, often many, are counted first (binary16: bin 0 is what the others do not hold).
  // (binary32, workgroups that share a set: two more bits instead of the copies)
  constexpr int kFineBits = kSampleBits + 2;
  static_assert(F16 || 1 << kFineBits == kCopies << kSampleBits, "the same words");
  u32 key[F16 ? 1 : kKeys], zeros = 0;
  auto add_piece = [&](int e) {
    if constexpr (F16) {
      const u32 wd[4] = {v[e].x, v[e].y, v[e].z, v[e].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const u32 x = live[e] ? wd[i] : 0u;
        const u32 b0 = (x >> (kKeyBits - kSampleBits)) & 1023u, b1 = (x >> (16 + kKeyBits - kSampleBits)) & 1023u;
        if (b0 != 0u && 2 * i < C) atomicAdd(&shist[b0 * kCopies + (lane & (kCopies - 1))], 1u);
        if (b1 != 0u && 2 * i + 1 < C) atomicAdd(&shist[b1 * kCopies + (lane & (kCopies - 1))], 1u);
      }
    } else {
      TX x[V];
      Elem<TX>::unpack(v[e], x);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const u32 k = live[e] && i < C ? Elem<TX>::key(x[i]) : kDead;
        key[e * V + i] = k;
        zeros += k == 0u ? 1u : 0u;
        if (k != kDead && k != 0u)
          atomicAdd(&shist[S > 1 ? k >> (kKeyBits - kFineBits)
                                 : (k >> (kKeyBits - kSampleBits)) * kCopies + (lane & (kCopies - 1))], 1u);
      }
    }
  };
#pragma unroll
  for (int e = 0; e < kPieces; ++e)
    if (e < steps) add_piece(e);
  if (!F16 && __builtin_expect(__ballot(zeros != 0) != 0, 0)) {
    zeros = group_sum_u32<64>(zeros);
    if (lane == 63) atomicAdd(&shist[0], zeros);
  }
  __syncthreads();

  // the set's working record: n, base radius, sigma, rank of this pass (binary64)
  GroupWork w;
  w.tokens = tokens_u;
  const u32 nn = tokens_u * (u32)C;      // (an image that samples has fewer than 2^32 elements)
  w.n = (long long)nn;
  w.prefix = 0;
  const double n = (double)nn;
  auto rank_of = [&](double share) {
    const u32 k = (u32)ceil(share * n);
    return k < 1u ? 1u : (k > nn ? nn : k);
  };
  const u32 k_pass = rank_of(pass == kPassBase ? sc.base_pct : sc.zr);
  w.k_rem = (long long)k_pass;
  // sigma and c_base, by one wavefront while others have something else to do: forty dependent binary64 steps
  auto finish_moments = [&]() {
    const bool has = lane < NW;
    const double S1 = group_sum_f64<64>(has ? s_s1[has ? lane : 0] : 0.0);
    const double S2 = group_sum_f64<64>(has ? s_s2[has ? lane : 0] : 0.0);
    const u32 km = group_max_u32<64>(has ? s_cmax[has ? lane : 0] : 0u);
    if (lane == 63) {
      const double mu = S1 / n;
      double var = S2 / n - mu * mu;
      var = var > 0.0 ? var : 0.0;
      w.sigma = (float)(sqrt(var) + sc.eps_std);
      // (the base-radius pass left its radius in the record)
      w.c_base = keep_base ? grp[idx].c_base : __uint_as_float(km);
      if (WHOLE) {
        s_sigma = w.sigma;
        s_cbase = w.c_base;
      } else {
        grp[idx] = w;
      }
    }
  };
  if (!WHOLE && !F16 && wave == NW - 1) finish_moments();
  // binary32: the interval between two order statistics of the sample, six standard deviations of its
  // elements and one of its tokens to either side of s, each resolved to 20 of its 31 bits: first key, last
  // key - first key, sampled ranks between them.  By the whole workgroup.  Where workgroups share a set a miss costs
  // one more round and keys in the interval room and time: four and a half, to 12 bits (a sixteenth of an octave, in
  // one step) unless that holds three times the sampled keys wanted, else to 22.
  auto interval32 = [&](const SampleRank& s, u32& first, u32& last, u32& drawn) {
    if constexpr (!F16) {
      const int dr = (int)(S > 1 ? 4.f * s.dev + 0.5f * s.dev_tokens : 6.f * s.dev + s.dev_tokens) + 2, rk = (int)s.rk;
      const u32* const hs[2] = {shist, shist};
      const u32 rs[2] = {(u32)(rk - dr < 1 ? 1 : rk - dr), (u32)(rk + dr > (int)m ? (int)m : rk + dr)};
      drawn = rs[1] - rs[0];
      // top digits of a key, and the ten bits after them
      const int top_at = S > 1 ? kKeyBits - kFineBits : kKeyBits - kSampleBits, next_at = top_at - 10;
      if (S > 1)
        find_ranks<NT, 2, 1, false, 1 << kFineBits>(hs, rs, stot, s_bin, s_before, nullptr);
      else
        find_ranks<NT, 2, kCopies, false>(hs, rs, stot, s_bin, s_before, nullptr);
      __syncthreads();
      const u32 b0 = s_bin[0], b1 = s_bin[1];
      if (MEET && S > 1) {
        // whole sixteenths of an octave, unless they hold far more than is wanted
        const u32 held = s_before[1] + shist[b1] - s_before[0];
        if (held <= 3u * drawn) {                      // the same for every thread
          first = b0 << top_at;
          first = first > 1u ? first : 1u;             // zeros are counted below
          last = ((b1 + 1u) << top_at) - 1u - first;
          return;
        }
      }
#pragma unroll
      for (int i = 0; i < kKeys; ++i) {
        if (i / V < steps) {
          const u32 top = key[i] >> top_at, next = (key[i] >> next_at) & 1023u;
          if (key[i] != kDead && top == b0) atomicAdd(&snext[0][next], 1u);
          if (key[i] != kDead && top == b1 && b1 != b0) atomicAdd(&snext[1][next], 1u);
        }
      }
      __syncthreads();
      const u32* const hn[2] = {snext[0], snext[b1 != b0 ? 1 : 0]};
      const u32 rn[2] = {rs[0] - s_before[0], rs[1] - s_before[1]};
      find_ranks<NT, 2, 1, false>(hn, rn, stot, s_bin + 2, s_before + 2, nullptr);
      __syncthreads();
      first = (b0 << top_at) | (s_bin[2] << next_at);
      first = first > 1u ? first : 1u;                 // zeros are counted below
      last = ((b1 << top_at) | (s_bin[3] << next_at)) + ((1u << next_at) - 1u) - first;
    }
  };
  if constexpr (WHOLE != 0) {
    // ---- 4: the set's own rows: counts below the interval(s) and inside, rank, projection
    constexpr int NR = WHOLE;                          // the last rank is the one that is projected
    constexpr int kBins = 2048;
    const TX* Xb = X + (long long)b * T * ld;
    u32 k[NR];
    if (NR == 2) k[0] = rank_of(sc.base_pct);
    k[NR - 1] = k_pass;
    u32 found = 0, base_key = 0;
    auto search = [&](const Lost& l) {
      return search_rows<TX, NT, true>(Xb, ld, tokens, C, wa.L, nullptr, j, order, l.k0, l.span, l.rank, -1,
                                       s_search, F16 ? cum : nullptr, m, l.from, l.to);
    };
    if constexpr (F16) {
      SampleRank sq[NR];
      const u32* hs[NR];
      u32 rs[NR];
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        sq[q] = sample_rank(k[q], nn, m, n_sel);
        hs[q] = shist;
        rs[q] = sq[q].rk;
      }
      find_ranks<NT, NR, kCopies, true>(hs, rs, stot, s_bin, s_before, cum, m);
      for (int i = tid; i < NR * kBins / 4; i += NT) reinterpret_cast<uint4*>(&hist[0][0])[i] = make_uint4(0, 0, 0, 0);
      __syncthreads();
      // Bins of a rank at most.  Workgroups that share a set meet in its W words, so two ranks have half each; but
      // where that does not reach for one of them and 512 do for the other, it has the rest (the zr quantile just
      // above 18 % zeros: [5, 1019, 604] with 4 sets and a percentile 61 us, 26 so, 48 by the chain).
      int room[NR];
      for (int q = 0; q < NR; ++q) room[q] = NR == 2 && S > 1 ? W / 2 : W;
      if (NR == 2 && S > 1 && W == 2048) {
        auto reach = [&](int q, int bins) { return bins_reach(cum, (int)s_bin[q], sq[q], m, bins); };
        const bool half_0 = reach(0, W / 2), half_1 = reach(NR - 1, W / 2);
        const bool more_0 = !half_0 && half_1 && reach(NR - 1, 512), more_1 = !half_1 && reach(0, 512);
        room[0] = more_1 ? 512 : more_0 ? 1536 : W / 2;
        room[NR - 1] = more_1 ? 1536 : more_0 ? 512 : W / 2;
      }
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        if (wave == q) {
          u32 first, wd;
          const int most = room[q];
          // Where an eighth of the sample lies in the rank's cell (ordinary data has a fiftieth there) a few keys hold
          // most of the set: the interval's bins get as many copies as there is room for, each in the next bank.
          const int cell = (int)s_bin[q];
          const bool hot = ((cell < 1023 ? cum[cell + 1] : m) - cum[cell]) * 8 >= m;
          int few = q == NR - 1 && Wfew < most ? Wfew : most;
          few = hot && few > 512 ? 512 : few;
          place_bins(cum, cell, sq[q], m, few, most, first, wd);
          if (lane == 0) {
            s_lo[q] = first; s_width[q] = wd; s_below[q] = 0;
            s_copies[q] = !hot || wd > 1024u ? 0u : wd <= 512u ? 2u : 1u;
          }
        }
      }
      __syncthreads();
      u32 first[NR], wd[NR], below[NR], copies[NR];    // (log2)
      bool hot = false;
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        first[q] = s_lo[q];
        wd[q] = s_width[q];
        below[q] = 0;
        copies[q] = (u32)__builtin_amdgcn_readfirstlane((int)s_copies[q]);
        hot = hot || copies[q] != 0;
      }
      // (two versions, because an address without copies takes an instruction less)
      auto look = [&](auto several) {
        u32* bins[NR];
        u32 by[NR];
#pragma unroll
        for (int q = 0; q < NR; ++q) {
          by[q] = decltype(several)::value ? copies[q] : 0u;
          bins[q] = decltype(several)::value ? hist[q] + (lane & ((1 << copies[q]) - 1)) : hist[q];
        }
        own.visit([&](const uint4& p) {
          const u32 wd4[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const s2v kk = __builtin_bit_cast(s2v, wd4[c] & 0x7FFF7FFFu);
#pragma unroll
            for (int q = 0; q < NR; ++q) {
              // both halves at once, see k_bracket_hist
              const u32 d2 = __builtin_bit_cast(u32, kk - __builtin_bit_cast(s2v, first[q] | (first[q] << 16)));
              below[q] += (u32)__builtin_popcount(d2 & 0x80008000u);
              const u32 dl = d2 & 0xFFFFu, dh = d2 >> 16;
              if (dl < wd[q]) atomicAdd(&bins[q][dl << by[q]], 1u);
              if (dh < wd[q]) atomicAdd(&bins[q][dh << by[q]], 1u);
            }
          }
        },
                  [&](TX x) {
                    const u32 kx = Elem<TX>::key(x);
#pragma unroll
                    for (int q = 0; q < NR; ++q) {
                      below[q] += kx < first[q] ? 1u : 0u;
                      if (kx >= first[q] && kx - first[q] < wd[q]) atomicAdd(&bins[q][kx - first[q] << by[q]], 1u);
                    }
                  });
      };
      if (__builtin_expect(hot, 0))
        look(std::true_type());
      else
        look(std::false_type());
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const u32 t = group_sum_u32<64>(below[q]);
        if (lane == 63 && t) atomicAdd(&s_below[q], t);
      }
      __syncthreads();
      if (__builtin_expect(hot, 0)) {                  // the copies of a bin together, at its place without copies
        u32 v[NR][2];
#pragma unroll
        for (int q = 0; q < NR; ++q) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const u32* at = &hist[q][((i * NT + tid) << copies[q]) & (kBins - 1)];
            v[q][i] = at[0] + (copies[q] > 0 ? at[1] : 0u) + (copies[q] > 1 ? at[2] + at[3] : 0u);
          }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NR; ++q)
          if (copies[q])
            for (int i = 0; i < 2; ++i) hist[q][i * NT + tid] = (u32)(i * NT + tid) < wd[q] ? v[q][i] : 0u;
        __syncthreads();
      }
      if (S > 1) {
        // The parts of a set meet in its global histogram, and the last to arrive goes on.  All that they
        // exchange is written and read by device-scope atomic operations, which are performed where all
        // XCDs see them, so no cache has to be written back or invalidated; s_waitcnt waits until those of
        // this wavefront have been, the barrier for the other wavefronts, and only then is the arrival counted.
        u32* gh = bhist + (size_t)idx * W;
        u32* ctl = wa.ctl + (size_t)idx * kSetCtl;
        static_assert(kCtlArrived == 0 && kCtlBelow == 1, "as below");
#pragma unroll
        for (int q = 0; q < NR; ++q) {
          for (int i = tid; i < (int)wd[q]; i += NT) {
            const u32 v = hist[q][i];
            if (v) atomicAdd(&gh[q * room[0] + i], v);
          }
          if (tid == q && s_below[q]) atomicAdd(&ctl[1 + q], s_below[q]);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) s_last = atomicAdd(&ctl[0], 1u) == (u32)S - 1u ? 1u : 0u;
        __syncthreads();
        if (s_last == 0) return;                       // the same for every thread
        constexpr int kPer = kBins / NT;
#pragma unroll
        for (int q = 0; q < NR; ++q) {
          u32 v[kPer];
#pragma unroll
          for (int i = 0; i < kPer; ++i) {
            const int at = i * NT + tid;
            v[i] = at < (int)wd[q] ? __hip_atomic_load(&gh[q * room[0] + at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
          }
#pragma unroll
          for (int i = 0; i < kPer; ++i) hist[q][i * NT + tid] = v[i];
          if (tid == q) s_below[q] = __hip_atomic_load(&ctl[1 + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
      }
      if (wave == NW - 1) finish_moments();
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        if (wave == q) {
          const BinPick p = pick_bin<false>(hist[q], (int)wd[q], s_below[q], k[q]);
          Lost l = lost_rank<true>(k[q], nn, s_below[q], p.inside, first[q], first[q] + wd[q]);
          if (p.ok) {
            l.k0 = first[q] + p.bin;
            l.span = 1u;
          }
          if (lane == 0) s_lost[q] = l;
        }
      }
      __syncthreads();
#pragma unroll 1
      for (int q = 0; q < NR; ++q) {
        u32 key_q = s_lost[q].k0;
        if (__builtin_expect(s_lost[q].span != 1u, 0)) {                            // the interval missed the rank
          if (tid == 0) atomicAdd(&status[1 + (q == NR - 1 ? kPassZr : kPassBase)], 1u);
          key_q = search(s_lost[q]);
        }
        if (q == NR - 1) found = key_q; else base_key = key_q;
      }
    } else {
      // A set's rank by several workgroups together.  The set's rows are S shares; a workgroup claims one (in the order
      // in which they come, not by its place in the grid), lists the keys of its rows that lie in the interval (in
      // LDS, thread by thread) and counts them in bins.  When the counts of all shares have met in the
      // workspace, every workgroup reads them and goes on with the bin that holds the rank; the one that claimed the first
      // share gets the keys of that bin, a few dozen, and picks among them.  Where a bin has too many keys
      // (ties, gaps), or the interval misses the rank, the same again with the range that is known to hold it.
      // Workgroups wait for each other, and nothing makes all of a launch run at the same time: whoever has waited
      // for wa.waits.patience claims another share, so that a wait only ever depends on workgroups that run, and one that
      // starts when nothing is left leaves.  (Words that a second call on the same workspace overwrites could keep
      // it waiting all the same: after wa.waits.limit the helpers leave, and the first does everything alone.)
      // What they exchange goes through device-scope atomic operations, as for binary16 above.
      // Bound by its chain of steps: [8, 1024, 768] with 16 sets from the first kernel on, us: range and tokens 4, sample
      // and interval 6, the rows 4 (25 MB at 6 TB/s), counts met and read 4, keys of the bin 3, skew.  Calibration by
      // the chain of five kernels, which reads the rows once more, and so: 46 and 34.4; with the interval's ends found in
      // two steps always 35.9; without the list, rows read
      // again for the bin's keys, 36.5; lists by wavefront with a ballot per element 37; the rows' first loads issued
      // before the sample (44 bytes of scratch) 36.4.
      enum { kProject, kLeave, kAlone };
      auto shared_rank = [&](u32 kq, u32 first, u32 last) {
        constexpr u32 kSeg = (kCopies << kSampleBits) / NT;      // keys a thread lists, where the sample was counted
        const int wbins = W / 2;                       // of the set's words these are bins, the others take the keys
        u32* gh = bhist + (size_t)idx * W;
        u32* gl = gh + wbins;
        u32* ctl = wa.ctl + (size_t)idx * kSetCtl;
        const u32 keep = wbins < NT ? (u32)wbins : (u32)NT;
        static_assert(NT + 16 <= 1 << kFinishBits, "the keys of the last bin fit the search's histogram");
        auto load = [&](const u32* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        const bool picks = s_parts[0] == 0;
        int n_parts = 1;                               // shares of this workgroup, listed in s_parts
        u32 events = 0;                                // how often every share has been counted to have arrived
        auto arrive = [&](int shares) {                // for thread 0: how many have with these
          return atomicAdd(&ctl[kCtlArrived], (u32)shares) + (u32)shares;
        };
        auto settle = [&]() {                          // what this workgroup has sent is where all see it
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          __syncthreads();
        };
        auto until = [&](u32 patience, auto&& so) {      // (looks until it is, or until it has waited long enough)
          bool is = so();
          if (!is) {
            const long long since = wall_clock64();
#pragma unroll 1
            do is = so();
            while (!is && wall_clock64() - since < (long long)patience);
          }
          return is;
        };
        auto reached = [&](int word, u32 value, u32 patience) {
          return known_to_all(&s_known, [&]() { return until(patience, [&]() { return load(&ctl[word]) >= value; }); });
        };
        const int share = (tokens + S - 1) / S;
        u32 k0 = first, span = last + 1u;              // the keys that are looked at: span of them from k0 on
        u32 need = kq, count = 0, shift = 0, ready = 0;
        // a bin has copies, each in the next bank: additions to one word take turns, and where a few values hold most
        // of the interval they would all be to a few
        const u32 cs = 31u - (u32)__clz(kBins / wbins), copy = (u32)lane & ((1u << cs) - 1u);      // (2 to 8 copies)
        auto count_key = [&](u32 d) { atomicAdd(&hist[0][((d >> shift) << cs) | copy], 1u); };
        auto rows_of = [&](int p, auto ahead) {
          const int from = p * share, rows = tokens - from < share ? tokens - from : share;     // (none if negative)
          return RowVisitor<TX, NT, 4, decltype(ahead)::value>(Xb, ld, C, wa.L, order + (rows > 0 ? from : 0), rows);
        };
        u32* seg = shist + tid;                        // every NT-th word
        u32 listed_n = 0;                              // of this thread; more than kSeg: not all of them are listed
        bool known = false;                            // the range holds the rank, and `need` counts from k0
#pragma unroll 1
        for (int round = 0;; ++round) {
          // bins of 2^shift keys
          shift = span <= (u32)wbins ? 0u : (u32)(__clz(wbins) - __clz(span - 1u) + 1);
          const u32 bins = ((span - 1u) >> shift) + 1u;          // <= wbins
          u32* words = round == 1 ? gl : gh;
          ++events;
          for (bool more = true; more;) {
            for (int i = tid; i < kBins / 4; i += NT) reinterpret_cast<uint4*>(&hist[0][0])[i] = make_uint4(0, 0, 0, 0);
            if (tid == 0) s_below[0] = 0;
            __syncthreads();
            u32 below = 0, old = known ? 0u : listed_n;
            if (!known || listed_n > kSeg) {           // the share's keys in the range, or those of all shares again
              if (known) listed_n = 0;
#pragma unroll 1
              for (int e = known ? 0 : n_parts - 1; e < n_parts; ++e) {
                auto look = [&](TX x) {
                  const u32 key_x = Elem<TX>::key(x);
                  u32 d;
                  below += __builtin_sub_overflow(key_x, k0, &d) ? 1u : 0u;
                  if (d < span) {
                    if (__builtin_expect(listed_n < kSeg, 1)) seg[listed_n * NT] = key_x;
                    else count_key(d);
                    ++listed_n;
                  }
                };
                rows_of(s_parts[e], std::true_type()).visit([&](const uint4& p) {
                  TX x[V];
                  Elem<TX>::unpack(p, x);
#pragma unroll
                  for (int c = 0; c < V; ++c) look(x[c]);
                }, look);
              }
            }
#pragma unroll
            for (u32 i = 0; i < kSeg; ++i) {
              const u32 d = seg[i * NT] - k0;
              if (i >= old && i < listed_n && d < span) count_key(d);
            }
            below = group_sum_u32<64>(below);
            if (lane == 63 && below) atomicAdd(&s_below[0], below);
            // (the words were cleared by the statistics kernel, and from the third round on by the last to have read them)
            if (ready != 0 && !reached(kCtlReady, ready, wa.waits.limit)) return picks ? kAlone : kLeave;
            __syncthreads();
            for (int i = tid; i < (int)bins; i += NT) {
              u32 v = 0;
#pragma unroll
              for (int c = 0; c < 8; ++c) v += c < 1 << cs ? hist[0][((i << cs) + c) & (kBins - 1)] : 0u;
              if (v) atomicAdd(&words[i], v);
            }
            if (tid == 0 && !known && s_below[0]) atomicAdd(&ctl[kCtlBelow], s_below[0]);
            settle();
            if (tid == 0) (void)arrive(known ? n_parts : 1);
            more = false;
            if (!known && !reached(kCtlArrived, (u32)S, wa.waits.patience)) {
              if (tid == 0) s_parts[n_parts] = (unsigned short)min(atomicAdd(&ctl[kCtlClaimed], 1u), 0xFFFFu);
              __syncthreads();
              more = (int)s_parts[n_parts] < S;
              n_parts += more ? 1 : 0;
            }
          }
          if (!reached(kCtlArrived, (u32)S * events, wa.waits.limit)) return picks ? kAlone : kLeave;
          for (int i = tid; i < wbins; i += NT) hist[0][i] = i < (int)bins ? load(&words[i]) : 0u;
          if (tid == 0) s_below[0] = known ? 0u : load(&ctl[kCtlBelow]);
          __syncthreads();
          if (picks && !known && wave == NW - 1) finish_moments();
          if (wave == 0) {
            const u32 under = s_below[0];
            const BinPick p = pick_bin<false>(hist[0], wbins, under, need);
            Lost l = lost_rank<false>(need, nn, under, p.inside, k0, k0 + span);
            if (p.ok) {
              const u32 from_key = p.bin << shift, left = span - from_key;
              l.k0 = k0 + from_key;
              l.span = left < 1u << shift ? left : 1u << shift;
              l.rank = p.need;
            }
            if (lane == 0) {
              s_lost[0] = l;
              s_last = p.ok ? p.count : 0xFFFFFFFFu;   // (a set has fewer elements)
            }
          }
          __syncthreads();
          count = s_last;
          k0 = s_lost[0].k0;
          span = s_lost[0].span;
          need = (u32)s_lost[0].rank;
          __syncthreads();                             // (s_last and s_lost are written again below)
          if (count == 0xFFFFFFFFu) {
            if (span > 1u && tid == 0 && picks) atomicAdd(&status[1 + kPassZr], 1u);
            listed_n = kSeg + 1u;                      // other keys are wanted
          }
          known = true;
          if (span == 1u) {
            found = k0;
            return picks ? kProject : kLeave;
          }
          if (round > 0) {
            // the words are wanted again: the last to have read them clears them
            ++events;
            settle();
            if (known_to_all(&s_known, [&]() { return arrive(n_parts) == (u32)S * events; })) {
              for (int i = tid; i < W; i += NT) (void)atomicExch(&gh[i], 0u);
              settle();
              if (tid == 0) (void)atomicExch(&ctl[kCtlReady], events);
            }
            ready = events;
          }
          if (count <= keep) break;
        }
        // the bin's keys, `count` of them in all workgroups: one more than the key, so that a word that has none is 0
        if (ready != 0 && !reached(kCtlReady, ready, wa.waits.limit)) return picks ? kAlone : kLeave;
        u32* keys = s_search.h;
        if (tid == 0) s_below[0] = 0;
        __syncthreads();
        u32* const next = picks ? &s_below[0] : &ctl[kCtlListed];
        auto hand_over = [&](u32 to, u32 key_x) {      // (to < count <= keep)
          if (to >= keep) return;
          if (picks) keys[to] = key_x;
          else (void)atomicExch(&gl[to], key_x + 1u);
        };
        u32 hits = 0;                                  // which of those listed
        if (__builtin_expect(listed_n > kSeg, 0)) {    // (not all of this thread's were listed)
          auto look = [&](TX x) {
            const u32 key_x = Elem<TX>::key(x);
            if (key_x - k0 < span) hand_over(atomicAdd(next, 1u), key_x);
          };
#pragma unroll 1
          for (int e = 0; e < n_parts; ++e)
            rows_of(s_parts[e], std::false_type()).visit([&](const uint4& p) {
              TX x[V];
              Elem<TX>::unpack(p, x);
#pragma unroll
              for (int c = 0; c < V; ++c) look(x[c]);
            }, look);
        } else {
#pragma unroll
          for (u32 i = 0; i < kSeg; ++i) hits |= i < listed_n && seg[i * NT] - k0 < span ? 1u << i : 0u;
        }
        const u32 mine_n = (u32)__popc(hits), incl = wave_scan_u32(mine_n);
        const u32 wave_n = (u32)__builtin_amdgcn_readlane((int)incl, 63);
        if (wave_n != 0) {                             // (one addition a wavefront)
          u32 to = 0;
          if (lane == 63) to = atomicAdd(next, wave_n);
          to = (u32)__builtin_amdgcn_readlane((int)to, 63) + incl - mine_n;
#pragma unroll
          for (u32 i = 0; i < kSeg; ++i)
            if (hits >> i & 1u) hand_over(to++, seg[i * NT]);
        }
        if (!picks) return kLeave;
        if (tid == 0) s_last = 1u;
        __syncthreads();
        const u32 at = s_below[0] + (u32)tid;          // (no more than NT in all)
        if (at < count) {
          u32 v = 0;
          until(wa.waits.limit, [&]() { return (v = load(&gl[tid])) != 0u; });
          keys[at] = v - 1u;
          if (v == 0) s_last = 0u;
        }
        if (tid < 16) keys[count + (u32)tid] = 0xFFFFFFFFu;
        __syncthreads();
        if (s_last == 0) return kAlone;
        pick_listed(keys, count, need, &s_bin[0]);
        __syncthreads();
        found = s_bin[0];
        return kProject;
      };
      auto one_rank = [&](int q) -> bool {             // false: this workgroup has done its part
        const u32 kq = q == NR - 1 ? k[NR - 1] : k[0];
        if (q > 0) {                                   // (other readers of these have passed a barrier since)
          for (int i = tid; i < 2 << kSampleBits; i += NT) (&snext[0][0])[i] = 0;
          __syncthreads();
        }
        u32 first, last, drawn, shift = 0, below = 0;
        interval32(sample_rank(kq, nn, m, n_sel), first, last, drawn);
        if constexpr (MEET) {
          if (S > 1) {
            const auto what = shared_rank(kq, first, last);
            if (what != kAlone) return what == kProject;
            if (tid == 0) wa.ctl[(size_t)idx * kSetCtl + kCtlAlone] = 1u;
          }
        }
        shift = last < (u32)kBins ? 0u : (u32)(__clz(kBins) - __clz(last) + 1);         // bins of 2^shift keys
        for (int i = tid; i < kBins; i += NT) hist[0][i] = 0;
        if (tid == 0) s_below[0] = 0;
        __syncthreads();
        auto count = [&](TX x) {
          const u32 d = Elem<TX>::key(x) - first;      // (keys and first are below 2^31)
          below += d >> 31;
          if ((d >> shift) < (u32)kBins) atomicAdd(&hist[0][d >> shift], 1u);
        };
        RowVisitor<TX, NT, 4, true>(Xb, ld, C, wa.L, order, tokens)
            .visit([&](const uint4& p) {
                             TX x[V];
                             Elem<TX>::unpack(p, x);
#pragma unroll
                             for (int c = 0; c < V; ++c) count(x[c]);
                           },
                           count);
        below = group_sum_u32<64>(below);
        if (lane == 63 && below) atomicAdd(&s_below[0], below);
        __syncthreads();
        if (q == 0 && wave == NW - 1) finish_moments();
        if (wave == 0) {
          const BinPick p = pick_bin<false>(hist[0], kBins, s_below[0], kq);
          Lost l = lost_rank<false>(kq, nn, s_below[0], p.inside, first, first + ((u32)kBins << shift));
          bool miss = true;
          if (p.ok) {
            l.k0 = first + (p.bin << shift);
            l.span = 1u << shift;
            l.rank = p.need;
            miss = false;
          }
          if (lane == 0) {
            s_lost[0] = l;
            s_last = miss ? 1u : 0u;
          }
        }
        __syncthreads();
        const Lost l = s_lost[0];
        if (tid == 0 && s_last && l.span != 1u) atomicAdd(&status[1 + (q == NR - 1 ? kPassZr : kPassBase)], 1u);
        const u32 key_q = l.span == 1u ? l.k0 : search(l);
        if (q == NR - 1) found = key_q; else base_key = key_q;
        return true;
      };
      // (no loop for one rank: what does not change in it would be computed before it and spilled)
      if constexpr (NR == 1) {
        if (!one_rank(0)) return;                      // the same for every thread
      } else {
#pragma unroll 1
        for (int q = 0; q < NR; ++q) one_rank(q);
      }
    }
    if (tid == 0) {
      w.sigma = s_sigma;
      w.c_base = NR == 2 ? Elem<TX>::key_to_float(base_key) : s_cbase;       // (the base radius Q_p(|x|))
      project_store(idx, w, found, F16, sc, wa.clip, wa.scale, wa.stats);
    }
    return;
  }
  const SampleRank sr = sample_rank(k_pass, nn, m, n_sel);
  const float mf = (float)m;
  Bracket e;
  e.below = 0;
  e.width = (u32)Wfew;
  e.shift = 0;
  if constexpr (F16) {
    const u32* const hs[1] = {shist};
    const u32 rs[1] = {sr.rk};
    find_ranks<NT, 1, 1, true>(hs, rs, stot, s_bin, s_before, cum, m);
    __syncthreads();
    if (wave == NW - 1) finish_moments();
    if (wave != 0) return;
    place_bins(cum, (int)s_bin[0], sr, m, Wfew, W, e.lo, e.width);
    for (int i = Wfew + lane; i < (int)e.width; i += 64) bhist[(size_t)idx * W + i] = 0;
  } else {
    // in W bins of 2^shift keys: a bin then holds about 2e-4 of the set's elements whatever the data's
    // offset and spread
    u32 last, drawn;
    interval32(sr, e.lo, last, drawn);
    while ((((unsigned long long)(u32)W << e.shift) - 1ull) < last) ++e.shift;
    // But it may also reach from the smallest key to a normal value, where the rank lies just
    // above the zeros of an activation, or hold a few values within 1e-5 of each other, and a bin
    // must not hold more keys than the second sweep can collect.  So the sample is counted in 64
    // (32) cells, as far as the interval must reach, and where one of them has more than that, a
    // cell is cut into as many bins as the sample's share of it: bins of equal mass, nearly.
    // (Bins of equal width collected up to 13 000 keys with 15 % zeros: [8, 1024, 768] with 16 sets
    // calibrated in 290 us, 62 so; without gaps 45, and 53 so, 60 if every interval is cut.)
    u32* head = lists + (size_t)idx * cap;
    if (tid < kListHead) head[tid] = tid == kHeadTie || tid == kHeadTieBin ? kNoKey : 0u;
    const float enough = (float)(cap - kListHead - cells) * mf / (float)n;     // sampled keys
    if (e.shift == 0 || (float)drawn <= enough) {        // the same for every thread
      if (tid == 0) br[idx] = e;
      return;
    }
    const u32 cshift = e.shift + (u32)__clz(cells) - (u32)__clz(W);
#pragma unroll
    for (int i = 0; i < kKeys; ++i) {
      if (i / V < steps) {
        const u32 d = key[i] - e.lo;
        if (key[i] != kDead && d <= last) atomicAdd(&s_cell[1 + (d >> cshift)], 1u);
      }
    }
    __syncthreads();
    u32 mine = lane < cells ? s_cell[1 + lane] : 0u;
    const u32 most = (u32)__builtin_amdgcn_readlane((int)group_max_u32<64>((mine << 6) | (u32)lane), 63);
    if ((float)(most >> 6) <= enough) {
      if (tid == 0) br[idx] = e;
      return;
    }
    e.width = last + 1u;                               // (no further than that)
    e.shift = cshift;
    // That cell may hold ties, which could be more than a list holds, with other values in the
    // same bin: the key that the sample holds most often there (of those that share its hash) is
    // counted by itself.
    u32 tie = kNoKey;
    {
      constexpr int kHash = 2048;
      const u32 heavy = most & 63u;
      for (int i = tid; i < kHash; i += NT) shist[i] = 0;
      __syncthreads();
      auto in_heavy = [&](u32 k) { return k != kDead && k - e.lo <= last && (k - e.lo) >> cshift == heavy; };
      auto hash = [&](u32 k) { return (k * 2654435761u) >> 21; };
#pragma unroll
      for (int i = 0; i < kKeys; ++i)
        if (i / V < steps && in_heavy(key[i])) atomicAdd(&shist[hash(key[i])], 1u);
      __syncthreads();
      u32 best = 0;
      for (int i = tid; i < kHash; i += NT) {
        const u32 c = (shist[i] << 11) | (u32)i;       // (at most 2^14 sampled keys)
        best = c > best ? c : best;
      }
      best = group_max_u32<64>(best);
      if (lane == 63) atomicMax(&s_mode, best);
      __syncthreads();
      const u32 often = s_mode >> 11;
#pragma unroll
      for (int i = 0; i < kKeys; ++i)
        if (i / V < steps && in_heavy(key[i]) && hash(key[i]) == (s_mode & (kHash - 1))) s_tie = key[i];   // any of them
      __syncthreads();
      if (often >= 4u) {
        tie = s_tie;
        if (lane == (int)heavy) mine -= often;
      }
    }
    if (wave != 0) return;
    // bins of a cell: one, and its share of the others by the sampled keys in it, or the average
    // with its neighbours if that is more (the density is smooth more often than the sample is)
    const u32 around = ((lane > 0 ? s_cell[lane] : 0u) + mine + (lane + 1 < cells ? s_cell[2 + lane] : 0u) + 2u) / 3u;
    u32 parts = lane < cells ? (mine > around ? mine : around) : 0u;
    u32 total = xor_reduce_sum<64, u32>(parts);
    total = total > 0u ? total : 1u;
    parts = lane < cells ? 1u + parts * (u32)(W - cells) / total : 0u;
    const u32 incl = wave_scan_u32(parts);
    const u32 cell = (incl - parts) | (parts << 16);
    if (lane < cells) head[kListHead + lane] = cell;
    const u32 at = tie != kNoKey ? tie - e.lo : 0u;
    const u32 tie_bin = bin_of(at, e.shift, (u32)__shfl((int)cell, (int)(at >> e.shift), 64));
    if (lane == 0 && tie != kNoKey) {
      head[kHeadTie] = tie;
      head[kHeadTieBin] = tie_bin;
    }
    e.shift |= kCells;
  }
  if (tid == 0) br[idx] = e;
}

template <typename TX>
static void sets_t(const TX* X, int B, int T, int C, long long ld, int G, int Wfew, int W, int cells,
                   const float* r,
                   const double* mean, const double* m2, int* gid, const Scalars& sc, int pass,
                   bool keep_base, GroupWork* grp, Bracket* br, unsigned* bhist, unsigned* lists,
                   int cap, unsigned* img_flag, unsigned* status, hipStream_t st) {
  constexpr int V = Elem<TX>::V;
  const int aligned = ((reinterpret_cast<uintptr_t>(X) & 15) == 0 && ld % V == 0 && C % V == 0) ? 1 : 0;
  // 8 Ki sampled elements are enough (binary32: a wider interval costs little), or the image is no
  // larger.  17 to 32 sets have no wider interval to fall back on: from 64 Ki elements a set on, where a
  // missed set's search costs most, they draw 16 Ki.  [32, 4096, 1024], 32 sets: 111.8 -> 116.0 us, but
  // after a GELU 140 -> 115, clamped to [0, 6] (16 % zeros, five missed sets of 0.1 M to 4 M elements, then
  // none) 1165 -> 110, with 15 % zeros 226 -> 194.
  const bool few = (Wfew >= 512 && G >= 8 && pass == kPassZr && (W > Wfew || (long long)T * C <= 65536ll * G)) ||
                   (long long)T * C <= 8192;
  const size_t order_bytes = T <= kListTokens ? (size_t)T * sizeof(unsigned short) : 0;
#define TDQ_SETS_SM(NT, RD, SM)                                                                        \
  hipLaunchKernelGGL((k_sets<TX, NT, RD, SM, 0>), dim3(G, B), dim3(NT), order_bytes, st, X, ld, T, C, G, Wfew, W, cells, aligned, r, \
                     mean, m2, gid, sc, pass, keep_base ? 1 : 0, grp, br, bhist, lists, cap,       \
                     img_flag, status, WholeArgs())
#define TDQ_SETS(NT, RD)                                                       \
  do {                                                                         \
    if constexpr (sizeof(TX) == 4) TDQ_SETS_SM(NT, RD, 8192);                  \
    else if (few) TDQ_SETS_SM(NT, RD, 8192);                                   \
    else TDQ_SETS_SM(NT, RD, 16384);                                           \
  } while (0)
  // as few threads as hold the image's range keys in registers: [32, 4096, 1024] calibrates
  // in 111 / 117 / 145 us with 256 / 512 / 1024 threads per set
  // ... but with no more sets than CUs twice the wavefronts: the layer of [8, 1024, 768] binary32, 16 sets,
  // 67.6 -> 64.1, [1, 1782, 56] 32 sets 48.2 -> 44.6, binary16 [6, 2080, 1376] 32 sets with a percentile 88.1 -> 83.0
  if ((long long)B * G <= 256 && T <= 1024)
    TDQ_SETS(512, 2);
  else if ((long long)B * G <= 256 && T <= 4096)
    TDQ_SETS(512, 8);
  else if (T <= 1024)
    TDQ_SETS(256, 4);
  else if (T <= kIdRounds * 256)
    TDQ_SETS(256, 16);
  else if (T <= kIdRounds * 512)
    TDQ_SETS(512, 16);
  else
    TDQ_SETS(1024, 16);
#undef TDQ_SETS
#undef TDQ_SETS_SM
}

hipError_t launch_sets(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                       int Wfew, int W, int cells, const float* r, const double* mean, const double* m2, int* gid,
                       const Scalars& sc, int pass, bool keep_base, GroupWork* grp, Bracket* br,
                       unsigned* bhist, unsigned* lists, int cap, unsigned* img_flag,
                       unsigned* status, hipStream_t st) {
  if (dt == TDQ_F16)
    sets_t<u16>(static_cast<const u16*>(X), B, T, C, ld, G, Wfew, W, cells, r, mean, m2, gid, sc, pass, keep_base,
                grp, br, bhist, lists, cap, img_flag, status, st);
  else
    sets_t<float>(static_cast<const float*>(X), B, T, C, ld, G, Wfew, W, cells, r, mean, m2, gid, sc, pass, keep_base,
                  grp, br, bhist, lists, cap, img_flag, status, st);
  return hipGetLastError();
}

template <typename TX, int WHOLE, bool MEET = false>
static void sets_whole_t(const TX* X, int B, int T, int C, long long ld, int G, int extra, int Wfew, int W,
                         const float* r, const double* mean, const double* m2, int* gid, const Scalars& sc,
                         unsigned* bhist, void* ctl, unsigned* img_flag, unsigned* status, float* clip,
                         float* scale, tdq_group_stats* stats, const Waits& waits, hipStream_t st) {
  constexpr int V = Elem<TX>::V;
  const int aligned = ((reinterpret_cast<uintptr_t>(X) & 15) == 0 && ld % V == 0 && C % V == 0) ? 1 : 0;
  WholeArgs wa;
  wa.extra = extra;
  wa.L = sweep_lanes_per_row(C, V);
  // binary32: more than a wavefront to a row as long as it has more than four pieces a lane and a workgroup's share
  // (about T / (G + extra) rows) leaves lanes without a row.  Calibration by the chain, with 64 lanes and so, us: [9, 20,
  // 16044] with 4 sets, values near 1, 79.9 / 126 / 55.5, [5, 3, 92859] with 2, clamped, 389 / 599 / 289, [3, 104, 8422]
  // with 5, a fifth masked, 65.7 / 86.3 / 55.3; 106 random calls of few rows 1.24 and 1.87 times as fast as the chain
  // in the geometric mean, 90 with extra = 0 1.33 times as fast as with 64 lanes, none slower.
  if (V == 4)
    while (wa.L < 512 && C / V > 4 * wa.L && (long long)T * wa.L < 512ll * (G + extra)) wa.L *= 2;
  wa.ctl = static_cast<u32*>(ctl);
  wa.clip = clip;
  wa.scale = scale;
  wa.stats = stats;
  wa.waits = waits;
  const size_t order_bytes = ((size_t)T * sizeof(unsigned short) + 15) & ~(size_t)15;
#define TDQ_WHOLE_RD(RD, SM)                                                                            \
  hipLaunchKernelGGL((k_sets<TX, 512, RD, SM, WHOLE, MEET>), dim3(G + extra, B), dim3(512), order_bytes, st, X, ld, T, \
                     C, G, Wfew, W, 0, aligned, r, mean, m2, gid, sc, kPassZr, 0, nullptr, nullptr, bhist, nullptr, \
                     0, img_flag, status, wa)
#define TDQ_WHOLE(SM)                                                            \
  do {                                                                           \
    if (T <= 512) TDQ_WHOLE_RD(1, SM);                                           \
    else if (T <= 1024) TDQ_WHOLE_RD(2, SM);                                     \
    else if (T <= 2048) TDQ_WHOLE_RD(4, SM);                                     \
    else if (T <= 4096) TDQ_WHOLE_RD(8, SM);                                     \
    else TDQ_WHOLE_RD(16, SM);                                                   \
  } while (0)
  static_assert(kWholeTokens == 512 * kIdRounds, "a thread holds its range keys in registers");
  // (16 Ki sampled elements: with 8 Ki a set of [2, 1024, 768], 16 sets, values clamped to [0, 6], missed its rank)
  if constexpr (sizeof(TX) == 4) TDQ_WHOLE(8192);
  else TDQ_WHOLE(16384);
#undef TDQ_WHOLE
#undef TDQ_WHOLE_RD
}

hipError_t launch_sets_whole(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G, int ranks,
                             int extra, int Wfew, int W, const float* r, const double* mean, const double* m2,
                             int* gid, const Scalars& sc, unsigned* bhist, void* ctl, unsigned* img_flag,
                             unsigned* status, float* clip, float* scale, tdq_group_stats* stats,
                             const Waits& waits, hipStream_t st) {
#define TDQ_SW(TX, ...)                                                                                      \
  sets_whole_t<TX, __VA_ARGS__>(static_cast<const TX*>(X), B, T, C, ld, G, extra, Wfew, W, r, mean, m2, gid, sc, bhist, \
                       ctl, img_flag, status, clip, scale, stats, waits, st)
  if (dt == TDQ_F16) {
    if (ranks == 1) TDQ_SW(u16, 1); else TDQ_SW(u16, 2);
  } else {
    if (ranks == 2) TDQ_SW(float, 2);
    else if (extra > 0) TDQ_SW(float, 1, true);
    else TDQ_SW(float, 1);
  }
#undef TDQ_SW
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// k_bracket_hist: the one sweep
// ---------------------------------------------------------------------------
// A group of L lanes takes R rows at a time and P pieces of 16 bytes of each: the set ids
// and all R P = 4 pieces are loaded before the first is looked at, so a wavefront has four
// kilobytes in flight whatever the row length -- what bounds this sweep otherwise is the
// chain set id -> interval -> piece of one row after another.  Measured, this kernel alone:
// [8, 7744, 512] 25.6 -> 17.1 us, [32, 4096, 1024] 52.1 -> 46.5 (5.8 TB/s), [16, 484, 320]
// 13.4 -> 6.1, [5, 1369, 333] (rows at odd addresses, read element by element before) 20.7 ->
// 7.5; without the in-loop histogram additions it takes the same time, without the final
// global additions 13.2 and 44.6 us on the first two.
template <typename TX, int L, int P>
__global__ __launch_bounds__(kSweepThreads) void k_bracket_hist(
    const TX* __restrict__ X, long long ld, int T_, int C, int G, int W, int lw, int cells,
    const int* __restrict__ gid, Bracket* __restrict__ br, u32* __restrict__ bhist,
    u32* __restrict__ lists, int cap, int rows_per_block) {
  constexpr int R = 4 / P;
  constexpr int V = Elem<TX>::V;
  // [G][W] bins, binary32: [G][cells] cells, then per set: below, lo, width (with cells: in keys),
  // binary32: shift, tie, ties
  extern __shared__ __attribute__((aligned(16))) u32 lds[];
  // walks X backwards: it runs right after the forward statistics sweep, so the end of
  // X is what the last-level cache still holds
  const int b = (int)(gridDim.y - 1 - blockIdx.y);
  const int chunk = (int)(gridDim.x - 1 - blockIdx.x);
  const int tid = threadIdx.x;
  const int nwords = G * W;
  u32* s_cells = lds + nwords;
  u32* s_below = s_cells + (V == 4 ? G * cells : 0);
  u32* s_lo = s_below + G;
  u32* s_width = s_lo + G;
  u32* s_shift = s_width + G;
  u32* s_tie = s_shift + G;
  u32* s_ties = s_tie + G;
  // most sets use the first 2^lw bins; the further ones of those that use more are cleared and
  // added one by one
  if constexpr (V == 8) {
    for (int i = tid; i < (G << lw) / 4; i += kSweepThreads) {
      const int g = i >> (lw - 2), at = i - (g << (lw - 2));
      *reinterpret_cast<uint4*>(&lds[g * W + 4 * at]) = make_uint4(0, 0, 0, 0);
    }
  } else {
    for (int i = tid; i < nwords / 4; i += kSweepThreads)
      reinterpret_cast<uint4*>(lds)[i] = make_uint4(0, 0, 0, 0);
    for (int i = tid; i < G * cells; i += kSweepThreads) {
      const int g = i / cells;
      s_cells[i] = lists[((size_t)b * G + g) * cap + kListHead + (i - g * cells)];
    }
  }
  for (int g = tid; g < G; g += kSweepThreads) {
    const Bracket e = br[(long long)b * G + g];
    s_below[g] = 0;
    s_lo[g] = e.lo;
    s_width[g] = e.width;
    if constexpr (V == 4) {
      s_shift[g] = e.shift;
      s_tie[g] = lists[((size_t)b * G + g) * cap + kHeadTie];
      s_ties[g] = 0;
    }
  }
  __syncthreads();
  const int lane = tid & 63;                      // (G <= 64)
  const bool wide = V == 8 && W > 1 << lw && __ballot(lane < G && (int)s_width[lane < G ? lane : 0] > 1 << lw) != 0;
  if (wide) {                                     // the same in every wavefront
    for (int g = 0; g < G; ++g)
      for (int i = (1 << lw) + tid; i < (int)s_width[g]; i += kSweepThreads) lds[g * W + i] = 0;
    __syncthreads();
  }

  const int row0 = chunk * rows_per_block;
  int nrows = T_ - row0;
  nrows = nrows < rows_per_block ? nrows : rows_per_block;
  constexpr int SLOTS = kSweepThreads / L;
  const int slot = tid / L, lr = tid % L;
  const int nvec = C / V;
  const long long first = (long long)b * T_ + row0;
  for (int rr = slot; rr < nrows; rr += SLOTS * R) {
    const TX* xp[R];
    int g[R];
    u32 below[R], ties[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {                 // rows past the end: the last one, not counted
      const int ri = rr + SLOTS * i;
      const long long row = first + (ri < nrows ? ri : nrows - 1);
      xp[i] = X + row * ld;
      g[i] = gid[row];
      below[i] = 0;
      ties[i] = 0;
    }
    // binary32: keys and lo are below 2^31, the sign of the difference says "key < lo", and such a
    // difference lies past the last bin (the number of bins is a power of two and bins << shift at
    // most 2^31, so 2^31 >> shift is at least their number) and past the last cell.  The cells of
    // several keys are read before the first is used, of those outside the interval as well: one
    // trip to LDS.
    auto count32 = [&](const auto& k, int i, u32 lo, u32 width, u32 shift) {
      constexpr int N = sizeof(k) / sizeof(u32);
      if (!(shift & kCells)) {
#pragma unroll
        for (int c = 0; c < N; ++c) {
          const u32 d = k[c] - lo, bin = d >> shift;
          below[i] += d >> 31;
          if (bin < width) atomicAdd(&lds[g[i] * W + bin], 1u);
        }
      } else {
        const u32 sh = shift & 63u, tie = s_tie[g[i]];
        u32 d[N], cell[N];
#pragma unroll
        for (int c = 0; c < N; ++c) {
          d[c] = k[c] - lo;
          below[i] += d[c] >> 31;
          ties[i] += k[c] == tie ? 1u : 0u;
          d[c] = k[c] != tie ? d[c] : 0xFFFFFFFFu;
          cell[c] = s_cells[g[i] * cells + (int)(d[c] < width ? d[c] >> sh : 0u)];
        }
#pragma unroll
        for (int c = 0; c < N; ++c)
          if (d[c] < width) atomicAdd(&lds[g[i] * W + bin_of(d[c], sh, cell[c])], 1u);
      }
    };
    for (int v0 = lr; v0 < nvec; v0 += P * L) {
      uint4 q[R][P];
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int k = 0; k < P; ++k) {
          const int v = v0 + k * L;
          q[i][k] = load16(xp[i] + (long long)(v < nvec ? v : v0) * V);
        }
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const u32 lo = s_lo[g[i]], width = s_width[g[i]];
        const u32 shift = V == 4 ? s_shift[g[i]] : 0u;
        const u32 lo2 = lo | (lo << 16);
        u32* h = lds + g[i] * W;
        if (rr + SLOTS * i < nrows) {
#pragma unroll
          for (int k = 0; k < P; ++k) {
            if (k > 0 && v0 + k * L >= nvec) break;
            const u32 wd[4] = {q[i][k].x, q[i][k].y, q[i][k].z, q[i][k].w};
            if constexpr (V == 4) {
              const u32 key[4] = {wd[0] & 0x7FFFFFFFu, wd[1] & 0x7FFFFFFFu, wd[2] & 0x7FFFFFFFu, wd[3] & 0x7FFFFFFFu};
              count32(key, i, lo, width, shift);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if constexpr (V == 8) {
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
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (rr + SLOTS * i < nrows) {
        const u32 lo = s_lo[g[i]], width = s_width[g[i]];
        for (int c = nvec * V + lr; c < C; c += L) {          // fewer than V elements
          const u32 k = Elem<TX>::key(xp[i][c]);
          if constexpr (V == 8) {
            below[i] += k < lo ? 1u : 0u;
            if (k >= lo && k - lo < width) atomicAdd(&lds[g[i] * W + (k - lo)], 1u);
          } else {
            const u32 key[1] = {k};
            count32(key, i, lo, width, s_shift[g[i]]);
          }
        }
      }
      if constexpr (V == 4) {
        if (__ballot(ties[i] != 0) != 0) {
          const u32 n = group_sum_u32<L>(ties[i]);            // (rows past the end: none)
          if (lr == L - 1 && n && rr + SLOTS * i < nrows) atomicAdd(&s_ties[g[i]], n);
        }
      }
      const u32 total = group_sum_u32<L>(below[i]);           // in the row's last lane
      if (lr == L - 1 && total) atomicAdd(&s_below[g[i]], total);
    }
  }
  __syncthreads();
  u32* gh = bhist + (size_t)b * G * W;
  for (int i = tid; i < (V == 8 ? G << lw : nwords); i += kSweepThreads) {
    const int g = i >> lw, at = V == 8 ? g * W + i - (g << lw) : i;
    const u32 v = lds[at];
    if (v) atomicAdd(&gh[at], v);
  }
  if (wide)
    for (int g = 0; g < G; ++g)
      for (int i = (1 << lw) + tid; i < (int)s_width[g]; i += kSweepThreads) {
        const u32 v = lds[g * W + i];
        if (v) atomicAdd(&gh[g * W + i], v);
      }
  for (int g = tid; g < G; g += kSweepThreads) {
    const u32 v = s_below[g];
    if (v) atomicAdd(&br[(long long)b * G + g].below, v);
    if constexpr (V == 4)
      if (s_ties[g]) atomicAdd(&lists[((size_t)b * G + g) * cap + kHeadTies], s_ties[g]);
  }
}

// Rows per workgroup of a sweep.
// Two workgroups per CU where that leaves each 128 Ki elements, one otherwise, and at least
// 32 Ki elements each: every workgroup clears G W bins and adds the non-zero ones to the
// image's with global atomics, which is what more workgroups cost.  Calibration of
// [8, 7744, 512] with 512 / 256 workgroups 47.3 / 44.5 us, of [32, 4096, 1024] 106.6 /
// 107.5; of [8, 1936, 320] with at least 32 / 16 / 8 Ki elements 40.5 / 41.9 / 44.1 us, of
// [8, 121, 512] 19.3 / 18.9 / 19.0 (64 Ki: 21.5).
static int sweep_rows(int B, int T, int C) {
  const long long rows_min = (32768 + C - 1) / C;
  long long target_blocks = ((long long)B * T * C >= 512ll * 131072 ? 512 : 256) / B;
  if (target_blocks < 1) target_blocks = 1;
  long long rpb = (T + target_blocks - 1) / target_blocks;
  if (rpb < rows_min) rpb = rows_min;
  return (int)(rpb > T ? T : rpb);
}

// The (L, P) of a sweep over rows of nvec pieces (see k_bracket_hist).
#define TDQ_SWEEP_CASES(CASE)                                                             \
  CASE(1, 1) CASE(2, 1) CASE(4, 1) CASE(8, 1) CASE(8, 2) CASE(8, 4) CASE(16, 2) CASE(16, 4) \
  CASE(32, 2) CASE(32, 4) CASE(64, 2) CASE(64, 4)

template <typename TX>
static void bracket_hist_t(const TX* X, int B, int T_, int C, long long ld, int G, int Wfew, int W,
                           int cells, unsigned* lists, int cap, const int* gid, Bracket* br, unsigned* bhist, hipStream_t st) {
  const int nvec = C / Elem<TX>::V;
  const int L = sweep_lanes_per_row(C, Elem<TX>::V);
  const int P = nvec > 2 * L ? 4 : nvec > L ? 2 : 1;
  const int rpb = sweep_rows(B, T_, C);
  const unsigned chunks = (unsigned)((T_ + rpb - 1) / rpb);
  const size_t lds_bytes =
      (size_t)G * (sizeof(TX) == 2 ? W + 3 : W + cells + 6) * sizeof(u32);
  int lw = 0;
  while (1 << lw < Wfew) ++lw;
#define TDQ_BH(LL, PP)                                                                          \
  if (L == LL && P == PP) {                                                                     \
    if (lds_bytes > 65536)                                                                      \
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bracket_hist<TX, LL, PP>),     \
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);    \
    hipLaunchKernelGGL((k_bracket_hist<TX, LL, PP>), dim3(chunks, B), dim3(kSweepThreads),      \
                       lds_bytes, st, X, ld, T_, C, G, W, lw, cells, gid, br, bhist, lists, cap, rpb);                 \
  }
  TDQ_SWEEP_CASES(TDQ_BH)
#undef TDQ_BH
}

hipError_t launch_bracket_hist(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                               int Wfew, int W, int cells, unsigned* lists, int cap, const int* gid,
                               Bracket* br, unsigned* bhist, hipStream_t st) {
  if (dt == TDQ_F16)
    bracket_hist_t<u16>(static_cast<const u16*>(X), B, T, C, ld, G, Wfew, W, cells, lists, cap, gid, br, bhist, st);
  else
    bracket_hist_t<float>(static_cast<const float*>(X), B, T, C, ld, G, Wfew, W, cells, lists, cap, gid, br, bhist, st);
  return hipGetLastError();
}

// First key and number of keys of a bin (binary32), by one wavefront; cell = the set's cell of this
// lane.
__device__ __forceinline__ void bin_keys(u32 cell, int cells, const Bracket& e, u32 bin, u32& key0, u32& span) {
  if (!(e.shift & kCells)) {
    key0 = e.lo + (bin << e.shift);
    span = 1u << e.shift;
    return;
  }
  const int lane = threadIdx.x & 63;
  const u32 shift = e.shift & 63u;
  const int c = (int)__popcll(__ballot(lane < cells && (cell & 0xFFFFu) <= bin)) - 1;
  const u32 its = (u32)__shfl((int)cell, c > 0 ? c : 0, 64), part = bin - (its & 0xFFFFu);
  // part j of m starts at the first fraction f of the cell with f m >= j 2^shift (exact: below 2^53)
  const double m = (double)(its >> 16);
  const u32 from = (u32)ceil((double)((unsigned long long)part << shift) / m);
  const u32 left = e.width - ((u32)c << shift);            // keys of the interval from the cell on
  u32 to = (u32)ceil((double)((unsigned long long)(part + 1u) << shift) / m);
  to = to < left ? to : left;
  key0 = e.lo + ((u32)c << shift) + from;
  span = to - from;
}

// ---------------------------------------------------------------------------
// k_bracket_gather, binary32 input only: a second sweep collects the keys that fall into the bin
// of every set that holds the rank (about 2e-4 of the elements), first per workgroup in LDS, and
// once that is full one by one.  Their number, known from the first sweep, is counted in
// GroupWork::prefix as they are added.  A bin with more keys than a list holds is not collected;
// if they all are equal, its smallest and largest key say so.  Every workgroup finds the bins
// itself.  Calibration of [8, 1024, 768]: 73.4 us with a sweep and a select kernel per eight key
// bits, 45.3 with the sampled interval (this kernel 11.5, with twice or four times the workgroups
// 11.0 and 16.8).
// ---------------------------------------------------------------------------
constexpr int kGatherWords = 8192;              // LDS words for collected keys, shared by the sets

template <int L, int P>
__global__ __launch_bounds__(kSweepThreads) void k_bracket_gather(
    const float* __restrict__ X, long long ld, int T_, int C, int G, int W, int cells,
    const int* __restrict__ gid, const Bracket* __restrict__ br, const u32* __restrict__ bhist,
    GroupWork* __restrict__ grp, u32* __restrict__ lists, int cap, int rows_per_block) {
  constexpr int R = 4 / P;
  __shared__ u32 s_key0[64], s_span[64], s_cnt[64], s_nmin[64], s_max[64], s_at[64], s_tie[64], s_take[64];
  __shared__ u32 s_list[kGatherWords];
  const int b = blockIdx.y, chunk = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int keep = kGatherWords / G;            // keys kept per set (G <= 64)
  const int keys_at = kListHead + cells, keys_cap = cap - keys_at;
  for (int g = tid >> 6; g < G; g += kSweepThreads / 64) {
    const long long idx = (long long)b * G + g;
    const GroupWork w = grp[idx];
    const Bracket e = br[idx];
    u32* head = lists + (size_t)idx * cap;
    const u32 tie = head[kHeadTie], ties = head[kHeadTies], tie_bin = head[kHeadTieBin];
    const u32 cell = head[kListHead + (lane < cells ? lane : 0)];
    u32 span = 0, key0 = 0, take = 0;
    if (w.tokens != 0) {                        // uniform over the wavefront
      const BinPick p = pick_bin<true>(bhist + (size_t)idx * W, W, e.below, (u32)w.k_rem, tie_bin, ties);
      if (p.ok && p.count != 0) {               // (a bin of ties alone needs no sweep)
        bin_keys(cell, cells, e, p.bin, key0, span);
        take = p.count <= (u32)keys_cap ? 1u : 0u;
        if (span == 1u) {                       // one key: that is the answer
          span = 0;
          if (chunk == 0 && lane == 0) {
            head[kHeadMin] = ~key0;
            head[kHeadMax] = key0;
          }
        }
      }
    }
    if (lane == 0) {
      s_key0[g] = key0;
      s_span[g] = span;
      s_cnt[g] = 0;
      s_nmin[g] = 0;
      s_max[g] = 0;
      s_tie[g] = tie;
      s_take[g] = take;
    }
  }
  __syncthreads();
  const int row0 = chunk * rows_per_block;
  int nrows = T_ - row0;
  nrows = nrows < rows_per_block ? nrows : rows_per_block;
  constexpr int SLOTS = kSweepThreads / L;
  const int slot = tid / L, lr = tid % L;
  const int nvec = C / 4;
  const long long first = (long long)b * T_ + row0;
  for (int rr = slot; rr < nrows; rr += SLOTS * R) {
    const float* xp[R];
    int g[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {               // rows past the end: the last one, not looked at
      const int ri = rr + SLOTS * i;
      const long long row = first + (ri < nrows ? ri : nrows - 1);
      xp[i] = X + row * ld;
      g[i] = gid[row];
    }
    auto look = [&](int gi, u32 key0, u32 span, u32 k) {
      if (k - key0 < span && k != s_tie[gi]) {
        if (~k > s_nmin[gi]) atomicMax(&s_nmin[gi], ~k);
        if (k > s_max[gi]) atomicMax(&s_max[gi], k);
        if (s_take[gi]) {
          const u32 at = atomicAdd(&s_cnt[gi], 1u);
          if (at < (u32)keep) {
            s_list[gi * keep + at] = k;
          } else {
            const long long idx = (long long)b * G + gi;
            const u32 to = atomicAdd(&grp[idx].prefix, 1u);
            if (to < (u32)keys_cap) lists[idx * cap + keys_at + to] = k;
          }
        }
      }
    };
    for (int v0 = lr; v0 < nvec; v0 += P * L) {
      uint4 q[R][P];
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int k = 0; k < P; ++k) {
          const int v = v0 + k * L;
          q[i][k] = load16(xp[i] + (long long)(v < nvec ? v : v0) * 4);
        }
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const u32 key0 = s_key0[g[i]], span = rr + SLOTS * i < nrows ? s_span[g[i]] : 0u;
#pragma unroll
        for (int k = 0; k < P; ++k) {
          if (k > 0 && v0 + k * L >= nvec) break;
          look(g[i], key0, span, q[i][k].x & 0x7FFFFFFFu);
          look(g[i], key0, span, q[i][k].y & 0x7FFFFFFFu);
          look(g[i], key0, span, q[i][k].z & 0x7FFFFFFFu);
          look(g[i], key0, span, q[i][k].w & 0x7FFFFFFFu);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (rr + SLOTS * i < nrows)
        for (int c = nvec * 4 + lr; c < C; c += L)
          look(g[i], s_key0[g[i]], s_span[g[i]], Elem<float>::key(xp[i][c]));
    }
  }
  __syncthreads();
  if (tid < G && s_max[tid]) {                  // (keys are at least 1)
    const long long idx = (long long)b * G + tid;
    const u32 n = s_cnt[tid] < (u32)keep ? s_cnt[tid] : (u32)keep;
    s_cnt[tid] = n;
    s_at[tid] = n ? atomicAdd(&grp[idx].prefix, n) : 0u;
    atomicMax(&lists[idx * cap + kHeadMin], s_nmin[tid]);
    atomicMax(&lists[idx * cap + kHeadMax], s_max[tid]);
  }
  __syncthreads();
  for (int i = tid; i < G * keep; i += kSweepThreads) {
    const int g = i / keep, at = i - g * keep;
    if ((u32)at < s_cnt[g] && s_at[g] + (u32)at < (u32)keys_cap)
      lists[((long long)b * G + g) * cap + keys_at + s_at[g] + at] = s_list[i];
  }
}

hipError_t launch_bracket_gather(const void* Xv, int B, int T_, int C, long long ld, int G, int W,
                                 int cells, const int* gid, const Bracket* br, const unsigned* bhist,
                                 GroupWork* grp, unsigned* lists, int cap, hipStream_t st) {
  const float* X = static_cast<const float*>(Xv);
  const int nvec = C / 4;
  const int L = sweep_lanes_per_row(C, 4);
  const int P = nvec > 2 * L ? 4 : nvec > L ? 2 : 1;
  const int rpb = sweep_rows(B, T_, C);
  const unsigned chunks = (unsigned)((T_ + rpb - 1) / rpb);
#define TDQ_BG(LL, PP)                                                                             \
  if (L == LL && P == PP)                                                                          \
    hipLaunchKernelGGL((k_bracket_gather<LL, PP>), dim3(chunks, B), dim3(kSweepThreads), 0, st, X, \
                       ld, T_, C, G, W, cells, gid, br, bhist, grp, lists, cap, rpb);
  TDQ_SWEEP_CASES(TDQ_BG)
#undef TDQ_BG
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// k_bracket_finish: one workgroup per set.  Its first wavefront verifies the interval and
// finds the bin; that is the key itself (binary16, one key per bin), or the workgroup finds
// it among the keys that the second sweep collected (binary32).  A chain of dependent trips to
// memory: the record, the interval and the bins are loaded together.
//
// On a miss, or if more keys were collected than fit, the workgroup searches the set's own rows
// for the key, only on the side of the interval (or in the bin) where it must lie: an LDS
// histogram of that range over 2048 bins, then of the bin, until a bin is one key.  One
// workgroup on one CU: bound by the loads it keeps in flight, so the ids of 2048 tokens are read
// together, a lane takes four pieces of 16 bytes at a time, and with few sets per call, which may
// be large, a workgroup has 1024 threads.  A binary16 rank that misses its one-key bins often lies close
// to them, so the first pass looks at the 2046 keys next to the interval one by one.  What a miss
// cost before (eight key bits a pass) was LDS additions that met in one word: nearly all elements
// lie on one side of the interval.  Calibration with 18 % zeros, 16 sets, binary16: [1, 1936, 1500]
// 208 us with 6 missed sets, 70 with 4 so; [8, 7744, 512] 584 with 54, 139 with 18.
// ---------------------------------------------------------------------------
template <typename TX, int NT>
__global__ __launch_bounds__(NT, NT == 256 ? 8 : 4) void k_bracket_finish(
    const TX* __restrict__ X, long long ld, int T, int C, int G, int L,
    const int* __restrict__ gid, const u32* __restrict__ bhist, int Wfew, int W, int cells,
    const u32* __restrict__ lists, int cap, int force_miss, Scalars sc, int pass, GroupWork* __restrict__ grp,
    const Bracket* __restrict__ br, float* __restrict__ clip, float* __restrict__ scale,
    tdq_group_stats* __restrict__ stats, const u32* __restrict__ img_flag, int B,
    u32* __restrict__ status) {
  constexpr bool F16 = sizeof(TX) == 2;
  constexpr u32 kKeysAll = F16 ? 1u << 15 : 1u << 31;
  __shared__ FinishLds<NT, false> lds;
  __shared__ u32 s_keys[F16 ? 1 : kListMax];
  __shared__ u32 s_ok, s_key, s_need, s_k0, s_span, s_tie, s_ties;
  __shared__ int s_window;
  __shared__ unsigned long long s_rank;
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
  auto finish = [&](u32 key) {                  // by one thread
    if (pass == kPassBase)
      grp[idx].c_base = Elem<TX>::key_to_float(key);     // the set's base radius Q_p(|x|)
    else
      project_store(idx, w, key, F16, sc, clip, scale, stats);
  };
  enum { kMiss = 0, kDone = 1, kInList = 2 };
  if (wave == 0) {
    u32 ok = kMiss, k0 = 0, span = kKeysAll;    // where a missed key lies, and its rank there
    int window = -1;
    unsigned long long rank = (unsigned long long)w.k_rem;
    if (!force_miss) {
      const Bracket e = br[idx];
      const u32* head = lists + (size_t)idx * cap;
      u32 lo = 0, hi = 0, tie = kNoKey, ties = 0, tie_bin = kNoKey;
      if constexpr (!F16) {
        lo = ~head[kHeadMin];
        hi = head[kHeadMax];
        tie = head[kHeadTie];
        ties = head[kHeadTies];
        tie_bin = head[kHeadTieBin];
      }
      // (the further bins of a set that uses more are looked at only if the first do not do)
      BinPick p = pick_bin<!F16>(bhist + (size_t)idx * W, Wfew, e.below, (u32)w.k_rem, tie_bin, ties);
      if (F16 && w.tokens != 0 && !p.ok && (int)e.width > Wfew && w.k_rem > e.below) {
        const u32 first = p.inside;
        p = pick_bin<false>(bhist + (size_t)idx * W + Wfew, W - Wfew, e.below + first, (u32)w.k_rem);
        p.inside += first;
        p.bin += (u32)Wfew;
      }
      if (w.tokens == 0) {
        ok = kDone;
        if (lane == 0 && pass == kPassZr) project_store(idx, w, 0u, F16, sc, clip, scale, stats);
      } else if (p.ok) {                        // wavefront-uniform
        u32 key = e.lo + p.bin;
        ok = kDone;
        if constexpr (!F16) {
          const u32 among = p.bin == tie_bin ? ties : 0u;       // ties in that bin
          key = p.count == 0 ? tie : lo;
          if (p.count != 0 && (lo != hi || among != 0)) {
            if (w.prefix == p.count) {          // all of them were collected
              ok = kInList;
            } else {
              ok = kMiss;
              bin_keys(head[kListHead + (lane < cells ? lane : 0)], cells, e, p.bin, k0, span);
              rank = p.need;
            }
          }
          if (lane == 0) {
            s_need = p.need;
            s_tie = tie;
            s_ties = among;
          }
        }
        if (ok == kDone && lane == 0) finish(key);
      } else {
        const Lost l = lost_rank<F16>((u32)w.k_rem, (u32)w.n, e.below, p.inside, e.lo,
                                      e.lo + (e.shift & kCells ? e.width : e.width << e.shift));
        k0 = l.k0;
        span = l.span;
        window = l.window;
        rank = l.rank;
        if (k0 == 0 && span == 1u) {            // below the interval, where there are only zeros
          ok = kDone;
          if (lane == 0) finish(0u);
        }
      }
    } else if (w.tokens == 0) {
      ok = kDone;
      if (lane == 0 && pass == kPassZr) project_store(idx, w, 0u, F16, sc, clip, scale, stats);
    }
    if (lane == 0) {
      s_ok = ok;
      s_k0 = k0;
      s_span = span;
      s_window = window;
      s_rank = rank;
    }
  }
  __syncthreads();
  if (s_ok == kDone) return;
  if constexpr (!F16) {
    if (s_ok == kInList) {
      // the key with fewer than `need` smaller ones and at least `need` not larger, among the
      // collected ones and the ties
      const int n = (int)w.prefix;
      const u32* keys = lists + (size_t)idx * cap + kListHead + cells;
      for (int i = tid; i < n; i += NT) s_keys[i] = keys[i];
      __syncthreads();
      const u32 need = s_need, tie = s_tie, ties = s_ties;
      for (int i = tid; i < n + (ties ? 1 : 0); i += NT) {
        const u32 mine = i < n ? s_keys[i] : tie;
        u32 less = tie < mine ? ties : 0u, equal = tie == mine ? ties : 0u;
        for (int c = 0; c < n; ++c) {
          const u32 k = s_keys[c];
          less += k < mine ? 1u : 0u;
          equal += k == mine ? 1u : 0u;
        }
        if (less < need && need <= less + equal) s_key = mine;     // equal keys write the same
      }
      __syncthreads();
      if (tid == 0) finish(s_key);
      return;
    }
  }
  // The interval missed rank k (or the validation switch asked for this route).
  if (tid == 0) atomicAdd(&status[1 + pass], 1u);
  const u32 key = search_rows<TX, NT, false>(X + (long long)b * T * ld, ld, T, C, L, gid + (long long)b * T, j,
                                             nullptr, s_k0, s_span, s_rank, s_window, lds);
  if (tid == 0) finish(key);
}

hipError_t launch_bracket_finish(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                                 int Wfew, int W, int cells, const int* gid, const unsigned* bhist,
                                 const unsigned* lists, int cap, bool force_miss, const Scalars& sc, int pass, GroupWork* grp,
                                 const Bracket* br, float* clip, float* scale, tdq_group_stats* stats,
                                 const unsigned* img_flag, unsigned* status, hipStream_t st) {
  const int L = sweep_lanes_per_row(C, dt == TDQ_F16 ? 8 : 4);
#define TDQ_FINISH(TX, NT)                                                                              \
  hipLaunchKernelGGL((k_bracket_finish<TX, NT>), dim3(B * G), dim3(NT), 0, st, static_cast<const TX*>(X), \
                     ld, T, C, G, L, gid, bhist, Wfew, W, cells, lists, cap, force_miss ? 1 : 0, sc, pass, grp,  \
                     br, clip, scale, stats, img_flag, B, status)
  const bool large = B * G <= 256;              // one workgroup per CU
  if (dt == TDQ_F16) {
    if (large) TDQ_FINISH(u16, 1024); else TDQ_FINISH(u16, 256);
  } else {
    if (large) TDQ_FINISH(float, 1024); else TDQ_FINISH(float, 256);
  }
#undef TDQ_FINISH
  return hipGetLastError();
}

}  // namespace tdq
