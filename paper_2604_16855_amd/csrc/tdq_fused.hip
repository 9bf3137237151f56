// Single-launch form of the activation path for shapes where launch latency, not
// bandwidth, sets the time (a few hundred kilobytes per image): what tdq_calibrate_groups
// followed by tdq_quantize_act compute, in ONE kernel, one workgroup of 1024 threads per
// image, the steps separated by workgroup barriers instead of kernel boundaries:
//   A  per-token range, mean and centred second moment  (Sec. 4.2)
//   B  token -> token set, per-set sums                 (assign_tokens; small images: a
//      wavefront per set)
//   C  per set: n, sigma, rank k                        (merge_partials)
//   D  k-th smallest |x| of every set: radix select on the magnitude bit pattern, 8 bits
//      per level, LDS histogram [G][256]                (Eq. zr_constraint, exact)
//   E  projection                                       (Eq. dcrp)
//   F  quantize + pack                                  (Eqs. clipx, dequant)
// (few images that fit a workgroup's registers: k_fused_sets, one workgroup per image and set.)
// X is read once per step that needs it (A, every level of D, F) and comes from the
// cache after the first; an image that fits the workgroup's registers is read once.  Same arithmetic as the multi-kernel path wherever a result is
// rounded: group ids, thresholds and codes are integer work, sigma is binary64.
#include <type_traits>

#include "tdq_device.hpp"

namespace tdq {

constexpr int kFusedThreads = 1024;
constexpr int kFusedMaxG = TDQ_FUSED_MAX_GROUPS;

// REG: the image fits the workgroup's registers (4 pieces of 16 bytes per thread, rows of
// whole aligned pieces, at most 1024 bytes binary16 / 2048 binary32, at most 1024 tokens): X
// is then read once, the tokens' statistics stay in LDS, and every set is formed by a
// wavefront of its own (key intervals as in k_sets) instead of set by set within batches of
// tokens.  196 x 64 binary32: 20.3 us with every step through memory, 16.3
// so (X in registers alone 17.8; the top digit counted in four copies of the histogram: 16.7).
constexpr int kRegPieces = 4;
constexpr int kRegTokens = 1024;
template <typename T>
constexpr int kRegPPL = sizeof(T) == 2 ? 1 : 2;  // pieces of a row per lane

template <typename T, bool REG>
__global__ __launch_bounds__(kFusedThreads) void k_fused_small(
    const T* __restrict__ X, long long ld, int T_, int C, int G, int L, int vec_ok, int q_vec_ok,
    Scalars sc, int with_base, float* __restrict__ r, double* __restrict__ mean,
    double* __restrict__ m2, int* __restrict__ gid, float* __restrict__ clip,
    float* __restrict__ scale, tdq_group_stats* __restrict__ stats, u32* __restrict__ image_flags,
    uint8_t* __restrict__ Q, long long ld_q) {
  constexpr int V = Elem<T>::V;
  constexpr bool F16 = sizeof(T) == 2;
  constexpr int NW = kFusedThreads / 64;
  constexpr int kLevels = F16 ? 2 : 4;
  __shared__ SetAcc wacc[REG ? 1 : NW * kFusedMaxG];
  __shared__ u32 s_key[REG ? kRegTokens : 1];
  __shared__ double s_mean[REG ? kRegTokens : 1], s_m2[REG ? kRegTokens : 1];
  __shared__ unsigned char s_gid[REG ? kRegTokens : 1];      // set ids (< kFusedMaxG)
  __shared__ u32 hist[kFusedMaxG * 256];
  __shared__ GroupWork grp[kFusedMaxG];
  __shared__ SetAcc s_set[REG ? kFusedMaxG : 1];
  __shared__ u32 s_min[NW], s_max[NW], s_lohi[2];

  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int lr = tid & (L - 1);                  // lane of the row group (L a power of two)
  const int rsub = tid / L, rpp = kFusedThreads / L;
  const T* Xb = X + (long long)b * T_ * ld;
  float* rb = r + (long long)b * T_;
  double* meanb = mean + (long long)b * T_;
  double* m2b = m2 + (long long)b * T_;
  int* gb = gid + (long long)b * T_;
  const int nvec = vec_ok ? C / V : 0;
  // up to half of the most sets there are two histograms, and both start clear
  const bool two = 2 * G <= kFusedMaxG;
  for (int i = tid; i < (two ? G * 512 : 0); i += kFusedThreads) hist[i] = 0;

  // pieces lr, lr + L of rows rsub, rsub + rpp, ...
  constexpr int PPL = kRegPPL<T>, RPT = REG ? kRegPieces / PPL : 1;
  uint4 xr[REG ? kRegPieces : 1];
  if constexpr (REG) {
#pragma unroll
    for (int i = 0; i < RPT; ++i)
#pragma unroll
      for (int k = 0; k < PPL; ++k) {
        const int row = rsub + rpp * i, v = lr + L * k;
        xr[i * PPL + k] = *reinterpret_cast<const uint4*>(
            Xb + (long long)(row < T_ ? row : T_ - 1) * ld + (long long)(v < nvec ? v : 0) * V);
      }
  }

  // ---- A: rows are shared out to groups of L lanes; every lane runs every pass (the
  // reductions are lane exchanges), rows past the end are clamped and not stored
  auto row_stats = [&](int row, const uint4* px) {
    const bool valid = row < T_;
    const T* xp = Xb + (long long)(valid ? row : T_ - 1) * ld;
    u32 kmax = 0;
    double a1 = 0.0, a2 = 0.0;
    // binary64 sums about the row's first value (any value of the row is a good enough
    // pivot in binary64; see "Moments" in tdq_device.hpp)
    double P;
    if constexpr (REG) {
      T e[V];
      Elem<T>::unpack(px[0], e);
      P = __shfl((double)Elem<T>::val(e[0]), (int)(threadIdx.x & 63) & ~(L - 1), 64);
    } else {
      P = (double)Elem<T>::val(xp[0]);
    }
    auto add = [&](const uint4& q) {
      T e[V];
      Elem<T>::unpack(q, e);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const double d = (double)Elem<T>::val(e[i]) - P;
        const u32 k = Elem<T>::key(e[i]);
        kmax = k > kmax ? k : kmax;
        a1 += d;
        a2 = fma(d, d, a2);
      }
    };
    if constexpr (REG) {
#pragma unroll
      for (int k = 0; k < PPL; ++k)
        if (lr + L * k < nvec) add(px[k]);
    } else {
      for (int v = lr; v < nvec; v += L) add(*reinterpret_cast<const uint4*>(xp + (long long)v * V));
      for (int c = nvec * V + lr; c < C; c += L) {
        const T x = xp[c];
        const double d = (double)Elem<T>::val(x) - P;
        const u32 k = Elem<T>::key(x);
        kmax = k > kmax ? k : kmax;
        a1 += d;
        a2 = fma(d, d, a2);
      }
    }
    for (int m = L >> 1; m > 0; m >>= 1) {       // butterfly: all L lanes end with the same bits
      const u32 ok = (u32)__shfl_xor((int)kmax, m, 64);
      kmax = ok > kmax ? ok : kmax;
      a1 += __shfl_xor(a1, m, 64);
      a2 += __shfl_xor(a2, m, 64);
    }
    if (lr == 0 && valid) {
      double mu, q;
      pivot_to_central(P, a1, a2, 1.0 / (double)C, mu, q);
      const float range = Elem<T>::key_to_float(kmax);
      if constexpr (REG) {
        s_key[row] = __float_as_uint(range);
        s_mean[row] = mu;
        s_m2[row] = q;
      } else {
        rb[row] = range;
        meanb[row] = mu;
        m2b[row] = q;
      }
    }
  };
  if constexpr (REG) {
#pragma unroll
    for (int i = 0; i < RPT; ++i)
      if (rpp * i < T_) row_stats(rsub + rpp * i, xr + i * PPL);
  } else {
    for (int row0 = 0; row0 < T_; row0 += rpp) row_stats(row0 + rsub, nullptr);
  }
  __syncthreads();                               // the workgroup's global writes are visible to it

  // ---- B, C: one wavefront per set
  if constexpr (REG) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u32 k1 = tid < T_ ? s_key[tid] : 0u;               // T_ <= kRegTokens = threads
    const u32 kmax = wave_max_u32(k1), kmin = wave_min_u32(tid < T_ ? k1 : 0xFFFFFFFFu);
    if (lane == 0) { s_min[wave] = kmin; s_max[wave] = kmax; }
    __syncthreads();
    u32 lo = s_min[0], hi = s_max[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      lo = s_min[w] < lo ? s_min[w] : lo;
      hi = s_max[w] > hi ? s_max[w] : hi;
    }
    const u32 span = (u32)kOctaveFloor << 23, floor_key = hi > span ? hi - span : 0u;
    lo = lo > floor_key ? lo : floor_key;
    if (tid == 0) { s_lohi[0] = lo; s_lohi[1] = hi; }
    const u32 width = hi - lo + 1u, wq = width / (u32)G, wr = width - wq * (u32)G;
    const double cn = (double)C;
    for (int j = wave; j < G; j += NW) {
      const u32 start = j == 0 ? 0u : lo + (u32)j * wq + ((u32)j * wr + (u32)G - 1u) / (u32)G;
      const u32 end =
          j == G - 1 ? hi + 1u : lo + (u32)(j + 1) * wq + ((u32)(j + 1) * wr + (u32)G - 1u) / (u32)G;
      u32 cnt = 0, cmax = 0;
      double a1 = 0.0, a2 = 0.0, piv = 0.0;
      for (int t0 = 0; t0 < T_; t0 += 64) {
        const int t = t0 + lane;
        const u32 k = t < T_ ? s_key[t] : 0u;
        const bool mine = t < T_ && k >= start && k < end;
        const unsigned long long mask = __ballot(mine);
        if (mask == 0) continue;                             // uniform over the wavefront
        if (cnt == 0) {                                      // the set's first token
          piv = s_mean[t0 + __ffsll((long long)mask) - 1];
          piv = (piv - piv == 0.0) ? piv : 0.0;
        }
        cnt += (u32)__popcll(mask);
        if (mine) {
          const double dm = s_mean[t] - piv, d1 = cn * dm;
          a1 += d1;
          a2 += s_m2[t] + d1 * dm;
          cmax = k > cmax ? k : cmax;
          s_gid[t] = (unsigned char)j;
          gb[t] = j;
        }
      }
      a1 = group_sum_f64<64>(a1);                            // totals in lane 63
      a2 = group_sum_f64<64>(a2);
      cmax = group_max_u32<64>(cmax);
      if (lane == 63) {
        SetAcc m;
        m.s1 = a1; m.s2 = a2; m.piv = piv; m.cnt = cnt; m.kmax = cmax;
        s_set[j] = m;
      }
    }
    __syncthreads();
  } else {
    assign_tokens(rb, meanb, m2b, T_, C, G, gb, wacc, s_min, s_max, s_lohi, 0, 1);
  }
  if (tid == 0 && image_flags) image_flags[b] = s_lohi[1] >= 0x7F800000u ? TDQ_DEV_NONFINITE : 0u;

  int gr[RPT];                                   // REG: the set of every row of this thread
  if constexpr (REG) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) gr[i] = rsub + rpp * i < T_ ? (int)s_gid[rsub + rpp * i] : 0;
  }

  int seq = 0;                                   // levels done: which of the two histograms is clear
  // one rank select per rank wanted: the percentile base radius first (if asked for)
  for (int pass = with_base ? kPassBase : kPassZr; pass >= kPassZr; --pass) {
    // ---- C
    if (tid < G) {
      GroupWork w = REG ? merge_partials(s_set, 0, tid, 1, G, C, sc, pass)
                        : merge_partials(wacc, 0, tid, NW, G, C, sc, pass);
      if (pass == kPassZr && with_base) w.c_base = grp[tid].c_base;
      grp[tid] = w;
    }
    // ---- D
#pragma unroll 1
    for (int lev = 0; lev < kLevels; ++lev) {
      const int bits = (F16 && lev == 1) ? 7 : ((!F16 && lev == 3) ? 7 : 8);
      const int done = 8 * lev;                                  // key bits fixed so far
      const int total_bits = F16 ? 15 : 31;
      const int shift = total_bits - done - bits;                // bits below this level's digit
      // (with two histograms the next level's is cleared while this level's is searched)
      u32* const hcur = hist + (two ? (seq & 1) * G * 256 : 0);
      u32* const hnext = hist + (two ? ((seq + 1) & 1) * G * 256 : 0);
      ++seq;
      if (!two) {
        for (int i = tid; i < G * 256; i += kFusedThreads) hist[i] = 0;
      }
      __syncthreads();
      auto count_row = [&](int row, int g, const uint4* px) {
        const u32 want = grp[g].prefix;                          // the `done` high bits
        u32* h = hcur + g * 256;
        auto count = [&](u32 key) {
          if (done == 0 || (key >> (total_bits - done)) == want)
            atomicAdd(&h[(key >> shift) & ((1u << bits) - 1u)], 1u);
        };
        auto count_piece = [&](const uint4& q) {
          T e[V];
          Elem<T>::unpack(q, e);
#pragma unroll
          for (int i = 0; i < V; ++i) count(Elem<T>::key(e[i]));
        };
        if constexpr (REG) {
#pragma unroll
          for (int k = 0; k < PPL; ++k)
            if (lr + L * k < nvec) count_piece(px[k]);
        } else {
          const T* xp = Xb + (long long)row * ld;
          for (int v = lr; v < nvec; v += L)
            count_piece(*reinterpret_cast<const uint4*>(xp + (long long)v * V));
          for (int c = nvec * V + lr; c < C; c += L) count(Elem<T>::key(xp[c]));
        }
      };
      if constexpr (REG) {
#pragma unroll
        for (int i = 0; i < RPT; ++i)
          if (rsub + rpp * i < T_) count_row(rsub + rpp * i, gr[i], xr + i * PPL);
      } else {
        for (int row = rsub; row < T_; row += rpp) count_row(row, gb[row], nullptr);
      }
      __syncthreads();
      if (two)
        for (int i = tid; i < G * 256; i += kFusedThreads) hnext[i] = 0;
      // a wavefront per set: every lane takes 4 consecutive bins, the running count
      // over the lanes finds the lane, then the bin, where it first reaches the rank
      for (int g = tid >> 6; g < G; g += NW) {
        const GroupWork w = grp[g];
        if (w.tokens == 0) continue;                               // uniform over the wavefront
        const int lane = tid & 63;
        const uint4 hb = *reinterpret_cast<const uint4*>(&hcur[g * 256 + 4 * lane]);
        const u32 c4[4] = {hb.x, hb.y, hb.z, hb.w};
        const bool in_range = 4 * lane < (1 << bits);
        long long mine = in_range ? (long long)c4[0] + c4[1] + c4[2] + c4[3] : 0;
        long long incl = mine;                                     // inclusive scan over the lanes
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const long long o = __shfl_up(incl, d, 64);
          if (lane >= d) incl += o;
        }
        const unsigned long long reached = __ballot(incl >= w.k_rem);
        // the ranks never exceed the count of the set's elements under the prefix
        const int first = reached ? __ffsll((long long)reached) - 1 : 63;
        if (lane == first) {
          long long below = incl - mine;
          int j = 0;
          for (; j < 3; ++j) {
            if (below + (long long)c4[j] >= w.k_rem) break;
            below += (long long)c4[j];
          }
          GroupWork nw = w;
          nw.k_rem = w.k_rem - below;
          nw.prefix = (w.prefix << bits) | (u32)(4 * lane + j);
          grp[g] = nw;
        }
      }
      __syncthreads();
    }
    // ---- E
    if (tid < G) {
      const GroupWork w = grp[tid];
      if (pass == kPassBase) {
        if (w.tokens != 0) grp[tid].c_base = Elem<T>::key_to_float(w.prefix);
      } else {
        project_store(b * G + tid, w, w.prefix, F16, sc, clip, scale, stats);
      }
    }
    __syncthreads();
  }

  // ---- F
  if constexpr (REG) {
    // pieces of V elements -> V / 2 bytes each
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int row = rsub + rpp * i;
      if (row >= T_) break;
      const float c = clip[b * G + gr[i]], d = scale[b * G + gr[i]];
      const float rcp = 1.0f / d;
      uint8_t* qp = Q + ((long long)b * T_ + row) * ld_q;
#pragma unroll
      for (int k = 0; k < PPL; ++k) {
        const int v = lr + L * k;
        if (v >= nvec) break;
        T e[V];
        Elem<T>::unpack(xr[i * PPL + k], e);
        u32 word = 0;
#pragma unroll
        for (int j = 0; j < V; ++j) word |= quant_nibble(Elem<T>::val(e[j]), c, d, rcp) << (4 * j);
        if constexpr (F16)
          *reinterpret_cast<u32*>(qp + (long long)v * 4) = word;
        else
          *reinterpret_cast<u16*>(qp + (long long)v * 2) = (u16)word;
      }
    }
    return;
  }
  const int n8 = (vec_ok && q_vec_ok) ? C / 8 : 0;               // units of 8 elements -> 4 bytes
  const int nbytes = (C + 1) / 2;
  for (int row = rsub; row < T_; row += rpp) {
    const T* xp = Xb + (long long)row * ld;
    uint8_t* qp = Q + ((long long)b * T_ + row) * ld_q;
    const int g = gb[row];
    const float c = clip[b * G + g], d = scale[b * G + g];
    const float rcp = 1.0f / d;
    for (int u = lr; u < n8; u += L) {
      u32 word = 0;
#pragma unroll
      for (int j = 0; j < 8 / V; ++j) {
        const uint4 q = *reinterpret_cast<const uint4*>(xp + (long long)u * 8 + j * V);
        T e[V];
        Elem<T>::unpack(q, e);
#pragma unroll
        for (int i = 0; i < V; ++i)
          word |= quant_nibble(Elem<T>::val(e[i]), c, d, rcp) << (4 * (j * V + i));
      }
      *reinterpret_cast<u32*>(qp + (long long)u * 4) = word;
    }
    for (int by = n8 * 4 + lr; by < nbytes; by += L) {
      const int c0 = 2 * by;
      u32 v = quant_nibble(Elem<T>::val(xp[c0]), c, d, rcp);
      if (c0 + 1 < C) v |= quant_nibble(Elem<T>::val(xp[c0 + 1]), c, d, rcp) << 4;
      qp[by] = (uint8_t)v;
    }
  }
}

// ---------------------------------------------------------------------------
// k_fused_sets: images that fit a workgroup's registers, one workgroup per (image, token set).  Every
// workgroup reads the whole image and finds all its tokens' ranges, because the sets follow from the smallest
// and the largest; moments, rank select, projection and quantization are those of its own set's rows only,
// so nothing passes between workgroups.  The rank: an LDS histogram of the key's top bits, then of
// the next ones of the keys in the bin found (2 levels binary16, 3 binary32), found by the whole workgroup.
// Moments: sums in binary64 about a value of the set (the first of its first token), so that a set of identical
// values adds exact zeros.
// Bound by a chain of a dozen barriers and by instruction issue (see k_sets); 512 threads because
// what every wavefront does alike costs by the wavefronts on a SIMD.  196 x 64 binary32 with 8 sets: 16.1 us by
// one workgroup per image, 9.5 so; [8, 64, 128] with 64 sets 24.0 and 9.0; [4, 100, 96] with 32 sets and a percentile
// 33.9 and 12.6.  (1024 threads: 8.8, 10.1 and 10.9, and slower with many sets.)
// ---------------------------------------------------------------------------
constexpr int kSetsThreads = 512;
constexpr int kSetsPieces = 8;                   // 16-byte pieces per thread, as many bytes as kFusedThreads x kRegPieces

template <typename T>
__global__ __launch_bounds__(kSetsThreads, 4) void k_fused_sets(
    const T* __restrict__ X, long long ld, int T_, int C, int G, int L, Scalars sc, int with_base,
    int* __restrict__ gid, float* __restrict__ clip, float* __restrict__ scale,
    tdq_group_stats* __restrict__ stats, u32* __restrict__ image_flags, uint8_t* __restrict__ Q,
    long long ld_q) {
  constexpr int V = Elem<T>::V, NT = kSetsThreads, NW = NT / 64;
  constexpr bool F16 = sizeof(T) == 2;
  constexpr int kKeyBits = F16 ? 15 : 31;
  constexpr int PPL = kRegPPL<T>, RPT = kSetsPieces / PPL;
  constexpr int kBins = F16 ? 1024 : 2048;       // 10 + 5 or 11 + 10 + 10 key bits
  constexpr int kLevels = F16 ? 2 : 3;
  __shared__ __attribute__((aligned(16))) u32 hist[kLevels][kBins];
  __shared__ u32 s_key[kRegTokens];
  __shared__ u32 s_min[NW], s_max[NW], s_cnt[NW], s_kmax[NW], s_first[NW], stot[1][NW], s_bin[1], s_before[1];
  __shared__ double s_s1[NW], s_s2[NW];
  __shared__ float s_c, s_d;
  const int j = blockIdx.x, b = blockIdx.y, idx = b * G + j;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lsh = 31 - __clz(L);
  const int lr = tid & (L - 1), rsub = tid >> lsh, rpp = NT >> lsh;
  const T* Xb = X + (long long)b * T_ * ld;
  const int nvec = C / V;

  // pieces lr, lr + L of rows rsub, rsub + rpp, ...
  uint4 xr[RPT][PPL];
#pragma unroll
  for (int i = 0; i < RPT; ++i)
#pragma unroll
    for (int k = 0; k < PPL; ++k) {
      const int row = rsub + rpp * i, v = lr + L * k;
      xr[i][k] = *reinterpret_cast<const uint4*>(Xb + (long long)(row < T_ ? row : T_ - 1) * ld +
                                                 (long long)(v < nvec ? v : 0) * V);
    }
  auto clear_hist = [&]() {
    for (int i = tid; i < kLevels * kBins / 4; i += NT)
      reinterpret_cast<uint4*>(&hist[0][0])[i] = make_uint4(0, 0, 0, 0);
  };
  clear_hist();

  // ---- the tokens' ranges (a lane that has no second piece counts its row's first piece twice)
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    if (i > 0 && rpp * i >= T_) break;           // uniform
    u32 km = 0;
#pragma unroll
    for (int k = 0; k < PPL; ++k) {
      T e[V];
      Elem<T>::unpack(xr[i][k], e);
#pragma unroll
      for (int c = 0; c < V; ++c) {
        const u32 key = Elem<T>::key(e[c]);
        km = key > km ? key : km;
      }
    }
    u32 o;
    if (L > 1) { o = dpp_u32<TDQ_DPP_ROW_SHR(1), 0xF>(km); km = o > km ? o : km; }
    if (L > 2) { o = dpp_u32<TDQ_DPP_ROW_SHR(2), 0xF>(km); km = o > km ? o : km; }
    if (L > 4) { o = dpp_u32<TDQ_DPP_ROW_SHR(4), 0xF>(km); km = o > km ? o : km; }
    if (L > 8) { o = dpp_u32<TDQ_DPP_ROW_SHR(8), 0xF>(km); km = o > km ? o : km; }
    if (L > 16) { o = dpp_u32<TDQ_DPP_ROW_BCAST15, 0xA>(km); km = o > km ? o : km; }
    if (L > 32) { o = dpp_u32<TDQ_DPP_ROW_BCAST31, 0xC>(km); km = o > km ? o : km; }
    const int row = rsub + rpp * i;
    if (lr == L - 1 && row < T_) s_key[row] = __float_as_uint(Elem<T>::key_to_float(km));
  }
  __syncthreads();

  // ---- the image's key range, the set's key interval (as in k_sets) and tokens
  constexpr int kPer = kRegTokens / NT;          // tokens per thread
  u32 k1[kPer], kinv = 0, khi = 0;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int t = u * NT + tid;
    k1[u] = t < T_ ? s_key[t] : 0xFFFFFFFFu;     // (no range key)
    kinv = ~k1[u] > kinv ? ~k1[u] : kinv;
    khi = k1[u] != 0xFFFFFFFFu && k1[u] > khi ? k1[u] : khi;
  }
  kinv = group_max_u32<64>(kinv);
  khi = group_max_u32<64>(khi);
  if (lane == 63) { s_min[wave] = ~kinv; s_max[wave] = khi; }
  __syncthreads();
  u32 lo = s_min[0], hi = s_max[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    lo = s_min[w] < lo ? s_min[w] : lo;
    hi = s_max[w] > hi ? s_max[w] : hi;
  }
  const u32 span = (u32)kOctaveFloor << 23, floor_key = hi > span ? hi - span : 0u;
  lo = lo > floor_key ? lo : floor_key;
  if (tid == 0 && j == 0 && image_flags) image_flags[b] = hi >= 0x7F800000u ? TDQ_DEV_NONFINITE : 0u;
  const u32 width = hi - lo + 1u, wq = width / (u32)G, wr = width - wq * (u32)G;
  const u32 start = j == 0 ? 0u : lo + (u32)j * wq + ((u32)j * wr + (u32)G - 1u) / (u32)G;
  const u32 end = j == G - 1 ? hi + 1u : lo + (u32)(j + 1) * wq + ((u32)(j + 1) * wr + (u32)G - 1u) / (u32)G;
  auto in_set = [&](u32 k) { return k >= start && k < end; };
  u32 cnt = 0, kmax = 0, first = 0xFFFFFFFFu;    // tokens, largest range, first token of this wavefront
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const bool mine = in_set(k1[u]);
    const unsigned long long mask = __ballot(mine);
    cnt += (u32)__popcll(mask);
    if (mine) {
      gid[(long long)b * T_ + u * NT + tid] = j;
      kmax = k1[u] > kmax ? k1[u] : kmax;
    }
    if (mask != 0 && first == 0xFFFFFFFFu) first = (u32)(u * NT + wave * 64 + __ffsll((long long)mask) - 1);
  }
  kmax = group_max_u32<64>(kmax);
  if (lane == 63) { s_cnt[wave] = cnt; s_kmax[wave] = kmax; s_first[wave] = first; }
  __syncthreads();
  u32 tokens = 0, t_first = 0xFFFFFFFFu, c_key = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    tokens += s_cnt[w];
    t_first = s_first[w] < t_first ? s_first[w] : t_first;
    c_key = s_kmax[w] > c_key ? s_kmax[w] : c_key;
  }
  GroupWork w;
  w.tokens = tokens;
  w.n = (long long)tokens * C;
  w.k_rem = 0;
  w.prefix = 0;
  w.c_base = __uint_as_float(c_key);
  w.sigma = 0.f;
  if (tokens == 0) {
    if (tid == 0) project_store(idx, w, 0u, F16, sc, clip, scale, stats);
    return;
  }
  bool own[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int row = rsub + rpp * i;
    own[i] = row < T_ && in_set(s_key[row < T_ ? row : 0]);
  }

  // ---- moments, and the top key bits of the set's elements
  double P = (double)Elem<T>::val(Xb[(long long)t_first * ld]);
  P = P - P == 0.0 ? P : 0.0;
  const double n = (double)w.n;
  double a1 = 0.0, a2 = 0.0;
  auto each = [&](auto&& f) {                    // the set's elements in this thread's registers
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
#pragma unroll
      for (int k = 0; k < PPL; ++k) {
        if (own[i] && lr + L * k < nvec) {
          // (opaque: keys and values kept from one use to the next would not fit the registers)
          uint4 q = xr[i][k];
          asm volatile("" : "+v"(q.x), "+v"(q.y), "+v"(q.z), "+v"(q.w));
          T e[V];
          Elem<T>::unpack(q, e);
#pragma unroll
          for (int c = 0; c < V; ++c) f(e[c]);
        }
      }
    }
  };
  constexpr int kTop = F16 ? 10 : 11;
  each([&](T x) {
    const double d = (double)Elem<T>::val(x) - P;
    a1 += d;
    a2 = fma(d, d, a2);
    atomicAdd(&hist[0][Elem<T>::key(x) >> (kKeyBits - kTop)], 1u);
  });
  a1 = group_sum_f64<64>(a1);
  a2 = group_sum_f64<64>(a2);
  if (lane == 63) { s_s1[wave] = a1; s_s2[wave] = a2; }
  __syncthreads();

  // ---- the ranks wanted: the percentile base radius first (if asked for)
  u32 key = 0;
#pragma unroll 1
  for (int pass = with_base ? kPassBase : kPassZr; pass >= kPassZr; --pass) {
    long long k = (long long)ceil((pass == kPassBase ? sc.base_pct : sc.zr) * n);
    k = k < 1 ? 1 : (k > w.n ? w.n : k);
    u32 rank = (u32)k;
    auto find = [&](const u32* h, auto bins) {
      const u32* const hs[1] = {h};
      const u32 rs[1] = {rank};
      find_ranks<NT, 1, 1, false, decltype(bins)::value>(hs, rs, stot, s_bin, s_before, nullptr);
      __syncthreads();
      rank -= s_before[0];
      return s_bin[0];
    };
    key = find(hist[0], std::integral_constant<int, kBins>{});
    if constexpr (F16) {
      each([&](T x) {
        const u32 kx = Elem<T>::key(x);
        if (kx >> 5 == key) atomicAdd(&hist[1][kx & 31u], 1u);
      });
      __syncthreads();
      key = key << 5 | find(hist[1], std::integral_constant<int, kBins>{});
    } else {
      each([&](T x) {
        const u32 kx = Elem<T>::key(x);
        if (kx >> 20 == key) atomicAdd(&hist[1][kx >> 10 & 1023u], 1u);
      });
      __syncthreads();
      key = key << 10 | find(hist[1], std::integral_constant<int, 1024>{});
      each([&](T x) {
        const u32 kx = Elem<T>::key(x);
        if (kx >> 10 == key) atomicAdd(&hist[kLevels - 1][kx & 1023u], 1u);
      });
      __syncthreads();
      key = key << 10 | find(hist[kLevels - 1], std::integral_constant<int, 1024>{});
    }
    if (pass == kPassBase) {
      w.c_base = Elem<T>::key_to_float(key);
      __syncthreads();
      for (int i = tid; i < (kLevels - 1) * kBins; i += NT) hist[1][i] = 0;
      __syncthreads();
    }
  }
  if (tid == 0) {
    double S1 = s_s1[0], S2 = s_s2[0];
#pragma unroll
    for (int q = 1; q < NW; ++q) { S1 += s_s1[q]; S2 += s_s2[q]; }
    const double mu = S1 / n;
    double var = S2 / n - mu * mu;
    var = var > 0.0 ? var : 0.0;
    w.sigma = (float)(sqrt(var) + sc.eps_std);
    const float2 cd = project_store(idx, w, key, F16, sc, clip, scale, stats);
    s_c = cd.x;
    s_d = cd.y;
  }
  __syncthreads();

  // ---- codes of the set's rows: pieces of V elements -> V / 2 bytes each
  const float c = s_c, d = s_d, rcp = 1.0f / d;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    if (!own[i]) continue;
    uint8_t* qp = Q + ((long long)b * T_ + rsub + rpp * i) * ld_q;
#pragma unroll
    for (int k = 0; k < PPL; ++k) {
      const int v = lr + L * k;
      if (v >= nvec) break;
      T e[V];
      Elem<T>::unpack(xr[i][k], e);
      u32 word = 0;
#pragma unroll
      for (int q = 0; q < V; ++q) word |= quant_nibble(Elem<T>::val(e[q]), c, d, rcp) << (4 * q);
      if constexpr (F16)
        *reinterpret_cast<u32*>(qp + (long long)v * 4) = word;
      else
        *reinterpret_cast<u16*>(qp + (long long)v * 2) = (u16)word;
    }
  }
}

template <typename T>
static hipError_t fused_t(const T* X, int B, int T_, int C, long long ld, int G, const Scalars& sc,
                          float* r, double* mean, double* m2, int* gid, float* clip, float* scale,
                          tdq_group_stats* stats, unsigned* image_flags, uint8_t* Q, long long ld_q,
                          hipStream_t st) {
  constexpr int V = Elem<T>::V;
  const int vec_ok = ((reinterpret_cast<uintptr_t>(X) & 15) == 0 && ld % V == 0) ? 1 : 0;
  const int q_vec_ok = ((reinterpret_cast<uintptr_t>(Q) & 3) == 0 && ld_q % 4 == 0) ? 1 : 0;
  const int L = lanes_per_row(C, 8);
  const int with_base = sc.base_pct > 0.0 ? 1 : 0;
  const bool reg = T_ <= kRegTokens && vec_ok && q_vec_ok && C % V == 0 && C / V <= L * kRegPPL<T> &&
                   (long long)T_ <= (long long)(kFusedThreads / L) * (kRegPieces / kRegPPL<T>);
  static_assert(kSetsThreads * kSetsPieces == kFusedThreads * kRegPieces, "the same images fit");
  // A workgroup per set reads its image again: better until the chip holds no more of them at once (two to
  // four per CU), us per image / per set: 512 sets [32, 196, 64] binary32 18.6 / 12.0; 1024 sets 23.0 / 18.2 of it but
  // [64, 196, 64] binary16 13.5 / 16.6 and [256, 49, 96] 12.3 / 15.2; 2048 sets [128, 196, 64] 13.7 / 28.3.
  if (reg && (long long)B * G <= 512)
    hipLaunchKernelGGL((k_fused_sets<T>), dim3(G, B), dim3(kSetsThreads), 0, st, X, ld, T_, C, G, L, sc,
                       with_base, gid, clip, scale, stats, image_flags, Q, ld_q);
  else if (reg)
    hipLaunchKernelGGL((k_fused_small<T, true>), dim3(B), dim3(kFusedThreads), 0, st, X, ld, T_, C, G, L,
                       vec_ok, q_vec_ok, sc, with_base, r, mean, m2, gid, clip, scale, stats,
                       image_flags, Q, ld_q);
  else
    hipLaunchKernelGGL((k_fused_small<T, false>), dim3(B), dim3(kFusedThreads), 0, st, X, ld, T_, C, G, L,
                       vec_ok, q_vec_ok, sc, with_base, r, mean, m2, gid, clip, scale, stats,
                       image_flags, Q, ld_q);
  return hipGetLastError();
}

hipError_t launch_fused_small(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                              const Scalars& sc, float* r, double* mean, double* m2, int* gid,
                              float* clip, float* scale, tdq_group_stats* stats,
                              unsigned* image_flags, uint8_t* Q, long long ld_q, hipStream_t st) {
  if (dt == TDQ_F16)
    return fused_t<u16>(static_cast<const u16*>(X), B, T, C, ld, G, sc, r, mean, m2, gid, clip, scale,
                        stats, image_flags, Q, ld_q, st);
  return fused_t<float>(static_cast<const float*>(X), B, T, C, ld, G, sc, r, mean, m2, gid, clip, scale,
                        stats, image_flags, Q, ld_q, st);
}

}  // namespace tdq
