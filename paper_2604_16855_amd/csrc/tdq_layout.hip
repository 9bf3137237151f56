// Convolutional feature maps as tokens (Supp. "Implementation details": the dynamic
// activation path maps X[B, C, H, W] to X'[B, HW, C] and applies DSTG + DCRP along the
// channel dimension): an exact re-layout X[b, c, t] -> Xt[b * T + t, c], t = h * W + w,
// after which every token-major entry point applies.
//
// One workgroup moves a tile of 64 channels x TT tokens (TT = 128 for binary16, 64 for
// binary32) through LDS: 16-byte loads along the token axis (the contiguous one of the
// input), 16-byte stores along the channel axis (the contiguous one of the output), so
// both sides move whole 128-byte lines per 8 lanes.  The transposition is on the LDS
// read side: 8 (4) two- (four-) byte reads per 16-byte store; rows of the LDS tile are 8
// bytes longer than the data, which leaves those reads with two-way bank conflicts at
// most.
#include <type_traits>

#include "tdq_device.hpp"

namespace tdq {

template <typename T>
__global__ __launch_bounds__(256) void k_tokenize_chw(const T* __restrict__ X, long long ld_c,
                                                      long long ld_b, int C, int T_,
                                                      T* __restrict__ Xt, long long ld_xt, int vin_ok,
                                                      int vout_ok) {
  constexpr int E = 16 / (int)sizeof(T);     // elements per 16 bytes
  constexpr int TC = 64;                     // channels per tile
  constexpr int TT = 16 * E;                 // tokens per tile
  constexpr int PITCH = TT + 8 / (int)sizeof(T);
  constexpr int PQ = TC / E;                 // 16-byte pieces per token row of the tile
  __shared__ __attribute__((aligned(16))) T tile[TC][PITCH];

  const int t0 = blockIdx.x * TT, c0 = blockIdx.y * TC, b = blockIdx.z;
  const int tid = threadIdx.x;
  const T* xb = X + (long long)b * ld_b;

  // in: thread t owns the piece t % 16 (E tokens) of channels t / 16 + 16 i
  {
    const int p = tid & 15;
    const int tok = t0 + p * E;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int ch = (tid >> 4) + 16 * i;
      const int c = c0 + ch;
      __attribute__((aligned(16))) T v[E];
      if (c < C && vin_ok && tok + E <= T_) {
        const uint4 q = *reinterpret_cast<const uint4*>(xb + (long long)c * ld_c + tok);
        *reinterpret_cast<uint4*>(v) = q;
      } else {
#pragma unroll
        for (int k = 0; k < E; ++k)
          v[k] = (c < C && tok + k < T_) ? xb[(long long)c * ld_c + tok + k] : (T)0;
      }
      // rows are 8 bytes apart from a multiple of 16: two 8-byte writes
      uint2* d = reinterpret_cast<uint2*>(&tile[ch][p * E]);
      const uint2* s = reinterpret_cast<const uint2*>(v);
      d[0] = s[0];
      d[1] = s[1];
    }
  }
  __syncthreads();
  // out: thread t owns the piece t % PQ (E channels) of tokens t / PQ + (256 / PQ) i
  {
    const int q = tid % PQ;
    const int c = c0 + q * E;
    constexpr int TPP = 256 / PQ;            // tokens per pass
#pragma unroll
    for (int i = 0; i < TT / TPP; ++i) {
      const int tl = tid / PQ + TPP * i;
      const int tok = t0 + tl;
      if (tok >= T_) continue;
      __attribute__((aligned(16))) T v[E];
#pragma unroll
      for (int k = 0; k < E; ++k) v[k] = tile[q * E + k][tl];
      T* dst = Xt + ((long long)b * T_ + tok) * ld_xt + c;
      if (vout_ok && c + E <= C) {
        *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(v);
      } else {
#pragma unroll
        for (int k = 0; k < E; ++k)
          if (c + k < C) dst[k] = v[k];
      }
    }
  }
}

template <typename T>
static hipError_t tokenize_t(const T* X, int B, int C, int T_, long long ld_c, long long ld_b, T* Xt,
                             long long ld_xt, hipStream_t st) {
  constexpr int E = 16 / (int)sizeof(T);
  const int vin_ok =
      ((reinterpret_cast<uintptr_t>(X) & 15) == 0 && ld_c % E == 0 && ld_b % E == 0) ? 1 : 0;
  const int vout_ok = ((reinterpret_cast<uintptr_t>(Xt) & 15) == 0 && ld_xt % E == 0) ? 1 : 0;
  const dim3 grid((unsigned)((T_ + 16 * E - 1) / (16 * E)), (unsigned)((C + 63) / 64), (unsigned)B);
  hipLaunchKernelGGL((k_tokenize_chw<T>), grid, dim3(256), 0, st, X, ld_c, ld_b, C, T_, Xt, ld_xt,
                     vin_ok, vout_ok);
  return hipGetLastError();
}

hipError_t launch_tokenize_chw(const void* X, tdq_dtype dt, int B, int C, int T, long long ld_c,
                               long long ld_b, void* Xt, long long ld_xt, hipStream_t st) {
  if (dt == TDQ_F16)
    return tokenize_t<u16>(static_cast<const u16*>(X), B, C, T, ld_c, ld_b, static_cast<u16*>(Xt),
                           ld_xt, st);
  return tokenize_t<float>(static_cast<const float*>(X), B, C, T, ld_c, ld_b,
                           static_cast<float*>(Xt), ld_xt, st);
}

// ---------------------------------------------------------------------------
// The re-layout fused with the statistics sweep of the token-set path: one read of the
// feature map yields the token-major copy Xt AND every token's range and moments
// (r_t = max_c |x|, mean_t, M2_t = sum_c (x - mean_t)^2; Sec. 4.2), so a convolutional input costs
// the token-set path one extra write of X, not an extra read and write.  A workgroup
// owns TT consecutive tokens of one image and walks the channel axis in tiles of 64 or 128:
// every thread keeps the partial statistics of its 2 tokens across the tiles; at the end
// the lanes that share a token (adjacent ones) are reduced with DPP.  The sums are taken
// about a per-token pivot taken from the first tile, see "Moments" in tdq_device.hpp:
// binary32 input, the token's first channel; binary16 input, the mean of its first
// min(C, 64 or 128) channels.  The map is read once, so a token cannot be summed again about a
// better pivot as in the token-major sweep; the mean of 64 of its values lies within
// sigma_t sqrt(C / 64) of the token's mean (Cauchy-Schwarz), which bounds what the
// binary32 partial sums can cost its M2 at (1 + C / 64) * 3 * 2^-24 per partial.
// ---------------------------------------------------------------------------
// Tiles of 64 channels x 128 bytes of tokens: what bounds this sweep on ordinary maps is the
// chain of tiles a workgroup walks, so the tokens are cut finely and a thread reads two
// neighbouring binary16 tokens with one LDS word.  [8, 320, 44, 44] binary16: this kernel 18.6
// us with 256 bytes of tokens, 11.7 so, 14.2 / 18.3 with 128 / 256 channels per tile; the
// whole calibration of [4, 4096, 64, 64] 225 -> 138 us, of [32, 1024, 64, 64] 195 -> 190.
// TC channels x PP 16-byte pieces of tokens per tile: 64 x 8, or 128 x 4 where that makes fewer workgroups than
// CUs (half the tiles in a chain, twice the workgroups).  Calibration, us, 64 x 8 and 128 x 4: [8, 320, 44, 44]
// (248 workgroups of 64 x 8) 29.4 and 27.0, [2, 2000, 20, 20] (14) 51.0 and 34.8, [1, 512, 30, 30] (15) 25.7 and 21.3;
// but [16, 320, 44, 44] (496) 32.2 and 32.9, [32, 256, 40, 40] (800) 36.4 and 40.3: half a line a load.
template <typename T, int TC, int PP>
__global__ __launch_bounds__(256) void k_tokenize_stats_chw(
    const T* __restrict__ X, long long ld_c, long long ld_b, int C, int T_, T* __restrict__ Xt,
    long long ld_xt, int vin_ok, int vout_ok, float* __restrict__ r, double* __restrict__ mean,
    double* __restrict__ m2, SelectClear cl) {
  constexpr bool F16 = sizeof(T) == 2;
  constexpr int E = 16 / (int)sizeof(T);
  constexpr int TT = PP * E;                 // 128 or 64 bytes of every channel
  constexpr int PITCH = TT + 4 / (int)sizeof(T);   // one bank further per row
  constexpr int PQ = TC / E;                 // lanes per token
  constexpr int NP = TT * PQ / 256;          // tokens per thread (2)
  constexpr int TPW = F16 ? 2 : 1;           // tokens a thread reads together (one 32-bit word)
  constexpr int LOADS = TC * PP / 256;       // 16-byte loads per thread and tile
  constexpr int ROWS = 256 / PP;             // channels per load
  __shared__ __attribute__((aligned(16))) T tile[TC][PITCH];

  const int t0 = (int)((blockIdx.z * gridDim.x + blockIdx.x) * TT), b = blockIdx.y;
  clear_select(cl, ((unsigned long long)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x,
               (unsigned long long)gridDim.x * gridDim.y * 256);      // (every z the same)
  if (t0 >= T_) return;                      // (the whole workgroup)
  const int tid = threadIdx.x;
  const T* xb = X + (long long)b * ld_b;
  const int q = tid % PQ;
  u32 kmax[NP];
  double a1[NP], a2[NP];
  typedef typename std::conditional<sizeof(T) == 2, float, double>::type PT;
  PT P[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) { kmax[i] = 0; a1[i] = 0.0; a2[i] = 0.0; P[i] = 0; }

  // the next tile's global loads are in flight while the current one is processed
  const int lp = tid % PP, ltok = t0 + lp * E;
  uint4 stage[LOADS];
  auto load_tile = [&](int c0) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int c = c0 + tid / PP + ROWS * i;
      if (c < C && vin_ok && ltok + E <= T_) {
        stage[i] = *reinterpret_cast<const uint4*>(xb + (long long)c * ld_c + ltok);
      } else {
        __attribute__((aligned(16))) T v[E];
#pragma unroll
        for (int k = 0; k < E; ++k)
          v[k] = (c < C && ltok + k < T_) ? xb[(long long)c * ld_c + ltok + k] : (T)0;
        stage[i] = *reinterpret_cast<const uint4*>(v);
      }
    }
  };
  // token i of this thread: tokens TPW (tid / PQ + ...) + 0 .. TPW - 1 of every group
  auto token = [&](int i) { return TPW * (tid / PQ + (256 / PQ) * (i / TPW)) + i % TPW; };
  load_tile(0);
  for (int c0 = 0; c0 < C; c0 += TC) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      u32* d = reinterpret_cast<u32*>(&tile[tid / PP + ROWS * i][lp * E]);
      d[0] = stage[i].x;
      d[1] = stage[i].y;
      d[2] = stage[i].z;
      d[3] = stage[i].w;
    }
    __syncthreads();
    if (c0 + TC < C) load_tile(c0 + TC);
    const int c = c0 + q * E;
#pragma unroll
    for (int g = 0; g < NP / TPW; ++g) {
      // E channels of TPW neighbouring tokens
      u32 w[E];
#pragma unroll
      for (int k = 0; k < E; ++k)
        w[k] = *reinterpret_cast<const u32*>(&tile[q * E + k][token(g * TPW)]);
#pragma unroll
      for (int h = 0; h < TPW; ++h) {
        const int i = g * TPW + h;
        const int tok = t0 + token(i);
        u32 p4[4];                                 // the token's E channels, packed
        if constexpr (F16) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            p4[k] = __builtin_amdgcn_perm(w[2 * k + 1], w[2 * k], h == 0 ? 0x05040100u : 0x07060302u);
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) p4[k] = w[k];
        }
        const uint4 pk = make_uint4(p4[0], p4[1], p4[2], p4[3]);
        T v[E];
        Elem<T>::unpack(pk, v);
        if (c0 == 0) {                             // the token's pivot, from the first tile
          if constexpr (F16) {
            float sum = 0.f;                       // channels past C are zeros in the tile
#pragma unroll
            for (int k = 0; k < E; ++k) sum += Elem<T>::val(v[k]);
            sum = xor_reduce_sum<PQ, float>(sum);  // the same bits in all lanes of the token
            P[i] = sum / (float)(C < TC ? C : TC);
          } else {
            P[i] = (double)Elem<T>::val(tile[0][token(i)]);
          }
        }
        // channels beyond C are zeros in the tile: they do not change the maximum, and are
        // kept out of the sums
        if constexpr (F16) {
          // as in the token-major statistics sweep: the 8 differences and their squares are
          // first summed in binary32, then accumulated in binary64
          float p1 = 0.f, p2 = 0.f;
#pragma unroll
          for (int k = 0; k < E; ++k) {
            const u32 key = Elem<T>::key(v[k]);
            kmax[i] = key > kmax[i] ? key : kmax[i];
            const float d = c + k < C ? Elem<T>::val(v[k]) - P[i] : 0.f;
            p1 += d;
            p2 = __builtin_fmaf(d, d, p2);
          }
          a1[i] += (double)p1;
          a2[i] += (double)p2;
        } else {
#pragma unroll
          for (int k = 0; k < E; ++k) {
            const u32 key = Elem<T>::key(v[k]);
            kmax[i] = key > kmax[i] ? key : kmax[i];
            const double d = c + k < C ? (double)Elem<T>::val(v[k]) - P[i] : 0.0;
            a1[i] += d;
            a2[i] = fma(d, d, a2[i]);
          }
        }
        if (tok < T_) {
          T* dst = Xt + ((long long)b * T_ + tok) * ld_xt + c;
          if (vout_ok && c + E <= C) {
            *reinterpret_cast<uint4*>(dst) = pk;
          } else {
#pragma unroll
            for (int k = 0; k < E; ++k)
              if (c + k < C) dst[k] = v[k];
          }
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const u32 km = group_max_u32<PQ>(kmax[i]);
    const double t1 = group_sum_f64<PQ>(a1[i]);
    const double t2 = group_sum_f64<PQ>(a2[i]);
    const int tok = t0 + token(i);
    if (q == PQ - 1 && tok < T_) {               // the group's last lane holds the totals
      const long long row = (long long)b * T_ + tok;
      double mu, qq;
      pivot_to_central((double)P[i], t1, t2, 1.0 / (double)C, mu, qq);
      r[row] = Elem<T>::key_to_float(km);
      mean[row] = mu;
      m2[row] = qq;
    }
  }
}

template <typename T>
static hipError_t tokenize_stats_t(const T* X, int B, int C, int T_, long long ld_c, long long ld_b,
                                   T* Xt, long long ld_xt, float* r, double* mean, double* m2,
                                   const SelectClear& cl, hipStream_t st) {
  constexpr int E = 16 / (int)sizeof(T);
  const int vin_ok =
      ((reinterpret_cast<uintptr_t>(X) & 15) == 0 && ld_c % E == 0 && ld_b % E == 0) ? 1 : 0;
  const int vout_ok = ((reinterpret_cast<uintptr_t>(Xt) & 15) == 0 && ld_xt % E == 0) ? 1 : 0;
  // (a grid has fewer than 2^32 threads along an axis: 2^29 tokens of binary32 are 2^24 workgroups)
  const unsigned tiles = (unsigned)((T_ + 8 * E - 1) / (8 * E)), most = 1u << 22;
  if (C > 64 && (long long)tiles * B <= 256) {
    hipLaunchKernelGGL((k_tokenize_stats_chw<T, 128, 4>), dim3((unsigned)((T_ + 4 * E - 1) / (4 * E)), (unsigned)B),
                       dim3(256), 0, st, X, ld_c, ld_b, C, T_, Xt, ld_xt, vin_ok, vout_ok, r, mean, m2, cl);
    return hipGetLastError();
  }
  const dim3 grid(tiles < most ? tiles : most, (unsigned)B, (tiles + most - 1) / most);
  hipLaunchKernelGGL((k_tokenize_stats_chw<T, 64, 8>), grid, dim3(256), 0, st, X, ld_c, ld_b, C, T_, Xt,
                     ld_xt, vin_ok, vout_ok, r, mean, m2, cl);
  return hipGetLastError();
}

hipError_t launch_tokenize_stats_chw(const void* X, tdq_dtype dt, int B, int C, int T, long long ld_c,
                                     long long ld_b, void* Xt, long long ld_xt, float* r, double* mean,
                                     double* m2, const SelectClear& cl, hipStream_t st) {
  if (dt == TDQ_F16)
    return tokenize_stats_t<u16>(static_cast<const u16*>(X), B, C, T, ld_c, ld_b,
                                 static_cast<u16*>(Xt), ld_xt, r, mean, m2, cl, st);
  return tokenize_stats_t<float>(static_cast<const float*>(X), B, C, T, ld_c, ld_b,
                                 static_cast<float*>(Xt), ld_xt, r, mean, m2, cl, st);
}

}  // namespace tdq
