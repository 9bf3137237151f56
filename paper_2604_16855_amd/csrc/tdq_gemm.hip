// W4A4 contraction on the int8 matrix cores of gfx950 with the dequantizing
// epilogue (Supp. Algorithm 1, step 10, written on the integer codes):
//   acc[m, n] = sum_i Qx[m, i] * Qw[n, i]            (int32, exact)
//   Y[m, n]   = (float(acc) * Delta[row m]) * s_w[n] (+ bias[n])
//
// Both operands arrive as packed two's-complement nibbles, K-contiguous.  The
// packed bytes are staged through LDS as they are (half the LDS traffic of int8)
// and expanded in registers: for a 32-bit word w of eight nibbles,
//   (w << 4) & 0xF0F0F0F0  holds the even elements and  w & 0xF0F0F0F0  the odd
// ones, each as an int8 equal to 16 * code (the sign lands in the byte's top bit
// for free).  Both operands carry the factor 16, so the int32 accumulator is
// 256 * acc and an arithmetic shift by 8 recovers acc exactly.  The order in
// which the K elements meet inside the matrix instruction is irrelevant as long
// as both operands use the same one, which they do by construction.
#include <stdlib.h>

#include <type_traits>

#include "tdq_internal.hpp"

namespace tdq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned int u32;

constexpr int BKB = 64;          // packed bytes of K per stage (128 codes)
constexpr int LDS_STRIDE = BKB + 16;   // +16 B pad: 16-byte reads of 8 rows hit 8 different bank groups
constexpr int GEMM_THREADS = 256;      // 4 wavefronts, 2 x 2
constexpr int XCDS = 8;

// Two packed words (16 codes) -> the four operand registers of one matrix instruction.
// `hi` is 0xF0F0F0F0; the pipelined kernel passes it in a scalar register so that the
// four ANDs are 4-byte instructions instead of 8-byte ones carrying a literal.
__device__ __forceinline__ v4i expand(u32 w0, u32 w1, u32 hi = 0xF0F0F0F0u) {
  v4i r;
  r[0] = (int)((w0 << 4) & hi);   // even codes of w0, times 16
  r[1] = (int)(w0 & hi);          // odd codes of w0, times 16
  r[2] = (int)((w1 << 4) & hi);
  r[3] = (int)(w1 & hi);
  return r;
}

// Keeps the first `keep` (1..15) bytes of a 16-byte piece and zeroes the rest.
__device__ __forceinline__ u32 tail_mask(int keep, int lo) {
  return keep >= lo + 4 ? 0xFFFFFFFFu : keep <= lo ? 0u : (0xFFFFFFFFu >> (8 * (lo + 4 - keep)));
}
__device__ __forceinline__ void mask_piece(uint4& q, int keep) {
  q.x &= tail_mask(keep, 0);
  q.y &= tail_mask(keep, 4);
  q.z &= tail_mask(keep, 8);
  q.w &= tail_mask(keep, 12);
}

template <typename OUT>
__device__ __forceinline__ void store_out(OUT* p, float v);
// Y is written once and not read again by this kernel: non-temporal stores keep the
// output stream from evicting the packed operands (above all the weights, which every
// tile re-reads) out of the L2.  Measured on the 131072 x 1024 x 4096 shape: plain
// stores cost 12 % (binary16 out) to 23 % (binary32 out) more time.  A non-temporal
// store that leaves part of a 128-byte line unwritten is expensive on the memory side,
// so the callers order their stores to complete lines within a few instructions.
template <>
__device__ __forceinline__ void store_out<float>(float* p, float v) {
  __builtin_nontemporal_store(v, p);
}
template <>
__device__ __forceinline__ void store_out<_Float16>(_Float16* p, float v) {
  // v is the binary32 result; it is rounded to binary16 in a second, separate step.
  // The empty asm keeps the compiler from merging the last binary32 operation with the
  // conversion into one mixed-precision instruction, which would round only once.
  asm volatile("" : "+v"(v));
  __builtin_nontemporal_store((_Float16)v, p);
}

typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
// Two binary32 results -> two binary16 values with one packed conversion (round to
// nearest even, as the scalar one).  As in store_out, the empty asm keeps the last
// binary32 operations from being merged with the conversion into mixed-precision
// instructions that would round only once.
__device__ __forceinline__ h2v round_pair_to_half(float a, float b) {
  asm volatile("" : "+v"(a), "+v"(b));
  const f2v v = {a, b};
  return __builtin_convertvector(v, h2v);
}

// 16 bytes of consecutive outputs with one store (p aligned to 16 bytes).
template <typename OUT>
struct OutVec;
template <>
struct OutVec<float> { static constexpr int W = 4; };
template <>
struct OutVec<_Float16> { static constexpr int W = 8; };
template <typename OUT>
__device__ __forceinline__ void store_out_vec(OUT* p, const float (&y)[OutVec<OUT>::W]);
template <>
__device__ __forceinline__ void store_out_vec<float>(float* p, const float (&y)[4]) {
  typedef float f4v __attribute__((ext_vector_type(4)));
  const f4v v = {y[0], y[1], y[2], y[3]};
  __builtin_nontemporal_store(v, reinterpret_cast<f4v*>(p));
}
template <>
__device__ __forceinline__ void store_out_vec<_Float16>(_Float16* p, const float (&y)[8]) {
  typedef _Float16 h8v __attribute__((ext_vector_type(8)));
  const h2v a = round_pair_to_half(y[0], y[1]), b = round_pair_to_half(y[2], y[3]);
  const h2v c = round_pair_to_half(y[4], y[5]), d = round_pair_to_half(y[6], y[7]);
  const h8v v = {a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
  __builtin_nontemporal_store(v, reinterpret_cast<h8v*>(p));
}

// STREAM: past the caches, as nothing reads it here again.
template <bool STREAM, typename V>
__device__ __forceinline__ void store_as(V v, V* p) {
  if constexpr (STREAM)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

// The first `rows` of 32 rows and `cols` of 64 columns of results, staged in LDS by the wavefront, to rows that
// need not start or end on 16-byte boundaries: neighbouring lanes take neighbouring outputs, with few columns of
// several rows, so that an instruction writes runs of lines, and whole groups of rows without a branch per row.
// (A run of outputs per lane instead, stored one by one, leaves every line in pieces to several instructions:
// 124818 x 32 x 803 by k_w4a4_gemm_blocks, binary16, 877 us, 75 so; 32768 x 1024 x 4095 by k_w4a4_gemm_blocks_f6
// 913 and 285.  A branch per row, as `rows` may end anywhere, 94 and 286, and 8.7 instead of 7.1 at 71 x 78 x 882.)
template <bool STREAM, typename OUT, typename GET>
__device__ __forceinline__ void store_rows(OUT* __restrict__ y, long long ld_y, int rows, int cols, int lane,
                                           GET&& get) {
  if (cols <= 0) return;
  const int lg = cols > 32 ? 6 : 32 - __clz(cols - 1 | 1);     // 2^lg lanes a row
  const int step = 64 >> lg, sub = lane >> lg, col = lane & ((1 << lg) - 1);
  const int limit = rows < 32 ? rows : 32;
  if (col >= cols) return;
  OUT* to = y + sub * ld_y + col;
  int r0 = 0;
#pragma unroll 1
  for (; r0 + 8 * step <= limit; r0 += 8 * step, to += 8 * step * ld_y) {
    OUT v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = get(r0 + k * step + sub, col);
#pragma unroll
    for (int k = 0; k < 8; ++k) store_as<STREAM>(v[k], to + k * step * ld_y);
  }
#pragma unroll 1
  for (int row = r0 + sub; row < limit; row += step, to += step * ld_y)
    store_as<STREAM>(get(row, col), to);
}

// Wavefront tile = 64 x 64 of Y, workgroup = 2 x 2 wavefronts, stages through registers: for
// products of long K whose shape does not suit 256 x 256 tiles (the dispatcher says where).
template <typename OUT>
__global__ __launch_bounds__(GEMM_THREADS, 3) void k_w4a4_gemm(
    const uint8_t* __restrict__ Qx, long long ld_q, const int* __restrict__ gid,
    const float* __restrict__ scale, int M, int T, int K, int N, int G,
    const uint8_t* __restrict__ Qw, long long ld_w, const float* __restrict__ w_scale,
    const float* __restrict__ bias, OUT* __restrict__ Y, long long ld_y, int* __restrict__ acc_dump,
    int m_tiles, int n_tiles) {
  constexpr int MT = 2, NT = 2, BM = 64 * MT, BN = 64 * NT;
  __shared__ __attribute__((aligned(16))) uint8_t sA[2][BM * LDS_STRIDE];
  __shared__ __attribute__((aligned(16))) uint8_t sB[2][BN * LDS_STRIDE];
  __shared__ float sRow[BM], sCol[BN], sBias[BN];

  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: give
  // every XCD whole rows of tiles so the activation tile it streams is reused by
  // consecutive workgroups of the same XCD.
  const int bid = blockIdx.x;
  const int xcd = bid % XCDS, idx = bid / XCDS;
  const int m_tile = (idx / n_tiles) * XCDS + xcd;
  const int n_tile = idx % n_tiles;
  if (m_tile >= m_tiles) return;
  const int m0 = m_tile * BM, n0 = n_tile * BN;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int kbytes = (K + 1) / 2;
  const int k_tiles = (kbytes + BKB - 1) / BKB;

  for (int i = tid; i < BM; i += GEMM_THREADS) {
    const int m = m0 + i;
    float rs = 0.f;
    if (m < M) {
      const int b = m / T;
      const int g = gid ? gid[m] : 0;
      rs = scale[(long long)b * G + g];
    }
    sRow[i] = rs;
  }
  for (int j = tid; j < BN; j += GEMM_THREADS) {
    const int n = n0 + j;
    sCol[j] = n < N ? w_scale[n] : 0.f;
    sBias[j] = (bias && n < N) ? bias[n] : 0.f;
  }

  // global -> register staging: a stage is BM (BN) rows x 64 B per operand, moved
  // as 16-byte pieces; thread t owns column piece (t & 3) of rows (t >> 2) + 64 i.
  const int pr0 = tid >> 2, pc = (tid & 3) * 16;
  const uint8_t* pa[MT];
  const uint8_t* pb[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    int r = m0 + pr0 + 64 * i;
    r = r < M ? r : M - 1;
    pa[i] = Qx + (long long)r * ld_q + pc;
  }
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    int r = n0 + pr0 + 64 * j;
    r = r < N ? r : N - 1;
    pb[j] = Qw + (long long)r * ld_w + pc;
  }
  uint4 ga[MT], gb[NT];
  auto load_stage = [&](int kt) {
    const int kb = kt * BKB + pc;          // first packed byte of this piece
    if (kb < kbytes) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
        ga[i] = *reinterpret_cast<const uint4*>(pa[i] + (long long)kt * BKB);
#pragma unroll
      for (int j = 0; j < NT; ++j)
        gb[j] = *reinterpret_cast<const uint4*>(pb[j] + (long long)kt * BKB);
      if (kb + 16 > kbytes) {              // piece straddles the end of the row: zero the rest
        const int keep = kbytes - kb;      // 1..15 bytes are real
#pragma unroll
        for (int i = 0; i < MT; ++i) mask_piece(ga[i], keep);
#pragma unroll
        for (int j = 0; j < NT; ++j) mask_piece(gb[j], keep);
      }
    } else {
#pragma unroll
      for (int i = 0; i < MT; ++i) ga[i] = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < NT; ++j) gb[j] = make_uint4(0, 0, 0, 0);
    }
  };
  auto store_stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
      *reinterpret_cast<uint4*>(&sA[buf][(pr0 + 64 * i) * LDS_STRIDE + pc]) = ga[i];
#pragma unroll
    for (int j = 0; j < NT; ++j)
      *reinterpret_cast<uint4*>(&sB[buf][(pr0 + 64 * j) * LDS_STRIDE + pc]) = gb[j];
  };

  v16i acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

  load_stage(0);
  store_stage(0);
  __syncthreads();

  // Lane l of a wavefront feeds row (l & 31) of a 32-row fragment and, of each
  // 32-byte slab (64 codes) of K, the 16 bytes at offset 16 * (l >> 5).
  const int frow = lane & 31, fhalf = (lane >> 5) * 16;
  const int a_off = (wm * 32 * MT + frow) * LDS_STRIDE + fhalf;
  const int b_off = (wn * 32 * NT + frow) * LDS_STRIDE + fhalf;
  for (int kt = 0; kt < k_tiles; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < k_tiles) load_stage(kt + 1);
#pragma unroll
    for (int ks = 0; ks < BKB / 32; ++ks) {
      uint4 fa[MT], fb[NT];
#pragma unroll
      for (int i = 0; i < MT; ++i)
        fa[i] = *reinterpret_cast<const uint4*>(&sA[cur][a_off + i * 32 * LDS_STRIDE + ks * 32]);
#pragma unroll
      for (int j = 0; j < NT; ++j)
        fb[j] = *reinterpret_cast<const uint4*>(&sB[cur][b_off + j * 32 * LDS_STRIDE + ks * 32]);
      v4i a0[MT], a1[MT], b0[NT], b1[NT];
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        a0[i] = expand(fa[i].x, fa[i].y);
        a1[i] = expand(fa[i].z, fa[i].w);
      }
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        b0[j] = expand(fb[j].x, fb[j].y);
        b1[j] = expand(fb[j].z, fb[j].w);
      }
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0[i], b0[j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1[i], b1[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < k_tiles) store_stage(cur ^ 1);
    __syncthreads();
  }

  // Epilogue.  Register r of a 32x32 accumulator fragment held by lane l is
  // element (row 8*(r/4) + 4*(l/32) + r%4, column l%32).
  const int ccol = lane & 31, rquad = (lane >> 5) * 4;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int cl = wn * 32 * NT + j * 32 + ccol;
      const int n = n0 + cl;
      const float ws = sCol[cl], bs = sBias[cl];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = wm * 32 * MT + i * 32 + (r >> 2) * 8 + rquad + (r & 3);
        const int m = m0 + rl;
        if (m < M && n < N) {
          const int a = acc[i][j][r] >> 8;            // exact: accumulator is 256 * acc
          if (acc_dump) acc_dump[(long long)m * N + n] = a;
          float y = ((float)a * sRow[rl]) * ws;
          if (bias) y = y + bs;
          store_out<OUT>(Y + (long long)m * ld_y + n, y);
        }
      }
    }
}

// ---------------------------------------------------------------------------
// Software-pipelined kernel for large shapes (K a multiple of 128 codes).
//
// A wavefront owns (32 MT) x (32 NT) of Y; a workgroup is 2 x 2 wavefronts.
//   MT = NT = 4: 256 x 256 tile, 256 accumulator registers, one wavefront per SIMD:
//                nothing but the wavefront's own instruction stream hides latency.
//   (The template also builds 256 x 128 and 128 x 256 tiles with two workgroups per
//   CU; on the 131072-row shapes of the largest configuration they measured within
//   3 % of the square tile, slower on K = 4096, so the dispatcher does not use them.)
// The stream is laid out by hand in bundles of one or two matrix instructions, the
// six expand operations of ONE operand fragment of the NEXT operand set (3 vector
// ops per matrix op at MT = NT = 4, which the vector unit absorbs while the matrix
// unit is busy) and at most one LDS read or one global load.  Per stage of 128
// codes (4 half-slabs of MT + NT bundles):
//   X0: set 0 of slab 0 | expand set 1 of slab 0 | LDS reads of slab 1
//   Y0: set 1 of slab 0 | expand set 0 of slab 1 | direct-to-LDS loads of stage + 2
//   wait for stage + 1, barrier
//   X1: set 0 of slab 1 | expand set 1 of slab 1 | LDS reads of slab 0 of stage + 1
//   Y1: set 1 of slab 1 | expand set 0 of that slab
//
// The activations are the row operand of the matrix instruction, so the 32 lanes of
// a half-wavefront hold 32 consecutive columns of one row of Y and every store
// instruction writes whole 128-byte (fp32) / 64-byte (fp16) row segments.  (With
// the operands swapped a lane would own 4 consecutive columns and could store 16
// bytes at once, but into 64 different rows per instruction: measured 40 % slower.)
//
// Stages arrive by direct-to-LDS loads (global_load_lds_dwordx4): no staging
// registers and no LDS write instructions in the wavefront's stream (an LDS write of
// 16 bytes per lane costs more than twice an LDS read of the same size on this
// chip), into a ring of three LDS slots so the loads run two stages ahead.
//
// LDS layout of a slot: rows of 64 bytes (4 pieces of 16), piece c of row r stored
// at position c ^ ((r >> 2) & 3): the 16-byte reads of 16 consecutive rows then
// fall on 16 different bank groups of the 64-bank LDS.  A direct load writes 64
// lanes x 16 bytes contiguously from the address in M0, so lane l of load i of
// wavefront w fills position l & 3 of row 64 i + 16 w + (l >> 2) and fetches the
// global piece that belongs there.
//
// These loads are issued from inline assembly, so the compiler neither sees that
// they write LDS nor counts them in vmcnt; the kernel waits for them itself: every
// stage issues exactly MT + NT per thread, hence "vmcnt(MT + NT)" = everything but
// the newest stage has landed.
// ---------------------------------------------------------------------------
template <int MT, int NT>
struct Frags {
  uint4 a[MT], b[NT];     // packed 16-byte pieces: .x .y feed operand set 0, .z .w set 1
};
template <int MT, int NT>
struct Operands {
  v4i a[MT], b[NT];
};

template <int SET, int MT, int NT>
__device__ __forceinline__ void expand_one(Operands<MT, NT>& dst, const Frags<MT, NT>& f, int e,
                                           u32 hi) {
  // e is a compile-time constant after unrolling
  if (e < MT) {
    dst.a[e] = SET == 0 ? expand(f.a[e].x, f.a[e].y, hi) : expand(f.a[e].z, f.a[e].w, hi);
  } else {
    dst.b[e - MT] = SET == 0 ? expand(f.b[e - MT].x, f.b[e - MT].y, hi)
                             : expand(f.b[e - MT].z, f.b[e - MT].w, hi);
  }
}

// MT * NT matrix instructions on `cur`, spread over MT + NT bundles, each with the
// expansion of one fragment of operand set EXP_SET from `f` into `nxt` and with
// mem(b), at most one memory instruction.
// One half (HALF = 0: words x / z -> elements 0, 1; HALF = 1: words y / w -> elements
// 2, 3) of the expansion of fragment e: three vector operations.
template <int SET, int HALF, int MT, int NT>
__device__ __forceinline__ void expand_half(Operands<MT, NT>& dst, const Frags<MT, NT>& f, int e,
                                            u32 hi) {
  const uint4& q = e < MT ? f.a[e] : f.b[e - MT];
  const u32 w = SET == 0 ? (HALF == 0 ? q.x : q.y) : (HALF == 0 ? q.z : q.w);
  v4i& d = e < MT ? dst.a[e] : dst.b[e - MT];
  d[2 * HALF] = (int)((w << 4) & hi);      // even codes of w, times 16
  d[2 * HALF + 1] = (int)(w & hi);         // odd codes of w, times 16
}

// MT * NT matrix instructions on `cur`, spread over MT + NT bundles, each with the
// expansion of one fragment of operand set EXP_SET from `f` into `nxt` and with
// mem(b), at most one memory instruction.  A wavefront issues in order, and a matrix
// instruction cannot start before the previous one has left the matrix pipe, so the
// vector work of a bundle is split between the shadows of its matrix instructions
// (matrix, three vector, matrix, three vector + memory) rather than queued behind both.
// ZERO: the matrix instructions start a fresh accumulation (C operand 0) instead of adding
// to acc: the first half-slab of a tile in a kernel that keeps its accumulators across tiles.
template <int EXP_SET, int MT, int NT, bool ZERO = false, typename MEM>
__device__ __forceinline__ void half_slab(v16i (&acc)[MT][NT], const Operands<MT, NT>& cur,
                                          Operands<MT, NT>& nxt, const Frags<MT, NT>& f, u32 hi,
                                          MEM mem) {
  constexpr int NB = MT + NT, NM = MT * NT;
  const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int lo = (b * NM) / NB, up = ((b + 1) * NM) / NB, mid = lo + (up - lo + 1) / 2;
#pragma unroll
    for (int m = lo; m < mid; ++m) {
      const int i = m / NT, j = m % NT;
      acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(cur.a[i], cur.b[j], ZERO ? zero : acc[i][j],
                                                        0, 0, 0);
    }
    expand_half<EXP_SET, 0>(nxt, f, b, hi);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = mid; m < up; ++m) {
      const int i = m / NT, j = m % NT;
      acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(cur.a[i], cur.b[j], ZERO ? zero : acc[i][j],
                                                        0, 0, 0);
    }
    expand_half<EXP_SET, 1>(nxt, f, b, hi);
    mem(b);
    __builtin_amdgcn_sched_barrier(0);
  }
}

__device__ __forceinline__ void dma16(const uint8_t* gptr, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(gptr), "s"(lds_base)
               : "memory");
}

// The same with a wavefront-uniform 64-bit base and a 32-bit per-lane byte offset.
__device__ __forceinline__ void dma16s(const uint8_t* base, unsigned off, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(base), "s"(lds_base)
               : "memory");
}

// 64 floats from 64 addresses -> 64 consecutive floats of LDS
__device__ __forceinline__ void dma4s(const float* sbase, unsigned voff, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
               :
               : "v"(voff), "s"(sbase), "s"(lds_base)
               : "memory");
}

// Output of a wavefront's (32 MT) x (32 NT) part of a tile that lies wholly inside Y:
// y = (float(acc) * row scale) * column scale (+ bias), each product rounded to binary32.
// Register r of a 32x32 accumulator fragment held by lane l is element
// (row 8*(r/4) + 4*(l/32) + r%4, column l%32).  Every address is a wavefront-uniform row
// pointer plus one per-lane 32-bit offset.  wtile = &Y[first row][first column] of the
// wavefront's part.  EDGE: only the first `rows` of its rows and
// `cols` of its columns are stored (by masks).
template <typename OUT, int MT, int NT, typename ACC, bool BIAS, bool EDGE = false, bool STREAM = true>
__device__ __forceinline__ void tile_store_fast(ACC (&acc)[MT][NT], const float* sRow,
                                                const float* sCol, const float* sBias, int lane,
                                                int wm, int wn, OUT* __restrict__ wtile,
                                                long long ld_y, int rows = 32 * MT, int cols = 32 * NT) {
  const int ccol = lane & 31, rquad = (lane >> 5) * 4;
  bool in[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) in[j] = !EDGE || j * 32 + ccol < cols;
  const unsigned lane_offu = (unsigned)(rquad * (int)ld_y + ccol);
  float ws[NT], bs[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    ws[j] = sCol[wn * 32 * NT + j * 32 + ccol];
    bs[j] = sBias[wn * 32 * NT + j * 32 + ccol];
  }
#pragma unroll
  for (int i = 0; i < MT; ++i) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 rs4 =
          *reinterpret_cast<const float4*>(&sRow[wm * 32 * MT + i * 32 + q * 8 + rquad]);
      const float rsv[4] = {rs4.x, rs4.y, rs4.z, rs4.w};
      // Two rows at a time.  The NT column blocks of one row are stored back to back:
      // together they cover whole cache lines of Y, written within a few instructions of
      // each other.
#pragma unroll
      for (int t = 0; t < 4; t += 2) {
        OUT* row0 = wtile + (long long)(i * 32 + q * 8 + t) * ld_y + lane_offu;   // uniform + lane
        const bool in0 = !EDGE || i * 32 + q * 8 + t + rquad < rows, in1 = !EDGE || i * 32 + q * 8 + t + 1 + rquad < rows;
        OUT* row1 = row0 + ld_y;
        float y0[NT], y1[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const auto a0 = acc[i][j][4 * q + t], a1 = acc[i][j][4 * q + t + 1];
          y0[j] = ((float)a0 * rsv[t]) * ws[j];
          y1[j] = ((float)a1 * rsv[t + 1]) * ws[j];
          if (BIAS) {
            y0[j] = y0[j] + bs[j];
            y1[j] = y1[j] + bs[j];
          }
        }
        if constexpr (sizeof(OUT) == 2) {
          // one packed conversion rounds the two rows' binary32 results to binary16
          h2v p[NT];
#pragma unroll
          for (int j = 0; j < NT; ++j) p[j] = round_pair_to_half(y0[j], y1[j]);
#pragma unroll
          for (int j = 0; j < NT; ++j)
            if (in[j] && in0) store_as<STREAM>((_Float16)p[j][0], row0 + j * 32);
#pragma unroll
          for (int j = 0; j < NT; ++j)
            if (in[j] && in1) store_as<STREAM>((_Float16)p[j][1], row1 + j * 32);
        } else {
#pragma unroll
          for (int j = 0; j < NT; ++j)
            if (in[j] && in0) store_as<STREAM>(y0[j], row0 + j * 32);
#pragma unroll
          for (int j = 0; j < NT; ++j)
            if (in[j] && in1) store_as<STREAM>(y1[j], row1 + j * 32);
        }
      }
    }
  }
}

// Output phase of the persistent kernel.  Its weight rows are dealt to the column blocks so
// that column block j of a wavefront holds output columns 4 c + j (c = lane % 32): the four
// accumulators acc[i][0..3][r] of a lane are then four ADJACENT outputs of one row, and a lane
// stores them with one instruction (8 bytes of binary16, 16 of binary32) -- 64 stores per
// wavefront and tile instead of 256, each completing 256 or 512 contiguous bytes of two rows.
// y = (float(acc) * row scale) * (column scale * 2^-8) (+ bias): the 2^-8 that takes the 256
// out of the int8 accumulators rides on the column scale (a power of two: the same bits).
// The accumulators are read where they are used and the scheduler may not move code across
// rows, which keeps the registers this needs at any one time to a few dozen.  The stores are
// the compiler's own (non-temporal, see store_out): a 16-byte store reads its data registers
// over several cycles and the compiler, not inline assembly, knows how long to keep them.
typedef float f4v __attribute__((ext_vector_type(4)));
typedef unsigned u2v __attribute__((ext_vector_type(2)));
template <typename OUT, bool BIAS>
__device__ __forceinline__ void tile_store_cols4(v16i (&acc)[4][4], const float* sRow, const float* sCol,
                                                 const float* sBias, int lane, int wm, int wn,
                                                 const OUT* __restrict__ wtile, long long ld_y) {
  const int ccol = lane & 31, rquad = (lane >> 5) * 4;
  // byte offset of the lane inside the wavefront's 128 rows; 132 rows of ld_y elements fit 32 bits (host)
  const unsigned lane_off = (unsigned)(rquad * (int)ld_y + 4 * ccol) * (unsigned)sizeof(OUT);
  const float4 w4 = *reinterpret_cast<const float4*>(&sCol[wn * 128 + 4 * ccol]);
  const float4 b4 = *reinterpret_cast<const float4*>(&sBias[wn * 128 + 4 * ccol]);
  const float ws[4] = {w4.x * 0.00390625f, w4.y * 0.00390625f, w4.z * 0.00390625f, w4.w * 0.00390625f};
  const float bs[4] = {b4.x, b4.y, b4.z, b4.w};
  // Every instruction of a lone wavefront costs an issue slot here (nothing else runs on the
  // SIMD during the output phase), so the store address costs one vector add per row: scalar
  // base of the wavefront's part of the tile + a 32-bit lane offset that walks down the rows
  // (rows 0-3, 8-11, ... of every 32: steps of one row and of five).
  typedef __attribute__((address_space(1))) char gchar;
  gchar* const base = reinterpret_cast<gchar*>(reinterpret_cast<unsigned long long>(wtile));
  unsigned voff = lane_off;
  const unsigned step1 = (unsigned)ld_y * (unsigned)sizeof(OUT), step5 = 5u * step1;
  // The four row scales of a group of four rows are read from LDS one group ahead: a lone
  // wavefront has nothing else to run while it waits for an LDS read.  The accumulators of a
  // row are copied out of the accumulation registers one row ahead, between the previous
  // row's last binary32 operation and its conversion / store: the instruction after an asm
  // statement then never reads what the statement wrote, and no wait state is inserted.
  const float* rs_src = sRow + wm * 128 + rquad;
  float4 rs_next = *reinterpret_cast<const float4*>(rs_src);
  int a_cur[4], a_nxt[4] = {0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < 4; ++j) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(a_cur[j]) : "a"(acc[0][j][0]));
#pragma unroll
  for (int g = 0; g < 16; ++g) {                   // row group g: rows 8 g .. 8 g + 3 (+ 4 for the upper lanes)
    const float rsv[4] = {rs_next.x, rs_next.y, rs_next.z, rs_next.w};
    if (g + 1 < 16) rs_next = *reinterpret_cast<const float4*>(rs_src + (g + 1) * 8);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float y[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        y[j] = ((float)a_cur[j] * rsv[t]) * ws[j];
        if (BIAS) y[j] = y[j] + bs[j];
      }
      __builtin_amdgcn_sched_barrier(0);
      const int r2 = 4 * g + t + 1;                // the next row's accumulators
      const int i2 = (r2 >> 4) & 3, q2 = (r2 >> 2) & 3, t2 = r2 & 3;
      if constexpr (sizeof(OUT) == 2) {
        // One asm statement copies the next row's accumulators out and rounds this row's pairs
        // of binary32 results to binary16 (packed conversion, to nearest even): the conversion
        // cannot be merged with the multiplication before it into a mixed-precision
        // instruction that would round only once, and the instruction after the statement --
        // the next row's address -- reads nothing the statement wrote.
        u2v v;
        if (r2 < 64)
          asm volatile(
              "v_accvgpr_read_b32 %2, %10\n\tv_accvgpr_read_b32 %3, %11\n\t"
              "v_accvgpr_read_b32 %4, %12\n\tv_accvgpr_read_b32 %5, %13\n\t"
              "v_cvt_pk_f16_f32 %0, %6, %7\n\tv_cvt_pk_f16_f32 %1, %8, %9"
              : "=&v"(v.x), "=&v"(v.y), "=&v"(a_nxt[0]), "=&v"(a_nxt[1]), "=&v"(a_nxt[2]), "=&v"(a_nxt[3])
              : "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3]), "a"(acc[i2][0][4 * q2 + t2]),
                "a"(acc[i2][1][4 * q2 + t2]), "a"(acc[i2][2][4 * q2 + t2]), "a"(acc[i2][3][4 * q2 + t2]));
        else
          asm volatile("v_cvt_pk_f16_f32 %0, %2, %3\n\tv_cvt_pk_f16_f32 %1, %4, %5"
                       : "=&v"(v.x), "=&v"(v.y)
                       : "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3]));
        __builtin_amdgcn_sched_barrier(0);
        const unsigned voff_next = voff + (t == 3 ? step5 : step1);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_nontemporal_store(v, reinterpret_cast<__attribute__((address_space(1))) u2v*>(base + voff));
        voff = voff_next;
      } else {
        if (r2 < 64) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(a_nxt[j]) : "a"(acc[i2][j][4 * q2 + t2]));
        }
        __builtin_amdgcn_sched_barrier(0);
        const f4v v = {y[0], y[1], y[2], y[3]};
        __builtin_nontemporal_store(v, reinterpret_cast<__attribute__((address_space(1))) f4v*>(base + voff));
        voff += t == 3 ? step5 : step1;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) a_cur[j] = a_nxt[j];
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Epilogue of the pipelined kernels.  Register r of a 32x32 accumulator fragment held
// by lane l is element (row 8*(r/4) + 4*(l/32) + r%4, column l%32).
template <typename OUT, int MT, int NT, typename ACC = v16i, bool KEEP = false>
__device__ __forceinline__ void pipe_epilogue(ACC (&acc)[MT][NT], const float* sRow,
                                              const float* sCol, const float* sBias, int lane,
                                              int wm, int wn, int m0, int n0, int M, int N,
                                              const float* __restrict__ bias, OUT* __restrict__ Y,
                                              long long ld_y, int* __restrict__ acc_dump) {
  constexpr int BM = 64 * MT;
  const int ccol = lane & 31, rquad = (lane >> 5) * 4;
  // Of a tile at an edge of Y each wavefront decides for itself: nothing of it inside, all of it, a
  // part of it.  KEEP: those of a tile cut in its columns all store by masks, and not past the caches.
  // (The whole tile by the path with two checks per output, and so, us: 12000 x 200 x 1000 binary32 16.9 and 14.3, 5000 x
  // 96 x 2000 binary16 10.6 and 8.8, 20000 x 77 x 333 8.8 and 7.3, 6845 x 333 x 777 binary32 9.9 and 9.2.)
  const int rows = M - (m0 + wm * 32 * MT), cols = N - (n0 + wn * 32 * NT);
  if (rows <= 0 || cols <= 0) return;
  if (!acc_dump && (long long)(BM + 8) * ld_y < (1ll << 31) / (long long)sizeof(OUT)) {
    OUT* wtile = Y + (long long)(m0 + wm * 32 * MT) * ld_y + (n0 + wn * 32 * NT);
    if (rows >= 32 * MT && cols >= 32 * NT && (!KEEP || n0 + 64 * NT <= N)) {
      if (bias)
        tile_store_fast<OUT, MT, NT, ACC, true>(acc, sRow, sCol, sBias, lane, wm, wn, wtile, ld_y);
      else
        tile_store_fast<OUT, MT, NT, ACC, false>(acc, sRow, sCol, sBias, lane, wm, wn, wtile, ld_y);
      return;
    }
    if constexpr (MT * NT <= 4) {
      if (bias)
        tile_store_fast<OUT, MT, NT, ACC, true, true, !KEEP>(acc, sRow, sCol, sBias, lane, wm, wn, wtile, ld_y, rows, cols);
      else
        tile_store_fast<OUT, MT, NT, ACC, false, true, !KEEP>(acc, sRow, sCol, sBias, lane, wm, wn, wtile, ld_y, rows, cols);
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int cl = wn * 32 * NT + j * 32 + ccol;
      const int n = n0 + cl;
      const float ws = sCol[cl], bs = sBias[cl];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rl = wm * 32 * MT + i * 32 + (r >> 2) * 8 + rquad + (r & 3);
        const int m = m0 + rl;
        if (m < M && n < N) {
          float y;
          if (acc_dump) {
            int a;
            if constexpr (std::is_same<ACC, v16i>::value) a = acc[i][j][r] >> 8;   // exact: 256 * acc
            else a = (int)acc[i][j][r];                                          // exact integer
            acc_dump[(long long)m * N + n] = a;
            y = ((float)a * sRow[rl]) * ws;
          } else {
            y = ((float)acc[i][j][r] * sRow[rl]) * ws;
          }
          if (bias) y = y + bs;
          store_out<OUT>(Y + (long long)m * ld_y + n, y);
        }
      }
    }
}

template <typename OUT, int MT, int NT>
__global__ __launch_bounds__(GEMM_THREADS, (MT * NT >= 16 ? 1 : 2)) void k_w4a4_gemm_pipe(
    const uint8_t* __restrict__ Qx, long long ld_q, const int* __restrict__ gid,
    const float* __restrict__ scale, int M, int T, int K, int N, int G,
    const uint8_t* __restrict__ Qw, long long ld_w, const float* __restrict__ w_scale,
    const float* __restrict__ bias, OUT* __restrict__ Y, long long ld_y, int* __restrict__ acc_dump,
    int m_tiles, int n_tiles) {
  constexpr int BM = 64 * MT, BN = 64 * NT, NB = MT + NT;
  constexpr int SLOT = (BM + BN) * BKB;      // bytes of one ring slot: A rows then B rows, 64 B each
  __shared__ __attribute__((aligned(1024))) uint8_t ring[3 * SLOT];
  __shared__ __attribute__((aligned(16))) float sRow[BM], sCol[BN], sBias[BN];

  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: give
  // every XCD whole rows of tiles so the activation tile it streams is reused by
  // consecutive workgroups of the same XCD.
  const int bid = blockIdx.x;
  const int xcd = bid % XCDS, idx = bid / XCDS;
  const int m_tile = (idx / n_tiles) * XCDS + xcd;
  const int n_tile = idx % n_tiles;
  if (m_tile >= m_tiles) return;
  const int m0 = m_tile * BM, n0 = n_tile * BN;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int k_tiles = ((K + 1) / 2) / BKB;          // host guarantees K % 128 == 0

  // Scales of the epilogue.  The token-set ids are fetched first; the scales that
  // depend on them are fetched after the first stages' loads have been issued, so
  // the latencies overlap.
  int my_m[(BM + GEMM_THREADS - 1) / GEMM_THREADS], my_g[(BM + GEMM_THREADS - 1) / GEMM_THREADS];
#pragma unroll
  for (int u = 0; u < (BM + GEMM_THREADS - 1) / GEMM_THREADS; ++u) {
    const int m = m0 + tid + u * GEMM_THREADS;
    my_m[u] = m < M ? m : M - 1;
    my_g[u] = gid ? gid[my_m[u]] : 0;
  }

  // global source of this lane's piece of load i (rows 64 i + 16 w + (l >> 2))
  const uint8_t* pa[MT];
  const uint8_t* pb[NT];
  {
    const int rl0 = 16 * wave + (lane >> 2);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int rl = 64 * i + rl0;                            // row inside the tile
      const int c = (lane & 3) ^ ((rl >> 2) & 3);             // logical piece stored at position l & 3
      int r = m0 + rl;
      r = r < M ? r : M - 1;
      pa[i] = Qx + (long long)r * ld_q + c * 16;
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int rl = 64 * i + rl0;
      const int c = (lane & 3) ^ ((rl >> 2) & 3);
      int n = n0 + rl;
      n = n < N ? n : N - 1;
      pb[i] = Qw + (long long)n * ld_w + c * 16;
    }
  }
  const unsigned ring_base =
      (unsigned)(size_t)(__attribute__((address_space(3))) uint8_t*)ring;
  const unsigned dma_base = __builtin_amdgcn_readfirstlane(ring_base + wave * 1024);
  auto dma_piece = [&](int slot, int kt, int e) {     // slot, e compile-time; e = 0 .. NB-1
    const int kc = kt < k_tiles ? kt : k_tiles - 1;    // past the end: harmless re-load
    const long long ko = (long long)kc * BKB;
    if (e < MT)
      dma16(pa[e] + ko, dma_base + slot * SLOT + e * 4096);
    else
      dma16(pb[e - MT] + ko, dma_base + slot * SLOT + BM * BKB + (e - MT) * 4096);
  };

  // fragment reads: lane (row r' = l & 31, half h = l >> 5) of fragment e reads piece
  // 2 ks + h of row 32 e + r' (+ the wavefront's offset); the swizzle only depends on r'
  const int frow = lane & 31, fh = lane >> 5, swz = (frow >> 2) & 3;
  const int a_row = (wm * 32 * MT + frow) * 64, b_row = BM * BKB + (wn * 32 * NT + frow) * 64;
  const int off_k0 = ((0 + fh) ^ swz) * 16, off_k1 = ((2 + fh) ^ swz) * 16;
  auto read_piece = [&](Frags<MT, NT>& f, int slot, int ks, int e) {   // slot, ks, e compile-time
    const int off = ks == 0 ? off_k0 : off_k1;
    if (e < MT)
      f.a[e] = *reinterpret_cast<const uint4*>(&ring[slot * SLOT + a_row + e * 2048 + off]);
    else
      f.b[e - MT] =
          *reinterpret_cast<const uint4*>(&ring[slot * SLOT + b_row + (e - MT) * 2048 + off]);
  };

  v16i acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
  Frags<MT, NT> f0, f1;
  Operands<MT, NT> s0, s1;
  u32 hi;                                   // 0xF0F0F0F0 in a scalar register
  asm volatile("s_mov_b32 %0, 0xf0f0f0f0" : "=s"(hi));
#pragma unroll
  for (int e = 0; e < NB; ++e) dma_piece(0, 0, e);
#pragma unroll
  for (int e = 0; e < NB; ++e) dma_piece(1, 1, e);
#pragma unroll
  for (int u = 0; u < (BM + GEMM_THREADS - 1) / GEMM_THREADS; ++u) {
    const int i = tid + u * GEMM_THREADS;
    if (i < BM) {
      const float rs = scale[(long long)(my_m[u] / T) * G + my_g[u]];
      // the accumulators carry a factor 256; folding 2^-8 into the row scale is exact
      sRow[i] = acc_dump ? rs : rs * 0.00390625f;
    }
  }
  for (int j = tid; j < BN; j += GEMM_THREADS) {
    const int n = n0 + j;
    sCol[j] = n < N ? w_scale[n] : 0.f;
    sBias[j] = (bias && n < N) ? bias[n] : 0.f;
  }
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NB) : "memory");      // stage 0 has landed
  __syncthreads();
#pragma unroll
  for (int e = 0; e < NB; ++e) read_piece(f0, 0, 0, e);
#pragma unroll
  for (int e = 0; e < NB; ++e) expand_one<0>(s0, f0, e, hi);

  // One stage: CUR holds stage kt, NXT stage kt + 1 (in flight until the barrier),
  // LD receives stage kt + 2 (the slot that held stage kt - 1).  The body is
  // branch-free so that its bundles stay in one scheduling region: stages past the
  // end re-load the last one into an idle slot that nobody reads.
#define TDQ_STAGE(kt, CUR, NXT, LD)                                                              \
  do {                                                                                           \
    __builtin_amdgcn_sched_barrier(0);                                                           \
    half_slab<1>(acc, s0, s1, f0, hi, [&](int b) { read_piece(f1, CUR, 1, b); });       /* X0 */ \
    half_slab<0>(acc, s1, s0, f1, hi, [&](int b) { dma_piece(LD, (kt) + 2, b); });      /* Y0 */ \
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NB) : "memory");                                    \
    __syncthreads();                                                                             \
    __builtin_amdgcn_sched_barrier(0);                                                           \
    half_slab<1>(acc, s0, s1, f1, hi, [&](int b) { read_piece(f0, NXT, 0, b); });       /* X1 */ \
    half_slab<0>(acc, s1, s0, f0, hi, [&](int) {});                                     /* Y1 */ \
  } while (0)

  int kt = 0;
  for (; kt + 2 < k_tiles; kt += 3) {
    TDQ_STAGE(kt, 0, 1, 2);
    TDQ_STAGE(kt + 1, 1, 2, 0);
    TDQ_STAGE(kt + 2, 2, 0, 1);
  }
  if (kt < k_tiles) TDQ_STAGE(kt, 0, 1, 2);
  if (kt + 1 < k_tiles) TDQ_STAGE(kt + 1, 1, 2, 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing of ours may still be landing
#undef TDQ_STAGE

  pipe_epilogue<OUT, MT, NT>(acc, sRow, sCol, sBias, lane, wm, wn, m0, n0, M, N, bias, Y, ld_y,
                             acc_dump);
}

// ---------------------------------------------------------------------------
// Kernel for the shapes that do not fill the chip with 256 x 256 tiles, and for any K.
// A workgroup is 2 x 2 wavefronts of (32 MT) x (32 NT) of Y, MT and NT 1 or 2; these layers
// are bound by latency (968 x 512 x 512: 11.3 us with the register-staged kernel's two
// buffers and scales fetched first, 4.8 here; 7744 x 320 x 1280, binary32: 16.0 and 12.5; 61952 x
// 512 x 64: 13.1 and 8.5), so the point is how many trips to memory follow one another:
//   * operands arrive by direct-to-LDS loads in stages of 64 bytes (128 codes) per row, a
//     ring of four slots, three stages in flight: all of a K of 384 at once, no staging
//     registers (LDS layout of a slot as in k_w4a4_gemm_pipe), and no more LDS than the
//     stages there are, so that a short K runs more workgroups per CU;
//   * the token-set ids are fetched with the first stages, the row scales that depend on
//     them while the matrix instructions run; they meet the accumulators through LDS after
//     the last stage;
//   * K tails: 16-byte pieces past the end of the rows are fetched from the row's first
//     piece instead and the activation fragments are masked to the bytes that count (a zero
//     in one operand is enough); the half of the last stage that no byte reaches is left out, and one that
//     is whole is not masked.  With several workgroups on a CU the loop takes what its instructions take, and
//     a masked stage has twice those of another (15488 x 320 x 640: 10.8 -> 9.4 us, 32768 x 320 x 1280 38.7 ->
//     35.2).  That stage stands behind the loop, so that the loop is whole stages only (8192 x 768 x 768 9.9 -> 9.5,
//     131072 x 1000 x 1024 176 -> 169).
// ---------------------------------------------------------------------------
// KEEP: how outputs are stored (launch_ring says when).
template <typename OUT, int MT, int NT, bool KEEP>
__global__ __launch_bounds__(GEMM_THREADS, (MT * NT >= 4 ? 2 : MT * NT >= 2 ? 3 : 6)) void k_w4a4_gemm_ring(
    const uint8_t* __restrict__ Qx, long long ld_q, const int* __restrict__ gid,
    const float* __restrict__ scale, int M, int T, int K, int N, int G,
    const uint8_t* __restrict__ Qw, long long ld_w, const float* __restrict__ w_scale,
    const float* __restrict__ bias, OUT* __restrict__ Y, long long ld_y, int* __restrict__ acc_dump,
    int m_tiles, int n_tiles) {
  constexpr int BM = 64 * MT, BN = 64 * NT, NL = MT + NT, D = 4;
  constexpr int SLOT = (BM + BN) * BKB;      // A rows then B rows, 64 B each
  extern __shared__ __attribute__((aligned(1024))) uint8_t ring[];        // min(D, stages) slots
  __shared__ __attribute__((aligned(16))) float sRow[BM], sCol[BN], sBias[BN];

  // whole rows of tiles per XCD, as in the other kernels
  const int bid = blockIdx.x;
  const int xcd = bid % XCDS, idx = bid / XCDS;
  const int m_tile = (idx / n_tiles) * XCDS + xcd;
  const int n_tile = idx % n_tiles;
  if (m_tile >= m_tiles) return;
  const int m0 = m_tile * BM, n0 = n_tile * BN;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int kbytes = (K + 1) / 2, row_bytes = 16 * ((K + 31) / 32);
  const int k_tiles = (kbytes + BKB - 1) / BKB;

  const int my_m = m0 + tid < M ? m0 + tid : M - 1;
  const int my_n = n0 + tid < N ? n0 + tid : N - 1;
  int my_g = 0;
  float my_ws = 0.f, my_bs = 0.f;
  if (tid < BM && gid) my_g = gid[my_m];
  if (tid < BN) {
    my_ws = w_scale[my_n];
    if (bias) my_bs = bias[my_n];
  }

  // load e of this wavefront fills 16 rows: block e * 4 + wave of the slot's BM / 16 blocks
  // of A and BN / 16 of B; lane l writes position l & 3 of row l >> 2
  const uint8_t* src[NL];
  const int brow = 16 * wave + (lane >> 2);
  const int piece = ((lane & 3) ^ ((brow >> 2) & 3)) * 16;      // (64 e rows further: the same)
#pragma unroll
  for (int e = 0; e < NL; ++e) {
    if (e < MT) {
      const int r = m0 + 64 * e + brow;
      src[e] = Qx + (long long)(r < M ? r : M - 1) * ld_q;
    } else {
      const int r = n0 + 64 * (e - MT) + brow;
      src[e] = Qw + (long long)(r < N ? r : N - 1) * ld_w;
    }
  }
  const unsigned ring_base = (unsigned)(size_t)(__attribute__((address_space(3))) uint8_t*)ring;
  const unsigned dma_base = __builtin_amdgcn_readfirstlane(ring_base + wave * 1024);
  auto load_stage = [&](int kt) {
    const int kb = kt * BKB + piece;
    const int off = kb < row_bytes ? kb : 0;                    // past the row's end: any piece of it
    const unsigned slot = dma_base + (unsigned)(kt & (D - 1)) * SLOT;
#pragma unroll
    for (int e = 0; e < NL; ++e) dma16(src[e] + off, slot + e * 4096);
  };
#pragma unroll
  for (int st = 0; st < D - 1; ++st)
    if (st < k_tiles) load_stage(st);
  float my_rs = 0.f;
  if (tid < BM) my_rs = scale[(long long)(my_m / T) * G + my_g];

  v16i acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

  const int frow = lane & 31, fh = lane >> 5, swz = (frow >> 2) & 3;
  const int a_row = (wm * 32 * MT + frow) * BKB, b_row = BM * BKB + (wn * 32 * NT + frow) * BKB;
  // halves KS0 and (if more than one) the next of a stage, 64 codes of K each; masked: `keep` bytes of the last count
  auto stage = [&](int kt, auto first, auto halves, bool masked, int keep) {
    const uint8_t* slot = ring + (kt & (D - 1)) * SLOT;
#pragma unroll
    for (int ks = decltype(first)::value; ks < decltype(first)::value + decltype(halves)::value; ++ks) {
      const int off = ((2 * ks + fh) ^ swz) * 16;
      uint4 fa[MT], fb[NT];
#pragma unroll
      for (int i = 0; i < MT; ++i) fa[i] = *reinterpret_cast<const uint4*>(slot + a_row + i * 32 * BKB + off);
#pragma unroll
      for (int j = 0; j < NT; ++j) fb[j] = *reinterpret_cast<const uint4*>(slot + b_row + j * 32 * BKB + off);
      if (masked) {
#pragma unroll
        for (int i = 0; i < MT; ++i) mask_piece(fa[i], keep - fh * 16);
      }
#pragma unroll
      for (int set = 0; set < 2; ++set) {
        v4i a[MT], b[NT];
#pragma unroll
        for (int i = 0; i < MT; ++i) a[i] = set == 0 ? expand(fa[i].x, fa[i].y) : expand(fa[i].z, fa[i].w);
#pragma unroll
        for (int j = 0; j < NT; ++j) b[j] = set == 0 ? expand(fb[j].x, fb[j].y) : expand(fb[j].z, fb[j].w);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], b[j], acc[i][j], 0, 0, 0);
      }
    }
  };
  typedef std::integral_constant<int, 0> C0;
  typedef std::integral_constant<int, 1> C1;
  typedef std::integral_constant<int, 2> C2;
  for (int kt = 0; kt < k_tiles; ++kt) {
    // stage kt has landed when at most the loads of the stages after it are outstanding
    const int newer = k_tiles - 1 - kt < D - 2 ? k_tiles - 1 - kt : D - 2;
    if (newer == 2)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NL) : "memory");
    else if (newer == 1)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // the slot of stage kt - 1: every wavefront drained its reads before this barrier
    if (kt + D - 1 < k_tiles) load_stage(kt + D - 1);
    if ((kt + 1) * BKB <= kbytes) stage(kt, C0(), C2(), false, 0);
  }
  // the last stage if it is not whole: the halves that hold something, masked if they are not whole either
  const int rest = kbytes - (k_tiles - 1) * BKB;                // uniform
  if (rest < BKB) {
    if (rest >= 32)
      stage(k_tiles - 1, C0(), C1(), false, 0);
    else
      stage(k_tiles - 1, C0(), C1(), true, rest);
    if (rest > 32) stage(k_tiles - 1, C1(), C1(), true, rest - 32);
  }

  if (tid < BM) sRow[tid] = acc_dump ? my_rs : my_rs * 0.00390625f;     // takes out the factor 256 (exact)
  if (tid < BN) {
    sCol[tid] = my_ws;
    sBias[tid] = my_bs;
  }
  __syncthreads();
  pipe_epilogue<OUT, MT, NT, v16i, KEEP>(acc, sRow, sCol, sBias, lane, wm, wn, m0, n0, M, N, bias, Y, ld_y, acc_dump);
}

// ---------------------------------------------------------------------------
// Wide-stage variant of the pipelined kernel (K a multiple of 256 codes): a stage is
// 128 bytes = one whole cache line of every operand row, so a line is fetched once
// (the 64-byte stages above fetch each line twice, two stages apart, and the L1
// cannot hold 512 lines in between), and the workgroup meets at one barrier per 256
// codes instead of two.  256 x 256 tile, 2 x 2 wavefronts of 4 x 4 blocks, two LDS
// slots of 64 KiB.  Per stage (4 slabs of 64 codes; Xs/Ys as above):
//   X0 | LDS reads of slab 1        Y0 | loads 8..15 of stage + 1
//   X1 | LDS reads of slab 2        Y1
//   X2 | LDS reads of slab 3        Y2
//   wait for stage + 1 (all of this thread's loads), barrier
//   X3 | LDS reads of slab 0 of stage + 1      Y3 | loads 0..7 of stage + 2
// The loads of stage + 2 go into the slot of the stage that is ending: its last
// fragment reads (slab 3) were issued before the barrier, and every wavefront drains
// its LDS reads before it arrives there.  LDS rows are 128 bytes, piece c of row r at
// position c ^ ((r >> 1) & 7): 16 consecutive rows fall on 16 different bank groups.
// ---------------------------------------------------------------------------
template <typename OUT>
__global__ __launch_bounds__(GEMM_THREADS, 1) void k_w4a4_gemm_wide(
    const uint8_t* __restrict__ Qx, long long ld_q, const int* __restrict__ gid,
    const float* __restrict__ scale, int M, int T, int K, int N, int G,
    const uint8_t* __restrict__ Qw, long long ld_w, const float* __restrict__ w_scale,
    const float* __restrict__ bias, OUT* __restrict__ Y, long long ld_y, int* __restrict__ acc_dump,
    int m_tiles, int n_tiles) {
  constexpr int MT = 4, NT = 4, BM = 256, BN = 256, NB = MT + NT;
  constexpr int BKW = 128;                     // packed bytes of K per stage (256 codes)
  constexpr int SLOT = (BM + BN) * BKW;        // 64 KiB: A rows then B rows, 128 B each
  __shared__ __attribute__((aligned(1024))) uint8_t ring[2 * SLOT];
  __shared__ __attribute__((aligned(16))) float sRow[BM], sCol[BN], sBias[BN];

  const int bid = blockIdx.x;
  const int xcd = bid % XCDS, idx = bid / XCDS;
  const int m_tile = (idx / n_tiles) * XCDS + xcd;
  const int n_tile = idx % n_tiles;
  if (m_tile >= m_tiles) return;
  const int m0 = m_tile * BM, n0 = n_tile * BN;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int k_tiles = (K / 2) / BKW;                // host guarantees K % 256 == 0

  const int my_m = m0 + tid < M ? m0 + tid : M - 1;
  const int my_g = gid ? gid[my_m] : 0;

  // global source of this lane's piece of load i: rows 32 i + 8 w + (l >> 3), 8 per load
  const uint8_t* pa[2 * MT];
  const uint8_t* pb[2 * NT];
  {
    const int rl0 = 8 * wave + (lane >> 3);
    const int c = (lane & 7) ^ ((rl0 >> 1) & 7);      // logical piece stored at position l & 7
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) {
      int r = m0 + 32 * i + rl0;
      r = r < M ? r : M - 1;
      pa[i] = Qx + (long long)r * ld_q + c * 16;
    }
#pragma unroll
    for (int i = 0; i < 2 * NT; ++i) {
      int n = n0 + 32 * i + rl0;
      n = n < N ? n : N - 1;
      pb[i] = Qw + (long long)n * ld_w + c * 16;
    }
  }
  const unsigned ring_base =
      (unsigned)(size_t)(__attribute__((address_space(3))) uint8_t*)ring;
  const unsigned dma_base = __builtin_amdgcn_readfirstlane(ring_base + wave * 1024);
  auto dma_piece = [&](int slot, int kt, int e) {     // slot, e compile-time; e = 0 .. 15
    const int kc = kt < k_tiles ? kt : k_tiles - 1;    // past the end: harmless re-load
    const long long ko = (long long)kc * BKW;
    if (e < 2 * MT)
      dma16(pa[e] + ko, dma_base + slot * SLOT + e * 4096);
    else
      dma16(pb[e - 2 * MT] + ko, dma_base + slot * SLOT + BM * BKW + (e - 2 * MT) * 4096);
  };

  // fragment reads: lane (row r' = l & 31, half h = l >> 5) of fragment e reads piece
  // 2 ks + h of row 32 e + r' (+ the wavefront's offset); the swizzle only depends on r'
  const int frow = lane & 31, fh = lane >> 5, swz = (frow >> 1) & 7;
  const int a_row = (wm * 128 + frow) * BKW, b_row = BM * BKW + (wn * 128 + frow) * BKW;
  const int off0 = ((0 + fh) ^ swz) * 16, off1 = ((2 + fh) ^ swz) * 16;
  const int off2 = ((4 + fh) ^ swz) * 16, off3 = ((6 + fh) ^ swz) * 16;
  auto read_piece = [&](Frags<MT, NT>& f, int slot, int ks, int e) {   // slot, ks, e compile-time
    const int off = ks == 0 ? off0 : ks == 1 ? off1 : ks == 2 ? off2 : off3;
    if (e < MT)
      f.a[e] = *reinterpret_cast<const uint4*>(&ring[slot * SLOT + a_row + e * 4096 + off]);
    else
      f.b[e - MT] =
          *reinterpret_cast<const uint4*>(&ring[slot * SLOT + b_row + (e - MT) * 4096 + off]);
  };

  v16i acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
  Frags<MT, NT> f0, f1;
  Operands<MT, NT> s0, s1;
  u32 hi;                                   // 0xF0F0F0F0 in a scalar register
  asm volatile("s_mov_b32 %0, 0xf0f0f0f0" : "=s"(hi));
#pragma unroll
  for (int e = 0; e < 2 * NB; ++e) dma_piece(0, 0, e);
#pragma unroll
  for (int e = 0; e < NB; ++e) dma_piece(1, 1, e);
  {
    const float rs = scale[(long long)(my_m / T) * G + my_g];
    // the accumulators carry a factor 256; folding 2^-8 into the row scale is exact
    sRow[tid] = acc_dump ? rs : rs * 0.00390625f;
    const int n = n0 + tid;
    sCol[tid] = n < N ? w_scale[n] : 0.f;
    sBias[tid] = (bias && n < N) ? bias[n] : 0.f;
  }
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NB) : "memory");      // stage 0 has landed
  __syncthreads();
#pragma unroll
  for (int e = 0; e < NB; ++e) read_piece(f0, 0, 0, e);
#pragma unroll
  for (int e = 0; e < NB; ++e) expand_one<0>(s0, f0, e, hi);

#define TDQ_WSTAGE(kt, CUR, OTH)                                                                 \
  do {                                                                                           \
    __builtin_amdgcn_sched_barrier(0);                                                           \
    half_slab<1>(acc, s0, s1, f0, hi, [&](int b) { read_piece(f1, CUR, 1, b); });       /* X0 */ \
    half_slab<0>(acc, s1, s0, f1, hi, [&](int b) { dma_piece(OTH, (kt) + 1, NB + b); }); /* Y0 */ \
    half_slab<1>(acc, s0, s1, f1, hi, [&](int b) { read_piece(f0, CUR, 2, b); });       /* X1 */ \
    half_slab<0>(acc, s1, s0, f0, hi, [&](int) {});                                     /* Y1 */ \
    half_slab<1>(acc, s0, s1, f0, hi, [&](int b) { read_piece(f1, CUR, 3, b); });       /* X2 */ \
    half_slab<0>(acc, s1, s0, f1, hi, [&](int) {});                                     /* Y2 */ \
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");                                  \
    __syncthreads();                                                                             \
    __builtin_amdgcn_sched_barrier(0);                                                           \
    half_slab<1>(acc, s0, s1, f1, hi, [&](int b) { read_piece(f0, OTH, 0, b); });       /* X3 */ \
    half_slab<0>(acc, s1, s0, f0, hi, [&](int b) { dma_piece(CUR, (kt) + 2, b); });     /* Y3 */ \
  } while (0)

  int kt = 0;
  for (; kt + 1 < k_tiles; kt += 2) {
    TDQ_WSTAGE(kt, 0, 1);
    TDQ_WSTAGE(kt + 1, 1, 0);
  }
  if (kt < k_tiles) TDQ_WSTAGE(kt, 0, 1);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing of ours may still be landing
#undef TDQ_WSTAGE

  pipe_epilogue<OUT, MT, NT>(acc, sRow, sCol, sBias, lane, wm, wn, m0, n0, M, N, bias, Y, ld_y,
                             acc_dump);
}

// ---------------------------------------------------------------------------
// Rolling variant of the wide-stage kernel for shapes of many whole tiles (M and N
// multiples of 256, an even number, at least four, of 256-code stages): a workgroup is
// persistent and walks its share of the tiles, and the stream of stages never drains
// between tiles -- the loads of the next tile's first two stages are issued during the
// current tile's last two, like any other stage's, and the next tile's token-set ids and
// scales are fetched during those two stages by direct loads into LDS.  What a tile
// boundary still costs is the output phase itself (the matrix pipe idles while a single
// wavefront per SIMD converts and stores 256 results per lane, tile_store_cols4); the
// workgroup launch, the two dependent loads of the scales and the first stage's load
// latency are gone.
//
// Operand addresses are a uniform 64-bit base (tile, stage) plus a 32-bit per-lane offset
// that does not depend on the tile, so changing tile costs no vector work.
// Stores and loads share one in-order counter (vmcnt): the only wait for loads that has
// output stores before it is the first stage barrier of the next tile, about a hundred
// matrix instructions after the last store was issued.
// Tile order: as in the other kernels every XCD takes whole rows of tiles; inside an XCD
// consecutive workgroups take consecutive tiles, so at any time an XCD's CUs work on a
// few rows of tiles whose operands its L2 holds.
// ---------------------------------------------------------------------------
template <typename OUT>
__global__ __launch_bounds__(GEMM_THREADS, 1) void k_w4a4_gemm_roll(
    const uint8_t* __restrict__ Qx, long long ld_q, const int* __restrict__ gid,
    const float* __restrict__ scale, int M, int T, int K, int N, int G,
    const uint8_t* __restrict__ Qw, long long ld_w, const float* __restrict__ w_scale,
    const float* __restrict__ bias, OUT* __restrict__ Y, long long ld_y, int m_tiles, int n_tiles,
    double inv_T) {
  constexpr int MT = 4, NT = 4, BM = 256, BN = 256, NB = MT + NT;
  constexpr int BKW = 128;                     // packed bytes of K per stage (256 codes)
  constexpr int SLOT = (BM + BN) * BKW;        // 64 KiB: A rows then B rows, 128 B each
  __shared__ __attribute__((aligned(1024))) uint8_t ring[2 * SLOT];
  // scales of the tile being computed and of the next one (sets alternate from tile to
  // tile), and the next tile's token-set ids
  __shared__ __attribute__((aligned(256))) float sRow[2][BM], sCol[2][BN], sBias[2][BN];
  __shared__ __attribute__((aligned(256))) int sGid[BM];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int k_tiles = (K / 2) / BKW;           // even, >= 2 (host)

  // this workgroup's tiles: index list of its XCD, every (gridDim / 8)-th entry
  const int xcd = blockIdx.x % XCDS, wslot = blockIdx.x / XCDS, per_xcd = gridDim.x / XCDS;
  const int xcd_tiles = (m_tiles / XCDS) * n_tiles;          // m_tiles is a multiple of 8 (host)
  const int n_my = wslot < xcd_tiles ? (xcd_tiles - wslot + per_xcd - 1) / per_xcd : 0;
  if (n_my == 0) return;
  auto tile_m0 = [&](int it) { return (((wslot + it * per_xcd) / n_tiles) * XCDS + xcd) * BM; };
  auto tile_n0 = [&](int it) { return ((wslot + it * per_xcd) % n_tiles) * BN; };

  // per-lane byte offsets of this lane's piece of load i (rows 32 i + 8 w + (l >> 3))
  unsigned offA[2 * MT], offB[2 * NT];
  {
    const int rl0 = 8 * wave + (lane >> 3);
    const int c = (lane & 7) ^ ((rl0 >> 1) & 7);      // logical piece stored at position l & 7
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) offA[i] = (unsigned)((32 * i + rl0) * ld_q + c * 16);
    // Weight rows are dealt to the column blocks: LDS row 128 wn + 32 j + c' of the B part
    // (column block j of wavefront column wn, matrix column c') holds weight row
    // 128 wn + 4 c' + j, so that a lane's four column blocks are four adjacent outputs
    // (tile_store_cols4).  The swizzle goes by the LDS row, as for A.
#pragma unroll
    for (int i = 0; i < 2 * NT; ++i) {
      const int lrow = 32 * i + rl0;                                   // LDS row, 0 .. 255
      const int wrow = (lrow & 128) + 4 * (lrow & 31) + ((lrow >> 5) & 3);
      offB[i] = (unsigned)(wrow * ld_w + c * 16);
    }
  }
  const unsigned ring_base =
      (unsigned)(size_t)(__attribute__((address_space(3))) uint8_t*)ring;
  const unsigned dma_base = __builtin_amdgcn_readfirstlane(ring_base + wave * 1024);

  // uniform operand bases of the current and the next tile
  const uint8_t* curA = Qx + (long long)tile_m0(0) * ld_q;
  const uint8_t* curB = Qw + (long long)tile_n0(0) * ld_w;
  const uint8_t* nxtA = curA;
  const uint8_t* nxtB = curB;
  // stage `rel` counted from the current tile's first: past its end it is a stage of the
  // next tile (or, after the last tile, a harmless re-load into a slot nobody reads)
  auto dma_piece = [&](int slot, int rel, int e) {      // slot, e compile-time; e = 0 .. 15
    const bool next = rel >= k_tiles;
    const long long ko = (long long)(next ? rel - k_tiles : rel) * BKW;
    if (e < 2 * MT)
      dma16s((next ? nxtA : curA) + ko, offA[e], dma_base + slot * SLOT + e * 4096);
    else
      dma16s((next ? nxtB : curB) + ko, offB[e - 2 * MT],
             dma_base + slot * SLOT + BM * BKW + (e - 2 * MT) * 4096);
  };

  // Fragment reads.  Lane (row r' = l & 31, half h = l >> 5) of fragment e reads piece
  // 2 ks + h of row 32 e + r' (+ the wavefront's offset); the swizzle only depends on r'.
  // The per-lane LDS address of (operand, ks) is kept in a register; slot and fragment are
  // added as one opaque base per half-slab plus an immediate, so that the compiler cannot
  // turn the 64 (slot, ks, fragment) addresses into 64 registers hoisted out of the loops.
  const int frow = lane & 31, fh = lane >> 5, swz = (frow >> 1) & 7;
  unsigned a_ks[4], b_ks[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int off = ((2 * ks + fh) ^ swz) * 16;
    a_ks[ks] = (unsigned)((wm * 128 + frow) * BKW + off);
    b_ks[ks] = (unsigned)(BM * BKW + (wn * 128 + frow) * BKW + off);
  }
  unsigned rd_a = 0, rd_b = 0;               // bases of the half-slab's reads (bytes into the ring)
  auto read_base = [&](int slot, int ks) {    // slot, ks compile-time
    rd_a = a_ks[ks] + (unsigned)(slot * SLOT);
    rd_b = b_ks[ks] + (unsigned)(slot * SLOT);
    asm volatile("" : "+v"(rd_a), "+v"(rd_b));
  };
  auto read_piece = [&](Frags<MT, NT>& f, int e) {   // e compile-time
    if (e < MT)
      f.a[e] = *reinterpret_cast<const uint4*>(&ring[rd_a + (unsigned)(e * 4096)]);
    else
      f.b[e - MT] = *reinterpret_cast<const uint4*>(&ring[rd_b + (unsigned)((e - MT) * 4096)]);
  };

  Frags<MT, NT> f0;                         // the two that cross a tile boundary: the first
  Operands<MT, NT> s0;                      // slab of the next stage, read and half expanded
  u32 hi;                                   // 0xF0F0F0F0 in a scalar register
  asm volatile("s_mov_b32 %0, 0xf0f0f0f0" : "=s"(hi));

  // sources that are valid to load from whether or not the optional arrays exist
  const float* bias_src = bias ? bias : w_scale;
  const float* gid_src = reinterpret_cast<const float*>(gid ? gid : reinterpret_cast<const int*>(scale));
  // Scalars of a tile -- token-set id and scale of row tid, scale and bias of column tid --
  // travel global -> LDS by direct loads as well, so no register holds them while the
  // matrix stream runs: `ids` and the column entries first; one stage later (the ids have
  // landed) the row scales that depend on them.  Image of a row: floor((m + 1/2) / T) in
  // binary64, exact for m, T < 2^31.  The id is clamped into range before it indexes the
  // scales.
  const unsigned lds_of_wave = (unsigned)(wave * 256);
  auto lds_addr = [&](const void* ptr) {
    return __builtin_amdgcn_readfirstlane(
        (unsigned)(size_t)(__attribute__((address_space(3))) const uint8_t*)ptr + lds_of_wave);
  };
  auto fetch_ids_cols = [&](int set, int m_first, int n_first) {
    dma4s(gid_src, gid ? (unsigned)(m_first + tid) * 4u : 0u, lds_addr(sGid));
    dma4s(w_scale, (unsigned)(n_first + tid) * 4u, lds_addr(sCol[set]));
    dma4s(bias_src, (unsigned)(n_first + tid) * 4u, lds_addr(sBias[set]));
  };
  auto fetch_row_scales = [&](int set, int m_first) {
    int g = gid ? sGid[tid] : 0;
    g = g < 0 ? 0 : (g > G - 1 ? G - 1 : g);
    const int img = (int)(((double)(m_first + tid) + 0.5) * inv_T);
    dma4s(scale, (unsigned)(img * G + g) * 4u, lds_addr(sRow[set]));
  };

  // ---- first tile: fill the stream
  {
#pragma unroll
    for (int e = 0; e < 2 * NB; ++e) dma_piece(0, 0, e);
#pragma unroll
    for (int e = 0; e < NB; ++e) dma_piece(1, 1, e);
    fetch_ids_cols(0, tile_m0(0), tile_n0(0));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    fetch_row_scales(0, tile_m0(0));
    read_base(0, 0);
#pragma unroll
    for (int e = 0; e < NB; ++e) read_piece(f0, e);
#pragma unroll
    for (int e = 0; e < NB; ++e) expand_one<0>(s0, f0, e, hi);
  }

  // One stage; see k_w4a4_gemm_wide.  FIRST: the tile's first stage (fresh accumulators).
#define TDQ_RSTAGE(kt, CUR, OTH, FIRST, AFTER_BARRIER)                                            \
  do {                                                                                           \
    __builtin_amdgcn_sched_barrier(0);                                                           \
    read_base(CUR, 1);                                                                           \
    half_slab<1, MT, NT, FIRST>(acc, s0, s1, f0, hi, [&](int b) { read_piece(f1, b); });         \
    half_slab<0>(acc, s1, s0, f1, hi, [&](int b) { dma_piece(OTH, (kt) + 1, NB + b); });         \
    read_base(CUR, 2);                                                                           \
    half_slab<1>(acc, s0, s1, f1, hi, [&](int b) { read_piece(f0, b); });                        \
    half_slab<0>(acc, s1, s0, f0, hi, [&](int) {});                                              \
    read_base(CUR, 3);                                                                           \
    half_slab<1>(acc, s0, s1, f0, hi, [&](int b) { read_piece(f1, b); });                        \
    half_slab<0>(acc, s1, s0, f1, hi, [&](int) {});                                              \
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");                                  \
    __syncthreads();                                                                             \
    __builtin_amdgcn_sched_barrier(0);                                                           \
    AFTER_BARRIER;                                                                               \
    read_base(OTH, 0);                                                                           \
    __builtin_amdgcn_sched_barrier(0);                                                           \
    half_slab<1>(acc, s0, s1, f1, hi, [&](int b) { read_piece(f0, b); });                        \
    half_slab<0>(acc, s1, s0, f0, hi, [&](int b) { dma_piece(CUR, (kt) + 2, b); });              \
  } while (0)

  for (int it = 0; it < n_my; ++it) {
    v16i acc[MT][NT];                       // started afresh by the tile's first half-slab
    Frags<MT, NT> f1;
    Operands<MT, NT> s1;
    const int m0 = tile_m0(it), n0 = tile_n0(it);
    const bool more = it + 1 < n_my;
    if (more) {
      nxtA = Qx + (long long)tile_m0(it + 1) * ld_q;
      nxtB = Qw + (long long)tile_n0(it + 1) * ld_w;
    }
    // The next tile's scalars are fetched in this tile's last two stages (straight-line
    // code: the stages before and inside the loop simply carry no fetch) and land before the
    // next tile's first stage barrier, long before its output phase.  After the last tile
    // they re-fetch its own.
    const int set = it & 1;
    const int nm0 = tile_m0(more ? it + 1 : it), nn0 = tile_n0(more ? it + 1 : it);
    TDQ_RSTAGE(0, 0, 1, true, (void)0);
    TDQ_RSTAGE(1, 1, 0, false, (void)0);
    for (int kt = 2; kt < k_tiles - 2; kt += 2) {
      TDQ_RSTAGE(kt, 0, 1, false, (void)0);
      TDQ_RSTAGE(kt + 1, 1, 0, false, (void)0);
    }
    // the tile's last two stages carry the fetches: ids and column entries first, one stage
    // (and its barrier's wait for every load) later the row scales that read the ids
    TDQ_RSTAGE(k_tiles - 2, 0, 1, false, fetch_ids_cols(set ^ 1, nm0, nn0));
    TDQ_RSTAGE(k_tiles - 1, 1, 0, false, fetch_row_scales(set ^ 1, nm0));
    // Output phase of this tile (whole tiles only).  The lane index is made opaque per
    // tile: everything the output phase derives from it would otherwise be hoisted out of
    // the tile loop and live in (spilled) registers throughout the matrix stream.
    {
      int lane_o = lane;
      asm volatile("" : "+v"(lane_o));
      OUT* wtile = Y + (long long)(m0 + wm * 128) * ld_y + (n0 + wn * 128);
      if (bias)
        tile_store_cols4<OUT, true>(acc, sRow[set], sCol[set], sBias[set], lane_o, wm, wn, wtile, ld_y);
      else
        tile_store_cols4<OUT, false>(acc, sRow[set], sCol[set], sBias[set], lane_o, wm, wn, wtile, ld_y);
    }
    curA = nxtA;
    curB = nxtB;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing of ours may still be landing
#undef TDQ_RSTAGE
}

template <typename OUT>
static void launch_tile(const uint8_t* Qx, long long ld_q, const int* gid, const float* scale, int M,
                        int T, int K, int N, int G, const uint8_t* Qw, long long ld_w,
                        const float* w_scale, const float* bias, void* Y, long long ld_y,
                        int* acc_dump, hipStream_t st) {
  constexpr int BM = 128, BN = 128;
  const int m_tiles = (M + BM - 1) / BM, n_tiles = (N + BN - 1) / BN;
  const long long m_groups = (m_tiles + XCDS - 1) / XCDS;
  const unsigned grid = (unsigned)(m_groups * XCDS * n_tiles);
  hipLaunchKernelGGL((k_w4a4_gemm<OUT>), dim3(grid), dim3(GEMM_THREADS), 0, st, Qx, ld_q,
                     gid, scale, M, T, K, N, G, Qw, ld_w, w_scale, bias, static_cast<OUT*>(Y), ld_y,
                     acc_dump, m_tiles, n_tiles);
}

template <typename OUT, int MT, int NT>
static void launch_ring(const uint8_t* Qx, long long ld_q, const int* gid, const float* scale, int M,
                        int T, int K, int N, int G, const uint8_t* Qw, long long ld_w,
                        const float* w_scale, const float* bias, void* Y, long long ld_y,
                        int* acc_dump, hipStream_t st) {
  constexpr int BM = 64 * MT, BN = 64 * NT;
  const int m_tiles = (M + BM - 1) / BM, n_tiles = (N + BN - 1) / BN;
  const long long m_groups = (m_tiles + XCDS - 1) / XCDS;
  const unsigned grid = (unsigned)(m_groups * XCDS * n_tiles);
  const int stages = ((K + 1) / 2 + BKB - 1) / BKB;
  constexpr int D = 4;
  const size_t lds = (size_t)(stages < D ? stages : D) * (BM + BN) * BKB;
  // Streaming stores leave the caches at once.  At rows between 64-byte boundaries the wavefronts of a tile cut in its columns
  // share pieces of memory with others, which then go out in parts: where the outputs are more than the L2s have room for
  // beside the operands (24 of 32 MiB) such tiles store as usual.  With two checks per output, which is slow and so spreads
  // the stores / streamed by masks / as usual by masks, us: 398437 x 136 x 59 binary32 39.3 / 55.2 / 24.0, 291908 x 108 x 63 31.8 /
  // 41.5 / 18.3.  3400 random calls, as usual over streamed: from 24 to 32 MiB 0.81 times with 33 to 63 outputs, 0.97 with 65 to
  // 127, beyond 64 MiB 0.51 and 0.6; more outputs 1.00 to 1.03 up to 48 MiB and 0.88 beyond; below 24 MiB 1.00 to 1.08.  (The
  // choice in the kernel: its code made streamed calls 1.02 to 1.05 times as slow.)
  const bool keep = N % BN != 0 && ((reinterpret_cast<uintptr_t>(Y) | (uintptr_t)ld_y * sizeof(OUT)) & 63) != 0 &&
                    (long long)M * N * (int)sizeof(OUT) > (N < 64 ? 20ll : N < 128 ? 24ll : 48ll) << 20;
#define TDQ_RING(KEEP)                                                                                          \
  hipLaunchKernelGGL((k_w4a4_gemm_ring<OUT, MT, NT, KEEP>), dim3(grid), dim3(GEMM_THREADS), lds, st, Qx, ld_q,  \
                     gid, scale, M, T, K, N, G, Qw, ld_w, w_scale, bias, static_cast<OUT*>(Y), ld_y, acc_dump,  \
                     m_tiles, n_tiles)
  if (keep) TDQ_RING(true); else TDQ_RING(false);
#undef TDQ_RING
}

template <typename OUT, int MT, int NT>
static void launch_pipe(const uint8_t* Qx, long long ld_q, const int* gid, const float* scale, int M,
                        int T, int K, int N, int G, const uint8_t* Qw, long long ld_w,
                        const float* w_scale, const float* bias, void* Y, long long ld_y,
                        int* acc_dump, hipStream_t st) {
  constexpr int BM = 64 * MT, BN = 64 * NT;
  const int m_tiles = (M + BM - 1) / BM, n_tiles = (N + BN - 1) / BN;
  const long long m_groups = (m_tiles + XCDS - 1) / XCDS;
  const unsigned grid = (unsigned)(m_groups * XCDS * n_tiles);
  hipLaunchKernelGGL((k_w4a4_gemm_pipe<OUT, MT, NT>), dim3(grid), dim3(GEMM_THREADS), 0, st, Qx,
                     ld_q, gid, scale, M, T, K, N, G, Qw, ld_w, w_scale, bias, static_cast<OUT*>(Y),
                     ld_y, acc_dump, m_tiles, n_tiles);
}

template <typename OUT>
static void launch_wide(const uint8_t* Qx, long long ld_q, const int* gid, const float* scale, int M,
                        int T, int K, int N, int G, const uint8_t* Qw, long long ld_w,
                        const float* w_scale, const float* bias, void* Y, long long ld_y,
                        int* acc_dump, hipStream_t st) {
  const int m_tiles = (M + 255) / 256, n_tiles = (N + 255) / 256;
  const long long m_groups = (m_tiles + XCDS - 1) / XCDS;
  const unsigned grid = (unsigned)(m_groups * XCDS * n_tiles);
  hipLaunchKernelGGL((k_w4a4_gemm_wide<OUT>), dim3(grid), dim3(GEMM_THREADS), 0, st, Qx, ld_q, gid,
                     scale, M, T, K, N, G, Qw, ld_w, w_scale, bias, static_cast<OUT*>(Y), ld_y,
                     acc_dump, m_tiles, n_tiles);
}

// Compute units of the current device (0 if the query fails), looked up once per device.
static int compute_units() {
  static int cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int cu = __atomic_load_n(&cached[dev], __ATOMIC_RELAXED);
  if (cu == 0) {
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    __atomic_store_n(&cached[dev], cu, __ATOMIC_RELAXED);
  }
  return cu;
}

template <typename OUT>
static void launch_roll(const uint8_t* Qx, long long ld_q, const int* gid, const float* scale, int M,
                        int T, int K, int N, int G, const uint8_t* Qw, long long ld_w,
                        const float* w_scale, const float* bias, void* Y, long long ld_y, int wgs,
                        hipStream_t st) {
  hipLaunchKernelGGL((k_w4a4_gemm_roll<OUT>), dim3(wgs), dim3(GEMM_THREADS), 0, st, Qx, ld_q, gid,
                     scale, M, T, K, N, G, Qw, ld_w, w_scale, bias, static_cast<OUT*>(Y), ld_y,
                     M / 256, N / 256, 1.0 / (double)T);
}

// Microseconds the 256 x 256 kernels (one workgroup per CU, whole rows of tiles per XCD) take
// on an M x K x N product, roughly: rounds of tiles, each its stages plus an output phase
// (measured: 8192 x 1024 x 4096 in 38 us, 4096^3 51, 16384 x 3072 x 768 34), and the
// bounds-checked output of edge tiles (33000 x 1024 x 1024: 70).
static double big_tile_us(int M, int K, int N, int cus) {
  const long long rows = ((M + 255) / 256 + XCDS - 1) / XCDS, per_xcd = rows * ((N + 255) / 256);
  const long long rounds = (per_xcd * XCDS + cus - 1) / cus;
  return (double)rounds * (K * 0.0105 + 5.5) + 2.0 + (M % 256 || N % 256 ? 12.0 : 0.0);
}
// The same for the smaller tiles, which spread over the chip whatever the shape: 1.55 POP/s
// (33000 x 1024 x 1024: 54 us, 8192 x 1024 x 4096: 46), long K 1.7 (12000 x 2048 x 2048: 64).
static double small_tile_us(int M, int K, int N) {
  return 2.0 * M * N * K / (K >= 2048 ? 1.7e9 : 1.55e9) + 6.0;
}

// The kernel a product takes where it does not qualify for the rolling one.
enum LinearKernel { kRing64x64 = 1, kRing64x128, kRing128x64, kRing128x128, kStaged128, kPipe256, kWide256 };

static LinearKernel linear_kernel(int M, int K, int N, int cus) {
  // 256 x 256 tiles where they are estimated to be faster (see above); their kernels need
  // whole stages of K: 256 codes (measured 2 to 3 % faster), else 128
  if (K % 128 == 0 && big_tile_us(M, K, N, cus) < small_tile_us(M, K, N)) return K % 256 == 0 ? kWide256 : kPipe256;
  // Otherwise tiles of 64 or 128.  Long K without big tiles: the register-staged kernel, three
  // workgroups per CU (20000 x 4096 x 500: 54 us against 59, 16384 x 3000 x 768: 47 against 50).
  auto tiles = [&](int bm, int bn) { return (long long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  const long long t22 = tiles(128, 128), rounds22 = (t22 + 2 * cus - 1) / (2 * cus);
  if (K >= 2048 && t22 >= 2 * cus) return kStaged128;
  // Wide and tall enough to fill two workgroups per CU of 128 x 128 evenly (at least 0.72 of the
  // last round in use): those, they fetch least (131072 x 1000 x 1024: 178 us against 203 with
  // 64 x 128 tiles; 7744 x 320 x 1280, whose 610 tiles are 1.2 rounds: 16 against 11).  Else
  // 64 x 128 if that gives nearly two workgroups per CU and the last column of tiles is more than
  // half full, else 128 x 64 if those fill three per CU (131072 x 320 x 320: 34 us, 48 with
  // 64 x 128, 51 with 128 x 128), else 64 x 64 (968 x 512 x 512: 4.8 us, 5.6 with 64 x 128, 11 with
  // 128 x 128).
  const bool half_empty = N % 128 >= 1 && N % 128 <= 64;
  if (K >= 256 && (!half_empty || N >= 1024) &&
      (double)M * N >= 0.72 * 16384.0 * (double)(rounds22 * 2 * cus))
    return kRing128x128;
  // (a launch has fewer than 2^32 threads: 2^30 rows of 65 to 128 outputs are 2^24 tiles of 64 rows)
  auto fits = [&](int bm, int bn) {
    const long long rows = ((M + bm - 1) / bm + XCDS - 1) / XCDS;
    return rows * XCDS * ((N + bn - 1) / bn) * GEMM_THREADS < 1ll << 32;
  };
  if (!half_empty && tiles(64, 128) * 8 >= 15ll * cus && fits(64, 128)) return kRing64x128;
  if (tiles(128, 64) >= 3 * cus && fits(128, 64)) return kRing128x64;
  return fits(64, 64) ? kRing64x64 : kRing128x128;
}

// (not part of the ABI: the tests ask which kernel their shapes take)
extern "C" int tdq_linear_kernel_of(int32_t M, int32_t K, int32_t N, int32_t cus) {
  return linear_kernel(M, K, N, cus);
}

hipError_t launch_w4a4_gemm(const uint8_t* Qx, long long ld_q, const int* gid, const float* scale,
                            int M, int T, int K, int N, int G, const uint8_t* Qw, long long ld_w,
                            const float* w_scale, const float* bias, void* Y, tdq_dtype y_dt,
                            long long ld_y, int* acc_dump, hipStream_t st) {
  const long long big_tiles = (long long)((M + 255) / 256) * ((N + 255) / 256);
  // Whole tiles only, an even number of 256-code stages, rows of tiles in multiples of the
  // 8 XCDs, and at least 8 tiles for each of one persistent workgroup per CU: the rolling
  // kernel.  (One workgroup fits a CU, so more workgroups than CUs would run in turns.)
  if (!acc_dump && M % 256 == 0 && N % 256 == 0 && K % 512 == 0 && K >= 1024 && (M / 256) % XCDS == 0 &&
      256ll * ld_q < (1ll << 32) && 256ll * ld_w < (1ll << 32) && ld_y % 4 == 0 &&
      132ll * ld_y * (y_dt == TDQ_F32 ? 4 : 2) < (1ll << 32) &&      // 32-bit store offsets inside 128 rows
      reinterpret_cast<uintptr_t>(Y) % (y_dt == TDQ_F32 ? 16 : 8) == 0) {
    const int wgs = (compute_units() / XCDS) * XCDS;
    if (wgs >= XCDS && big_tiles >= 8ll * wgs) {
      if (y_dt == TDQ_F32)
        launch_roll<float>(Qx, ld_q, gid, scale, M, T, K, N, G, Qw, ld_w, w_scale, bias, Y, ld_y, wgs, st);
      else
        launch_roll<_Float16>(Qx, ld_q, gid, scale, M, T, K, N, G, Qw, ld_w, w_scale, bias, Y, ld_y,
                              wgs, st);
      return hipGetLastError();
    }
  }
  const int cus = compute_units() >= XCDS ? compute_units() : 256;
#define TDQ_GEMM_ARGS                                                                             \
  (Qx, ld_q, gid, scale, M, T, K, N, G, Qw, ld_w, w_scale, bias, Y, ld_y, acc_dump, st)
#define TDQ_GEMM_MODES(OUT)                                                                      \
  switch (linear_kernel(M, K, N, cus)) {                                                         \
    case kWide256: launch_wide<OUT> TDQ_GEMM_ARGS; break;                                        \
    case kPipe256: launch_pipe<OUT, 4, 4> TDQ_GEMM_ARGS; break;                                  \
    case kStaged128: launch_tile<OUT> TDQ_GEMM_ARGS; break;                                      \
    case kRing128x128: launch_ring<OUT, 2, 2> TDQ_GEMM_ARGS; break;                              \
    case kRing128x64: launch_ring<OUT, 2, 1> TDQ_GEMM_ARGS; break;                               \
    case kRing64x128: launch_ring<OUT, 1, 2> TDQ_GEMM_ARGS; break;                               \
    case kRing64x64: launch_ring<OUT, 1, 1> TDQ_GEMM_ARGS; break;                                \
  }
  if (y_dt == TDQ_F32) { TDQ_GEMM_MODES(float) } else { TDQ_GEMM_MODES(_Float16) }
#undef TDQ_GEMM_MODES
#undef TDQ_GEMM_ARGS
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Block-scaled contraction for the paper-literal granularity (Supp. Algorithm 1, step 10
// with one step Delta[m, kb] per token m and block kb of g = 32 channels):
//   Y[m, n] = s_w[n] * sum_kb Delta[m, kb] * acc_kb[m, n],
//   acc_kb[m, n] = sum_{i in block kb} Qx[m, i] * Qw[n, i]   (|acc_kb| <= 32 * 64)
// The int32 accumulation cannot run over the whole of K any more: one matrix
// instruction (K = 32) is exactly one block, and its 16 results per lane are turned into
// floats and folded into a binary32 accumulator with the block's step,
//   f <- fma(float(acc_kb), Delta[m, kb], f),   kb ascending,
// i.e. 32 vector operations per matrix instruction: this kernel is bound by the vector
// unit, not by the matrix cores (which idle three quarters of the time).
// The floats cost a subtraction each, not a conversion: the matrix instruction starts from
// the bits of 1.5 * 2^23 instead of zero.  On this chip v_cvt_f32_i32 takes 4.8 cycles of a
// SIMD with several wavefronts, an addition, a multiply-add or a bitwise operation 2.6 to
// 3.1 (conversions, shifts, minima and three-operand integer forms run at half the rate).  The factor 256
// of the nibble expansion is taken out once at the end (a power of two: exact).
//
// The weights are the row operand and the activations the column operand: a lane of the result then
// holds ONE activation row, so a block's step is one register instead of sixteen, and a stage's four steps
// of a row are one LDS read.  2 x 2 wavefronts of 32 MB activations x 64 weights; operands by direct-to-LDS
// loads in stages of 64 bytes (4 blocks) per row, three slots, two stages in flight (LDS layout of a slot
// as in k_w4a4_gemm_pipe); 64 x 128 tiles (MB = 1) leave three workgroups on a CU, so that one's vector
// work covers another's waits and the last round of tiles is even.  A lane's results are runs of 4 outputs in
// 32 rows, so they leave through LDS as whole lines.
// 128 x 128 tiles staged through registers, two workgroups per CU, and now, us: 8192 x 768 x 768 20.3 and 16.5, 968 x
// 512 x 512 15.9 and 7.8, 7744 x 320 x 1280 26.9 and 14.7, 4096 x 4096 x 64 66.3 and 38.0, 131072 x 1024 x 4096 1354 and
// 1271, 131072 x 4096 x 1024 1346 and 1215.  What it gave is waits (for LDS 47 M cycles and 2 M in the last but one) and
// even rounds of tiles.  The loop has 42.6 vector instructions per matrix instruction (38.8 with MB = 2): 32 of the
// rescale, 9 or 6 of nibble expansion, addresses.  Conversions, with the masked stage inside the loop (four copies of
// accumulators more), and now: 8192 x 768 x 768 17.5 and 15.9, 7744 x 320 x 1280 14.8 and 13.6, 32768 x 320 x 1280 49.1
// and 41.6, 131072 x 1024 x 4096 1325 and 1255, 131072 x 4096 x 1024 1262 and 1177.  (The subtrahend as a literal: in a
// vector register it made the kernel 1 to 5 % slower.)
// The 8-byte reads of the fragments meet in their banks (80 M cycles over 256 CUs); the vector work covers it.
// ---------------------------------------------------------------------------
// 64 floats from 64 addresses -> 64 consecutive floats of LDS
__device__ __forceinline__ void dma4(const float* gptr, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
               :
               : "v"(gptr), "s"(lds_base)
               : "memory");
}

// STREAM: how outputs are stored (launch_w4a4_gemm_blocks says when).
template <typename OUT, int MB, bool STREAM>
__global__ __launch_bounds__(GEMM_THREADS, (MB == 1 ? 3 : 2)) void k_w4a4_gemm_blocks(
    const uint8_t* __restrict__ Qx, long long ld_q, const float* __restrict__ bscale, long long ld_s,
    int M, int K, int N, const uint8_t* __restrict__ Qw, long long ld_w,
    const float* __restrict__ w_scale, const float* __restrict__ bias, OUT* __restrict__ Y,
    long long ld_y, int m_tiles, int n_tiles, int y_vec_ok) {
  constexpr int NA = 2, BM = 64 * MB, BN = 128, D = 3;
  constexpr int SB = BKB / 16;                         // blocks (= 16-byte pieces) per stage
  constexpr int SLOT = (BM + BN) * BKB;                // activation rows then weight rows, 64 B each
  constexpr int NL = (BM + BN) / 64 + MB;              // direct loads per wavefront and stage
  constexpr int W = OutVec<OUT>::W;                    // outputs per 16-byte store
  constexpr int PITCH = 64 * (int)sizeof(OUT) + 16;    // a row of 64 outputs on its way out
  __shared__ __attribute__((aligned(1024))) uint8_t ring[D * SLOT];
  __shared__ __attribute__((aligned(256))) float sD[D][BM][SB];
  __shared__ __attribute__((aligned(16))) float sCol[BN], sBias[BN];
  static_assert(4 * 32 * PITCH <= D * SLOT, "the results of 32 rows of every wavefront fit the ring");

  const int bid = blockIdx.x;
  const int xcd = bid % XCDS, idx = bid / XCDS;
  const int m_tile = (idx / n_tiles) * XCDS + xcd;
  const int n_tile = idx % n_tiles;
  if (m_tile >= m_tiles) return;
  const int m0 = m_tile * BM, n0 = n_tile * BN;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int kbytes = (K + 1) / 2, KB = (K + 31) / 32;
  const int k_tiles = (KB + SB - 1) / SB;

  if (tid < BN) {
    const int n = n0 + tid < N ? n0 + tid : N - 1;
    sCol[tid] = w_scale[n];
    sBias[tid] = bias ? bias[n] : 0.f;
  }

  // load e of this wavefront fills 16 rows: lane l writes position l & 3 of row l >> 2; the last MB
  // loads are the steps of 16 rows, lane l that of row l >> 2 and block l & 3
  const uint8_t* src[MB + NA];
  const float* dsrc[MB];
  const int brow = 16 * wave + (lane >> 2);
  const int piece = ((lane & 3) ^ ((brow >> 2) & 3)) * 16;
#pragma unroll
  for (int e = 0; e < MB + NA; ++e) {
    if (e < MB) {
      const int r = m0 + 64 * e + brow < M ? m0 + 64 * e + brow : M - 1;
      src[e] = Qx + (long long)r * ld_q;
      dsrc[e] = bscale + (long long)r * ld_s;
    } else {
      const int r = n0 + 64 * (e - MB) + brow;
      src[e] = Qw + (long long)(r < N ? r : N - 1) * ld_w;
    }
  }
  const unsigned ring_base = (unsigned)(size_t)(__attribute__((address_space(3))) uint8_t*)ring;
  const unsigned sd_base = (unsigned)(size_t)(__attribute__((address_space(3))) float*)&sD[0][0][0];
  auto load_stage = [&](int kt, int slot) {
    const int kb = kt * BKB + piece;
    const int off = kb < 16 * KB ? kb : 0;               // past the row's end: any piece of it
    const int blk = kt * SB + (lane & 3);
    const unsigned to = __builtin_amdgcn_readfirstlane(ring_base + slot * SLOT + wave * 1024);
    const unsigned to_d = __builtin_amdgcn_readfirstlane(sd_base + slot * (BM * SB * 4) + wave * 256);
#pragma unroll
    for (int e = 0; e < MB + NA; ++e) dma16(src[e] + off, to + e * 4096);
#pragma unroll
    for (int e = 0; e < MB; ++e) dma4(dsrc[e] + (blk < KB ? blk : KB - 1), to_d + e * 1024);
  };
  load_stage(0, 0);
  if (k_tiles > 1) load_stage(1, 1);

  float accf[NA][MB][16];
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < MB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) accf[i][j][r] = 0.f;

  // Lane l feeds row (l & 31) of a 32-row fragment and, of each 16-byte block of K, the 8 bytes at offset
  // 8 (l >> 5); of a 32 x 32 result it owns activation l & 31 and weights 8 q + 4 (l >> 5) + 0..3.
  const int frow = lane & 31, fh = lane >> 5, swz = (frow >> 2) & 3;
  const int x_row = (wm * 32 * MB + frow) * BKB + 8 * fh, w_row = (BM + wn * 64 + frow) * BKB + 8 * fh;
  // The block's sum is added to the bits of 1.5 * 2^23: as a binary32 number the result is that plus the sum,
  // exactly (|256 acc| <= 2^19), and a subtraction, which runs at twice the rate of a conversion, leaves the sum.
  u32 magic_bits = 0x4B400000u;
  asm volatile("" : "+v"(magic_bits));
  const float magic = 12582912.f;                      // stays a literal of the instruction
  v16i start;
#pragma unroll
  for (int r = 0; r < 16; ++r) start[r] = (int)magic_bits;
  asm volatile("" : "+v"(start));
  auto stage = [&](int kt, int slot, auto tail) {
    const uint8_t* at = ring + slot * SLOT;
    float4 d[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) d[j] = *reinterpret_cast<const float4*>(&sD[slot][wm * 32 * MB + j * 32 + frow][0]);
#pragma unroll
    for (int kb = 0; kb < SB; ++kb) {
      if (decltype(tail)::value && kt * SB + kb >= KB) break;            // uniform
      const int off = (kb ^ swz) * 16;
      v4i a[NA], b[MB];
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const uint2 f = *reinterpret_cast<const uint2*>(at + w_row + i * 32 * BKB + off);
        a[i] = expand(f.x, f.y);
      }
#pragma unroll
      for (int j = 0; j < MB; ++j) {
        uint2 f = *reinterpret_cast<const uint2*>(at + x_row + j * 32 * BKB + off);
        if (decltype(tail)::value) {                   // bytes past the row's end do not count
          const int keep = kbytes - ((kt * SB + kb) * 16 + 8 * fh);
          f.x &= tail_mask(keep, 0);
          f.y &= tail_mask(keep, 4);
        }
        b[j] = expand(f.x, f.y);
      }
      v16i t[NA][MB];
#pragma unroll
      for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
          t[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], b[j], start, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j) {
          const float dl = kb == 0 ? d[j].x : kb == 1 ? d[j].y : kb == 2 ? d[j].z : d[j].w;
#pragma unroll
          for (int r = 0; r < 16; ++r)
            accf[i][j][r] = __builtin_fmaf(__builtin_bit_cast(float, (int)t[i][j][r]) - magic, dl, accf[i][j][r]);
        }
    }
  };
  // Stages whose four blocks are whole, then (if there is one) the last, masked one: with the choice inside the
  // loop the compiler keeps two sets of accumulators and copies them.
  const int whole_stages = kbytes / BKB;
  int slot = 0;
  auto enter = [&](int kt) {
    // stage kt has landed when at most the loads of the stage after it are outstanding
    if (kt + 1 < k_tiles)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // the slot of stage kt - 1: every wavefront drained its reads before this barrier
    if (kt + 2 < k_tiles) load_stage(kt + 2, slot == 0 ? 2 : slot - 1);
  };
  for (int kt = 0; kt < whole_stages; ++kt) {
    enter(kt);
    stage(kt, slot, std::false_type{});
    slot = slot == D - 1 ? 0 : slot + 1;
  }
  if (whole_stages < k_tiles) {
    enter(whole_stages);
    stage(whole_stages, slot, std::true_type{});
  }
  __syncthreads();

  // Output, 32 rows of 64 outputs per wavefront at a time, through its own part of the ring.
  uint8_t* mine = ring + wave * 32 * PITCH;
  const int n_first = n0 + wn * 64;
  const bool whole = y_vec_ok && (n_first + 64 <= N || N % W == 0);   // the outputs are whole stores
  constexpr int LPR = 64 / W, RPI = 64 / LPR;          // lanes per row, rows per store instruction
#pragma unroll
  for (int j = 0; j < MB; ++j) {
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int nl = i * 32 + 8 * q + 4 * fh;        // first of 4 outputs, in this wavefront's 64
        const float4 ws = *reinterpret_cast<const float4*>(&sCol[wn * 64 + nl]);
        const float4 bs = *reinterpret_cast<const float4*>(&sBias[wn * 64 + nl]);
        float y[4] = {(accf[i][j][4 * q] * 0.00390625f) * ws.x, (accf[i][j][4 * q + 1] * 0.00390625f) * ws.y,
                      (accf[i][j][4 * q + 2] * 0.00390625f) * ws.z, (accf[i][j][4 * q + 3] * 0.00390625f) * ws.w};
        if (bias) {
          y[0] += bs.x;
          y[1] += bs.y;
          y[2] += bs.z;
          y[3] += bs.w;
        }
        uint8_t* to = mine + frow * PITCH + nl * (int)sizeof(OUT);
        if constexpr (sizeof(OUT) == 2) {
          const h2v p0 = round_pair_to_half(y[0], y[1]), p1 = round_pair_to_half(y[2], y[3]);
          *reinterpret_cast<uint2*>(to) = make_uint2(__builtin_bit_cast(u32, p0), __builtin_bit_cast(u32, p1));
        } else {
          *reinterpret_cast<float4*>(to) = make_float4(y[0], y[1], y[2], y[3]);
        }
      }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (this wavefront's own writes, in order)
    if (whole) {                                         // (uniform)
      typedef u32 v4u __attribute__((ext_vector_type(4)));
#pragma unroll
      for (int it = 0; it < 32 / RPI; ++it) {
        const int row = it * RPI + lane / LPR, part = lane % LPR;
        const int m = m0 + wm * 32 * MB + j * 32 + row;
        const uint8_t* from = mine + row * PITCH + part * 16;
        if (m < M && n_first + part * W < N)
          store_as<STREAM>(*reinterpret_cast<const v4u*>(from),
                           reinterpret_cast<v4u*>(Y + (long long)m * ld_y + n_first + part * W));
      }
    } else {
      const int m = m0 + wm * 32 * MB + j * 32;
      store_rows<STREAM, OUT>(Y + (long long)m * ld_y + n_first, ld_y, M - m, N - n_first, lane, [&](int row, int c) {
        return *reinterpret_cast<const OUT*>(mine + row * PITCH + c * (int)sizeof(OUT));
      });
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before the next 32 rows overwrite it
  }
}

hipError_t launch_w4a4_gemm_blocks(const uint8_t* Qx, long long ld_q, const float* bscale,
                                   long long ld_s, int M, int K, int N, const uint8_t* Qw,
                                   long long ld_w, const float* w_scale, const float* bias, void* Y,
                                   tdq_dtype y_dt, long long ld_y, hipStream_t st) {
  const int esz = y_dt == TDQ_F32 ? 4 : 2;
  const int y_vec_ok = (reinterpret_cast<uintptr_t>(Y) & 15) == 0 && ld_y * esz % 16 == 0 ? 1 : 0;
  const int n_tiles = (N + 127) / 128;
  // 128 rows a tile where there are many tiles: 39 vector instructions per matrix instruction instead of 43 weigh
  // more than an even last round and a third workgroup per CU.  64 / 128 rows, us: 32768 x 320 x 1280 (2560
  // tiles of 128) 43.1 / 47.3, 131072 x 4096 x 1024 (8192) 1137 / 1114.
  const bool tall = (long long)((M + 127) / 128) * n_tiles >= 4096;
  const int bm = tall ? 128 : 64;
  const int m_tiles = (M + bm - 1) / bm;
  const unsigned grid = (unsigned)((long long)((m_tiles + XCDS - 1) / XCDS) * XCDS * n_tiles);
  // Streaming stores leave the caches at once.  Rows that start between 64-byte boundaries share those pieces of memory
  // with the next tile's, which then go out in two parts, and with few stages the outputs of all tiles are under way together
  // (binary32: four workgroups a CU with 32 KiB each are an XCD's whole L2).  Such calls of many tiles store as usual.
  // Streamed / as usual, us: binary32 49334 x 224 x 1268 77 / 56, 32611 x 192 x 1519 64 / 47, 70006 x 160 x 3592 297 / 201, 64592
  // x 96 x 937 90 / 51; binary16 67922 x 23 x 848 36.1 / 23.9.  Of 1359 random binary32 calls (most of them K up to 256, rows
  // anywhere) 587 change, 0.74 times the time in the geometric mean, 42 of them more than 3 % slower, up to 1.14; of 900
  // binary16 ones with more than 3000 tiles 94, 0.84, 10, up to 1.13.  Streamed stay rows on 64 bytes (35663 x 252 x 4016 binary32
  // 149 / 169), one wavefront's columns (as usual 1.03 to 1.1 times), more channels (1.04 to 1.07, 222846 x 224 x 632
  // by tall tiles 142 / 169; binary16 from 65 on even, from 129 on 1.04), and fewer tiles (even).
  const bool apart = (reinterpret_cast<uintptr_t>(Y) & 63) == 0 && ld_y * esz % 64 == 0;
  const long long tiles = (long long)((M + 63) / 64) * n_tiles;
  const bool stream = apart || N <= 64 ||
                      (y_dt == TDQ_F32 ? K > (tall ? 160 : 256) || tiles <= 1536 : K > 64 || tiles <= 4096);
#define TDQ_BLK(OUT, MB, STREAM)                                                                               \
  hipLaunchKernelGGL((k_w4a4_gemm_blocks<OUT, MB, STREAM>), dim3(grid), dim3(GEMM_THREADS), 0, st, Qx, ld_q, bscale, ld_s, \
                     M, K, N, Qw, ld_w, w_scale, bias, static_cast<OUT*>(Y), ld_y, m_tiles, n_tiles, y_vec_ok)
#define TDQ_BLK_OUT(OUT)                                                            \
  if (stream) {                                                                     \
    if (tall) TDQ_BLK(OUT, 2, true); else TDQ_BLK(OUT, 1, true);                    \
  } else {                                                                          \
    if (tall) TDQ_BLK(OUT, 2, false); else TDQ_BLK(OUT, 1, false);                  \
  }
  if (y_dt == TDQ_F32) {
    TDQ_BLK_OUT(float)
  } else {
    TDQ_BLK_OUT(_Float16)
  }
#undef TDQ_BLK_OUT
#undef TDQ_BLK
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The contraction on the 6-bit matrix format of gfx950.  The sixteen int4 codes are all
// exactly representable in bf6 (e3m2: 1 sign, 3 exponent, 2 mantissa bits), products and
// sums of integers below 2^24 are exact in the binary32 accumulator, and
// v_mfma_scale_f32_32x32x64_f8f6f4 with unit scales runs at twice the int8 rate per
// instruction (K = 64 in the time the int8 instruction takes for K = 32) with no nibble
// expansion in the loop: measured register-only on random codes 5.3 POP/s against 3.2
// for the int8 instruction (the clock drops less under its load).
//
// Operand storage ("f6 fragments"): rows in blocks of 32, K in blocks of 64; the block
// (rb, kb) is 1536 contiguous bytes at ((rb * KB + kb) * 1536), KB = number of 64-blocks
// of K (even, zero-padded), holding the 64 lanes' operands of ONE matrix instruction in
// lane order: lane l = (row % 32) + 32 * ((k % 64) / 32) owns 24 bytes, code j = k % 32
// in bits [6 j, 6 j + 6) (little endian).  A workgroup's stage (128 codes of K for 256
// rows of each operand) is 16 chunks of 3072 contiguous bytes, copied by 48 direct-to-LDS
// loads of 1 KiB, and a lane reads its operand as three 8-byte LDS reads, 24 bytes apart
// from its neighbours': conflict-free without any swizzle.
// ---------------------------------------------------------------------------
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
constexpr int F6_FRAG = 1536;            // bytes of one (32 rows, 64 codes) block

// Packed nibbles [R, ld] -> f6 fragments.  One wavefront per fragment (32 rows x 64 codes),
// the four wavefronts of a workgroup on four consecutive fragments of the same rows, so
// that together they read whole 128-byte lines.  Lane l loads the 16 bytes of (row l / 2,
// half l % 2), the lane that owns (row, half) in the fragment's order fetches them with a
// lane permute, sign-extends the 32 nibbles, and one conversion instruction (even codes
// in its first operand, odd ones in its second) packs them.  Codes at and beyond K, rows
// at and beyond R are zero.
typedef int v6i_pack __attribute__((ext_vector_type(6)));
__global__ __launch_bounds__(256) void k_pack_f6(const uint8_t* __restrict__ Q, long long ld, int R,
                                                 int K, int KB, long long n_blocks, int vec_ok,
                                                 uint8_t* __restrict__ F) {
  const int l = threadIdx.x & 63;
  const long long blk = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (blk >= n_blocks) return;                             // whole wavefronts only
  const int kb = (int)(blk % KB);
  const long long rb = blk / KB;
  const long long row = rb * 32 + (l >> 1);
  const int k0 = kb * 64 + 32 * (l & 1);
  u32 n[4] = {0u, 0u, 0u, 0u};
  if (row < R && k0 < K) {
    const uint8_t* src = Q + row * ld + k0 / 2;
    const int live = K - k0;                               // codes of this piece that exist
    const int nb = live >= 32 ? 16 : (live + 1) / 2;       // bytes that hold them
    if (vec_ok && nb == 16) {
      const uint4 q = *reinterpret_cast<const uint4*>(src);
      n[0] = q.x; n[1] = q.y; n[2] = q.z; n[3] = q.w;
    } else {
      for (int j = 0; j < nb; ++j) n[j >> 2] |= (u32)src[j] << (8 * (j & 3));
    }
    if (live < 32) {                                       // the pad nibble of an odd K is not a code
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int keep = live - 8 * w;
        n[w] &= keep >= 8 ? 0xFFFFFFFFu : (keep <= 0 ? 0u : (1u << (4 * keep)) - 1u);
      }
    }
  }
  const int from = (2 * (l & 31) + (l >> 5)) * 4;          // the lane that loaded this lane's piece
  u32 m[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) m[w] = (u32)__builtin_amdgcn_ds_bpermute(from, (int)n[w]);
  v16f ev, od;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const u32 wd = m[i >> 2];
    const int sh = 8 * (i & 3);                            // codes 2 i and 2 i + 1: bits sh, sh + 4
    ev[i] = (float)((int)(wd << (28 - sh)) >> 28);
    od[i] = (float)((int)(wd << (24 - sh)) >> 28);
  }
  const v6i_pack r = __builtin_amdgcn_cvt_scalef32_2xpk16_bf6_f32(ev, od, 1.0f);
  uint2* dst = reinterpret_cast<uint2*>(F + (blk * 64 + l) * 24);
  dst[0] = make_uint2((u32)r[0], (u32)r[1]);
  dst[1] = make_uint2((u32)r[2], (u32)r[3]);
  dst[2] = make_uint2((u32)r[4], (u32)r[5]);
}

hipError_t launch_pack_f6(const uint8_t* Q, long long ld, int R, int K, uint8_t* F, hipStream_t st) {
  const int KB = 2 * ((K + 127) / 128);
  const long long n_blocks = (long long)((R + 31) / 32) * KB;
  const int vec_ok = ((reinterpret_cast<uintptr_t>(Q) & 15) == 0 && ld % 16 == 0) ? 1 : 0;
  hipLaunchKernelGGL(k_pack_f6, dim3((unsigned)((n_blocks + 3) / 4)), dim3(256), 0, st, Q, ld, R, K, KB,
                     n_blocks, vec_ok, F);
  return hipGetLastError();
}

template <typename OUT>
__global__ __launch_bounds__(GEMM_THREADS, 1) void k_w4a4_gemm_f6(
    const uint8_t* __restrict__ A6, const uint8_t* __restrict__ B6, int KB,
    const int* __restrict__ gid, const float* __restrict__ scale, int M, int T, int N, int G,
    const float* __restrict__ w_scale, const float* __restrict__ bias, OUT* __restrict__ Y,
    long long ld_y, int* __restrict__ acc_dump, int m_tiles, int n_tiles) {
  constexpr int MT = 4, NT = 4, BM = 256, BN = 256;
  constexpr int KS = 2;                          // 64-blocks of K per stage
  constexpr int CH = KS * F6_FRAG;               // one row block's bytes of a stage
  constexpr int SLOT = 16 * CH;                  // 8 row blocks of A, then 8 of B: 48 KiB
  constexpr int NDMA = SLOT / 1024 / 4;          // direct loads per wavefront and stage: 12
  __shared__ __attribute__((aligned(1024))) uint8_t ring[3 * SLOT];
  __shared__ __attribute__((aligned(16))) float sRow[BM], sCol[BN], sBias[BN];

  const int bid = blockIdx.x;
  const int xcd = bid % XCDS, idx = bid / XCDS;
  const int m_tile = (idx / n_tiles) * XCDS + xcd;
  const int n_tile = idx % n_tiles;
  if (m_tile >= m_tiles) return;
  const int m0 = m_tile * BM, n0 = n_tile * BN;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int stages = KB / KS;                    // KB is even
  const int MBk = (M + 31) / 32, NBk = (N + 31) / 32;

  // piece pi = wave + 4 e of a stage: chunk pi / 3 (row block), 1 KiB part pi % 3
  const uint8_t* src[NDMA];
#pragma unroll
  for (int e = 0; e < NDMA; ++e) {
    const int pi = wave + 4 * e;
    const int c = pi / 3, part = pi % 3;
    long long rb;
    const uint8_t* base;
    if (c < 8) {
      rb = (long long)m_tile * 8 + c;
      rb = rb < MBk ? rb : MBk - 1;              // past the end: a harmless re-read
      base = A6;
    } else {
      rb = (long long)n_tile * 8 + (c - 8);
      rb = rb < NBk ? rb : NBk - 1;
      base = B6;
    }
    src[e] = base + rb * KB * F6_FRAG + part * 1024 + lane * 16;
  }
  const unsigned ring_base = (unsigned)(size_t)(__attribute__((address_space(3))) uint8_t*)ring;
  {
    const int my_m = m0 + tid < M ? m0 + tid : M - 1;
    const int my_g = gid ? gid[my_m] : 0;
    sRow[tid] = scale[(long long)(my_m / T) * G + my_g];
    const int n = n0 + tid;
    sCol[tid] = n < N ? w_scale[n] : 0.f;
    sBias[tid] = (bias && n < N) ? bias[n] : 0.f;
  }

  v16f acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int a_off = wm * 4 * CH + lane * 24, b_off = (8 + wn * 4) * CH + lane * 24;
  // fragment f of a K block: f < 4 the wavefront's row blocks of A, else of B
  auto read_frag = [&](v8i (&fa)[MT], v8i (&fb)[NT], int slot, int kk, int f) {   // all compile-time
    const int off = (f < MT ? a_off + f * CH : b_off + (f - MT) * CH) + kk * F6_FRAG;
    const uint2* p = reinterpret_cast<const uint2*>(&ring[slot * SLOT + off]);
    const uint2 q0 = p[0], q1 = p[1], q2 = p[2];
    const v8i v = {(int)q0.x, (int)q0.y, (int)q1.x, (int)q1.y, (int)q2.x, (int)q2.y, 0, 0};
    if (f < MT) fa[f] = v; else fb[f - MT] = v;
  };
  auto mma = [&](const v8i (&fa)[MT], const v8i (&fb)[NT], int t) {               // t compile-time
    acc[t >> 2][t & 3] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
        fa[t >> 2], fb[t & 3], acc[t >> 2][t & 3], 3, 3, 0, 127, 0, 127);
  };
  // stage st (clamped to the last one: past the end a harmless re-load) -> slot
  auto dma_piece = [&](int slot, int st, int e) {                                  // slot, e compile-time
    const int sc = st < stages ? st : stages - 1;
    dma16(src[e] + (long long)sc * CH,
          __builtin_amdgcn_readfirstlane(ring_base + slot * SLOT + (wave + 4 * e) * 1024));
  };

  // Three slots.  The instruction stream of stage s (slot s % 3; two K blocks, 32 matrix
  // instructions) is laid out by hand in bundles fenced with sched_barrier — one
  // wavefront per SIMD, nothing else hides latency — and has no branch (a branch would
  // end the basic block and with it the order):
  //   K block 0, 16 matrix instructions: the 8 fragments of K block 1 are read;
  //   wait until stage s + 1 has landed (all but the newest 12 loads), barrier: now every
  //     wavefront has read the last of slot s % 3, and stage s + 1 is whole;
  //   K block 1, 16 matrix instructions: the 8 fragments of K block 0 of stage s + 1 are
  //     read and the 12 direct loads of stage s + 3 are issued into slot s % 3 — two full
  //     stages (about 2000 cycles) before anything reads them.
  v8i a0[MT], b0[NT], a1[MT], b1[NT];
#pragma unroll
  for (int e = 0; e < NDMA; ++e) dma_piece(0, 0, e);
#pragma unroll
  for (int e = 0; e < NDMA; ++e) dma_piece(1, 1, e);
#pragma unroll
  for (int e = 0; e < NDMA; ++e) dma_piece(2, 2, e);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NDMA) : "memory");                  // stage 0 has landed
  __syncthreads();
#pragma unroll
  for (int f = 0; f < MT + NT; ++f) read_frag(a0, b0, 0, 0, f);

#define TDQ_F6_STAGE(s, CUR, NXT)                                                                \
  do {                                                                                           \
    _Pragma("unroll") for (int t = 0; t < 16; ++t) {                                             \
      __builtin_amdgcn_sched_barrier(0);                                                         \
      mma(a0, b0, t);                                                                            \
      if ((t & 1) == 0) read_frag(a1, b1, CUR, 1, t >> 1);                                       \
    }                                                                                            \
    __builtin_amdgcn_sched_barrier(0);                                                           \
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(NDMA) : "memory");                       \
    __syncthreads();                                                                             \
    _Pragma("unroll") for (int t = 0; t < 16; ++t) {                                             \
      __builtin_amdgcn_sched_barrier(0);                                                         \
      mma(a1, b1, t);                                                                            \
      if ((t & 1) == 0) read_frag(a0, b0, NXT, 0, t >> 1);                                       \
      else if (t < 12) { dma_piece(CUR, (s) + 3, t - 1); dma_piece(CUR, (s) + 3, t); }           \
    }                                                                                            \
    __builtin_amdgcn_sched_barrier(0);                                                           \
  } while (0)

  int s = 0;
  for (; s + 2 < stages; s += 3) {
    TDQ_F6_STAGE(s, 0, 1);
    TDQ_F6_STAGE(s + 1, 1, 2);
    TDQ_F6_STAGE(s + 2, 2, 0);
  }
  if (s < stages) {
    TDQ_F6_STAGE(s, 0, 1);
    if (s + 1 < stages) TDQ_F6_STAGE(s + 1, 1, 2);
  }
#undef TDQ_F6_STAGE
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // nothing of ours may still be landing

  pipe_epilogue<OUT, MT, NT, v16f>(acc, sRow, sCol, sBias, lane, wm, wn, m0, n0, M, N, bias, Y, ld_y,
                                   acc_dump);
}

hipError_t launch_w4a4_gemm_f6(const uint8_t* A6, const uint8_t* B6, int K, const int* gid,
                               const float* scale, int M, int T, int N, int G, const float* w_scale,
                               const float* bias, void* Y, tdq_dtype y_dt, long long ld_y,
                               int* acc_dump, hipStream_t st) {
  const int KB = 2 * ((K + 127) / 128);
  const int m_tiles = (M + 255) / 256, n_tiles = (N + 255) / 256;
  const long long m_groups = (m_tiles + XCDS - 1) / XCDS;
  const unsigned grid = (unsigned)(m_groups * XCDS * n_tiles);
  if (y_dt == TDQ_F32)
    hipLaunchKernelGGL((k_w4a4_gemm_f6<float>), dim3(grid), dim3(GEMM_THREADS), 0, st, A6, B6, KB, gid,
                       scale, M, T, N, G, w_scale, bias, static_cast<float*>(Y), ld_y, acc_dump, m_tiles,
                       n_tiles);
  else
    hipLaunchKernelGGL((k_w4a4_gemm_f6<_Float16>), dim3(grid), dim3(GEMM_THREADS), 0, st, A6, B6, KB,
                       gid, scale, M, T, N, G, w_scale, bias, static_cast<_Float16*>(Y), ld_y, acc_dump,
                       m_tiles, n_tiles);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The block-scaled contraction (one step per row and 32-code block) on f6 fragments.
// The 6-bit instruction covers 64 codes = two blocks, lanes 0-31 supplying the even
// block and lanes 32-63 the odd one of an operand; zeroing the other half of one operand
// makes it deliver one block's sum, already as a float, so the rescale is one fused
// multiply-add per element and block (16 per matrix instruction) instead of a conversion
// and a multiply-add on top of the nibble expansion (38).  Same arithmetic as
// k_w4a4_gemm_blocks (f <- fma(acc_kb, Delta[m, kb], f), kb ascending): same bits.
//
// The weights are the instruction's row operand and the activations its column operand,
// so a lane holds ONE activation row m (= lane % 32) and 16 output channels: Delta[m, kb]
// is one register per lane instead of sixteen.
//
// 128 x 128 tile, 4 x 2 wavefronts of 32 x 64, two workgroups per CU; a stage is 128 codes of
// K = four scale blocks = four "rounds" of 2 matrix instructions + 32 multiply-adds per
// wavefront.  The kernel is bound by the issue of vector instructions: a matrix instruction
// leaves room for four or five of them, each further one costs its own 2.7 cycles
// (register-only, zeros: 13.9 ns alone, 15 with 4 multiply-adds, 28.7 with 16).  A round consumes
// the results of the round before, one at a time, and re-issues the matrix instruction into the
// result registers just freed; operands of a round are read from LDS during the round before.
// Four wavefronts per SIMD (128 registers each) cover what is left of the waits: with 2 x 2
// wavefronts of 64 x 64, two per SIMD, us then and now: 32768 x 1024 x 4096 260 and 234,
// 131072 x 4096 x 1024 889 and 846, 131072 x 1024 x 4096 990 and 940, 7744 x 320 x 1280 14.7 and
// 13.0, 968 x 512 x 512 8.6 and 7.0, 4096 x 4096 x 64 34.6 and 26.5 (the operands of a fragment are
// then read from LDS four times instead of three; it has the room).
//   Ring of three slots of 24 KiB + the stage's scales [4][128], all by direct-to-LDS
//   loads (4 per wavefront and stage, no staging registers).  Everything read from the
//   slot of stage s is read by round 2 of stage s; the barrier in that round publishes
//   stage s + 1, and right behind it the loads of stage s + 3 go into the slot of stage
//   s: two full stages of flight.  A half-zero operand is read as such: the lanes of the
//   unwanted half read 24 zero bytes (one multiply-add on the address, no selects on the
//   data).  No branch inside the stage: a branch would end the basic block and the
//   compiler would regroup the instructions.
// ---------------------------------------------------------------------------

constexpr int BF6_THREADS = 512;
template <typename OUT>
__global__ __launch_bounds__(BF6_THREADS, 4) void k_w4a4_gemm_blocks_f6(
    const uint8_t* __restrict__ A6, const uint8_t* __restrict__ B6, int KB64,
    const float* __restrict__ bscale, long long ld_s, int M, int K, int N,
    const float* __restrict__ w_scale, const float* __restrict__ bias, OUT* __restrict__ Y,
    long long ld_y, int m_tiles, int n_tiles, int y_vec_ok) {
  // WM x 2 wavefronts of 32 x 64
  constexpr int WM = 4;
  constexpr int MT = 1, NT = 2, BM = WM * 32, BN = 128;
  constexpr int NW = 2 * WM, THREADS = BF6_THREADS;
  constexpr int KS = 2;                          // 64-blocks of K per stage
  constexpr int SBK = 2 * KS;                    // scale blocks per stage
  constexpr int CH = KS * F6_FRAG;               // 3072 bytes per row block and stage
  constexpr int ACH = WM;                    // row blocks of A; then 4 of B
  constexpr int SLOT = (ACH + 4) * CH;
  constexpr int PIECES = SLOT / 1024;            // 1 KiB direct loads per stage: 24
  constexpr int NDMA = PIECES / NW;              // per wavefront: 3
  constexpr int NVM = NDMA + 1;                  // + a scale load
  static_assert(NW * 64 == THREADS && NDMA * NW == PIECES && BM == NW * 16, "every wavefront has the same loads");
  __shared__ __attribute__((aligned(1024))) uint8_t ring[3 * SLOT];
  __shared__ __attribute__((aligned(256))) float sD[3][BM][SBK];
  __shared__ __attribute__((aligned(16))) float sCol[BN], sBias[BN];
  __shared__ __attribute__((aligned(32))) unsigned sZero[8];
  typedef unsigned u2v __attribute__((ext_vector_type(2)));
  typedef const __attribute__((address_space(3))) u2v* lds_u2;

  const unsigned bid = blockIdx.y * gridDim.x + blockIdx.x;      // gridDim.x is a multiple of XCDS
  const int xcd = bid % XCDS, idx = bid / XCDS;
  const int m_tile = (idx / n_tiles) * XCDS + xcd;
  const int n_tile = idx % n_tiles;
  if (m_tile >= m_tiles) return;
  const int m0 = m_tile * BM, n0 = n_tile * BN;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;        // wm < WM
  const int stages = KB64 / KS;
  const int KB = (K + 31) / 32;                  // scale blocks that exist
  const int MBk = (M + 31) / 32, NBk = (N + 31) / 32;

  for (int j = tid; j < BN; j += THREADS) {
    const int n = n0 + j;
    sCol[j] = n < N ? w_scale[n] : 0.f;
    sBias[j] = (bias && n < N) ? bias[n] : 0.f;
  }
  if (tid < 8) sZero[tid] = 0u;

  // piece wave + NW e of a stage: chunk (row block) piece / 3, 1 KiB part piece % 3
  const uint8_t* sbase[NDMA];
  int piece[NDMA];
#pragma unroll
  for (int e = 0; e < NDMA; ++e) {
    const int pi = wave + NW * e;
    piece[e] = pi;
    const int c = pi / 3, part = pi % 3;
    long long rb;
    const uint8_t* base;
    if (c < ACH) {
      rb = (long long)m_tile * ACH + c;
      rb = rb < MBk ? rb : MBk - 1;              // past the end: a harmless re-read
      base = A6;
    } else {
      rb = (long long)n_tile * 4 + (c - ACH);
      rb = rb < NBk ? rb : NBk - 1;
      base = B6;
    }
    sbase[e] = base + rb * KB64 * F6_FRAG + part * 1024;
  }
  const unsigned lane16 = lane * 16;
  const unsigned ring_base = (unsigned)(size_t)(__attribute__((address_space(3))) uint8_t*)ring;
  const unsigned sd_base = (unsigned)(size_t)(__attribute__((address_space(3))) float*)&sD[0][0][0];
  const unsigned zero_addr = (unsigned)(size_t)(__attribute__((address_space(3))) uint8_t*)sZero;
  // scales of a stage, [BM][4] in LDS: one load brings 16 rows x 4 blocks, four lanes per
  // row, so it touches 16 lines (a lane per row would touch 64 for the same 256 bytes,
  // and the L2 request rate is what this kernel runs against); wavefront w brings row
  // group w.  Rows and blocks past the end are
  // clamped to real ones (their products are zero or unused); only the last stage can
  // have fewer than four blocks.
  const float* d_row0 = bscale + (long long)m0 * ld_s;
  const int last_real = KB - 1 - (stages - 1) * SBK;       // 0..3 (or more: no clamp)
  unsigned d_voff, d_voff_last;
  {
    int row = wave * 16 + (lane >> 2);
    row = m0 + row < M ? row : M - 1 - m0;
    const int b = lane & 3;
    d_voff = ((unsigned)row * (unsigned)ld_s + (unsigned)b) * 4u;
    d_voff_last = ((unsigned)row * (unsigned)ld_s + (unsigned)(b < last_real ? b : last_real)) * 4u;
  }
  // stage st (clamped to the last: past the end a harmless re-load) -> slot (run-time
  // 0, 1, 2 in turn: with compile-time slots the compiler hoists every LDS address out
  // of the loop and spills them)
  auto dma_stage = [&](int slot, int st) {
    const int sc = st < stages ? st : stages - 1;
#pragma unroll
    for (int e = 0; e < NDMA; ++e)
      dma16s(sbase[e] + (long long)sc * CH, lane16,
             __builtin_amdgcn_readfirstlane(ring_base + slot * SLOT + piece[e] * 1024));
    const bool last = sc == stages - 1;
    dma4s(d_row0 + sc * SBK, last ? d_voff_last : d_voff,
          __builtin_amdgcn_readfirstlane(sd_base + (slot * BM + wave * 16) * SBK * 4));
  };

  // operand reads.  x (activations): lanes of half h read their 24 bytes, the others the
  // zeros: address = base + flag * offset, one instruction, kept where it is written.
  const bool lower = lane < 32;
  const unsigned x_lane = ring_base + (wm * MT * CH + lane * 24);
  const unsigned w_lane = ring_base + ((ACH + wn * 2) * CH + lane * 24);
  const unsigned x_base[2] = {lower ? x_lane : zero_addr, lower ? zero_addr : x_lane};
  const unsigned x_flag[2] = {lower ? 1u : 0u, lower ? 0u : 1u};
  const unsigned d_lane = sd_base + (wm * 32 * MT + (lane & 31)) * SBK * 4;
  auto read24 = [&](unsigned addr) {
    const lds_u2 p = (lds_u2)(size_t)addr;
    const u2v q0 = p[0], q1 = p[1], q2 = p[2];
    const v8i v = {(int)q0.x, (int)q0.y, (int)q1.x, (int)q1.y, (int)q2.x, (int)q2.y, 0, 0};
    return v;
  };
  auto read_x = [&](v8i (&dst)[MT], int slot, int kk, int h) {          // kk, h compile-time
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const unsigned off = (unsigned)(slot * SLOT + i * CH + kk * F6_FRAG);   // scalar
      unsigned addr;
      asm volatile("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(addr) : "v"(x_flag[h]), "s"(off), "v"(x_base[h]));
      dst[i] = read24(addr);
    }
  };
  auto read_w = [&](v8i (&dst)[NT], int slot, int kk) {
    const unsigned w_slot = w_lane + (unsigned)(slot * SLOT);
#pragma unroll
    for (int j = 0; j < NT; ++j) dst[j] = read24(w_slot + (unsigned)(j * CH + kk * F6_FRAG));
  };
  typedef float f4v __attribute__((ext_vector_type(4)));
  typedef const __attribute__((address_space(3))) f4v* lds_f4;
  auto read_dl = [&](f4v (&dst)[MT], int slot) {           // the lane's rows, the stage's 4 blocks
    const lds_f4 p = (lds_f4)(size_t)(d_lane + (unsigned)(slot * SBK * BM * 4));
#pragma unroll
    for (int i = 0; i < MT; ++i) dst[i] = p[i * 32];
  };

  float accf[MT][NT][16];
  v16f t[MT][NT];
  f4v dcur[MT];                                  // the stage's scales of the lane's rows
  float dlast[MT];                               // those of the previous stage's last block
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    dlast[i] = 0.f;
    dcur[i] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        accf[i][j][r] = 0.f;
        t[i][j][r] = 0.f;
      }
  }
  const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto consume = [&](int i, int j, float d) {
#pragma unroll
    for (int r = 0; r < 16; ++r) accf[i][j][r] = __builtin_fmaf(t[i][j][r], d, accf[i][j][r]);
  };

  v8i xbuf[2][MT], wbuf[2][NT];                  // activations by half h, weights by kk
  dma_stage(0, 0);
  dma_stage(1, 1);
  dma_stage(2, 2);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NVM) : "memory");   // stage 0 has landed
  __syncthreads();
  read_x(xbuf[0], 0, 0, 0);
  read_w(wbuf[0], 0, 0);

  // Round R of the stage in slot CUR (NXT: the next stage's).  R and the register
  // indices are compile-time constants.  Round 0 consumes the last group of the stage
  // before (scale kept in dlast) and reads this stage's scales; round R > 0 consumes
  // group R - 1.
#define TDQ_BF6_SLOT(R, I, J)                                                                     \
  do {                                                                                            \
    __builtin_amdgcn_sched_barrier(0);                                                            \
    consume(I, J, (R) == 0 ? dlast[I] : dcur[I][((R) + 3) & 3]);                                  \
    t[I][J] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wbuf[(R) >> 1][J], xbuf[(R) & 1][I], \
                                                              zero, 3, 3, 0, 127, 0, 127);        \
  } while (0)
#define TDQ_BF6_ROUND(s, CUR, NXT, R, MORE)                                                       \
  do {                                                                                            \
    /* the next round's activations first: two slots until they are used */                      \
    __builtin_amdgcn_sched_barrier(0);                                                            \
    if ((R) < 3) read_x(xbuf[((R) + 1) & 1], CUR, ((R) + 1) >> 1, ((R) + 1) & 1);                 \
    else read_x(xbuf[0], NXT, 0, 0);                                                              \
    TDQ_BF6_SLOT(R, 0, 0);                                                                        \
    if ((R) == 0) {                                                                               \
      read_dl(dcur, CUR);                         /* the old ones were spent in round 3 */        \
      read_w(wbuf[1], CUR, 1);                    /* for rounds 2 and 3 */                        \
    }                                                                                             \
    if ((R) == 2) {                                                                               \
      __builtin_amdgcn_sched_barrier(0);                                                          \
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((MORE) ? NVM : 0) : "memory");          \
      __builtin_amdgcn_s_barrier();                                                               \
      if (MORE) dma_stage(CUR, (s) + 3);                                                          \
      read_w(wbuf[0], NXT, 0);                    /* for rounds 0 and 1 of the next stage */      \
    }                                                                                             \
    TDQ_BF6_SLOT(R, 0, 1);                                                                        \
    if ((R) == 3) dlast[0] = dcur[0][3];                                                          \
    __builtin_amdgcn_sched_barrier(0);                                                            \
  } while (0)

  int cur = 0, nxt = 1, nn = 2;
  // The last three stages load nothing and have a loop of their own.  (With one loop, whose stages must not
  // branch and so loaded the last stage again, a tile of 8 stages loaded 11 and waited for them before
  // its output: with 2 x 2 wavefronts 32768 x 1024 x 4096 265.6 us, 248.2 so; 131072 x 4096 x 1024 888 and 869.)
  int s = 0;
#pragma unroll 1
  for (; s + 3 < stages; ++s) {
    TDQ_BF6_ROUND(s, cur, nxt, 0, true);
    TDQ_BF6_ROUND(s, cur, nxt, 1, true);
    TDQ_BF6_ROUND(s, cur, nxt, 2, true);
    TDQ_BF6_ROUND(s, cur, nxt, 3, true);
    const int o = cur;
    cur = nxt;
    nxt = nn;
    nn = o;
  }
#pragma unroll 1
  for (; s < stages; ++s) {
    TDQ_BF6_ROUND(s, cur, nxt, 0, false);
    TDQ_BF6_ROUND(s, cur, nxt, 1, false);
    TDQ_BF6_ROUND(s, cur, nxt, 2, false);
    TDQ_BF6_ROUND(s, cur, nxt, 3, false);
    const int o = cur;
    cur = nxt;
    nxt = nn;
    nn = o;
  }
#undef TDQ_BF6_ROUND
#undef TDQ_BF6_SLOT
  consume(0, 0, dlast[0]);                       // the last round's results
  consume(0, 1, dlast[0]);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // nothing of ours may still be landing

  // Register r of result (i, j) is row m = 32 i + lane % 32 of the wavefront's 32 MT and
  // channel 32 j + 8 (r / 4) + 4 (lane / 32) + r % 4: a lane holds short runs of 32 rows,
  // which as stores would touch 32 lines with 8 or 16 bytes each.  So the wavefront's
  // results (already scaled) go, 32 rows at a time, through its own 8.5 KiB of the ring,
  // now free, and leave row-major: every store instruction writes whole 128-byte lines.
  __syncthreads();                               // every wavefront's loads have landed
  constexpr int TP = 68;                         // pitch in floats: 16-byte aligned rows, staggered banks
  float* T = reinterpret_cast<float*>(ring) + wave * (32 * TP);
  const int ml = lane & 31, nq = (lane >> 5) * 4;
  constexpr int W = 16 / (int)sizeof(OUT);       // outputs per 16-byte store: 4 or 8
  constexpr int LPR = 64 / W;                    // lanes per row of 64
  constexpr int RPI = 64 / LPR;                  // rows per store instruction
  const int rsub = lane / LPR, col = (lane % LPR) * W;
  const int nbase = n0 + wn * 64 + col;
  const bool whole = y_vec_ok && (n0 + wn * 64 + 64 <= N || N % W == 0);   // the outputs are whole stores
#pragma unroll
  for (int i = 0; i < MT; ++i) {                 // 32 rows at a time
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        const int cw = j * 32 + rq * 8 + nq;     // channel within the wavefront's 64
        const float4 sc4 = *reinterpret_cast<const float4*>(&sCol[wn * 64 + cw]);
        const float4 bi4 = *reinterpret_cast<const float4*>(&sBias[wn * 64 + cw]);
        float4 y = make_float4(accf[i][j][4 * rq] * sc4.x, accf[i][j][4 * rq + 1] * sc4.y,
                               accf[i][j][4 * rq + 2] * sc4.z, accf[i][j][4 * rq + 3] * sc4.w);
        if (bias) {
          y.x = y.x + bi4.x;
          y.y = y.y + bi4.y;
          y.z = y.z + bi4.z;
          y.w = y.w + bi4.w;
        }
        *reinterpret_cast<float4*>(&T[ml * TP + cw]) = y;
      }
    if (whole) {                                 // (uniform)
#pragma unroll
      for (int it = 0; it < 32 / RPI; ++it) {
        const int row = it * RPI + rsub;
        const int m = m0 + wm * 32 * MT + i * 32 + row;
        float y[W];
#pragma unroll
        for (int q = 0; q < W / 4; ++q) {
          const float4 v = *reinterpret_cast<const float4*>(&T[row * TP + col + 4 * q]);
          y[4 * q] = v.x; y[4 * q + 1] = v.y; y[4 * q + 2] = v.z; y[4 * q + 3] = v.w;
        }
        if (m < M && nbase < N) store_out_vec<OUT>(Y + (long long)m * ld_y + nbase, y);
      }
    } else {
      const int m = m0 + wm * 32 * MT + i * 32, n = n0 + wn * 64;
      store_rows<true, OUT>(Y + (long long)m * ld_y + n, ld_y, M - m, N - n, lane,
                      [&](int row, int c) { return (OUT)T[row * TP + c]; });
    }
  }
}

hipError_t launch_w4a4_gemm_blocks_f6(const uint8_t* A6, const uint8_t* B6, const float* bscale,
                                      long long ld_s, int M, int K, int N, const float* w_scale,
                                      const float* bias, void* Y, tdq_dtype y_dt, long long ld_y,
                                      hipStream_t st) {
  const int KB64 = 2 * ((K + 127) / 128);
  const int m_tiles = (M + 127) / 128, n_tiles = (N + 127) / 128;
  // An axis of a grid holds fewer than 2^32 threads, and 2^30 rows are 2^23 tiles of 512: two axes (workgroups past
  // the last tile return)
  const long long tiles = (long long)((m_tiles + XCDS - 1) / XCDS) * XCDS * n_tiles, axis = 1 << 22;
  const dim3 grid(tiles < axis ? (unsigned)tiles : (unsigned)axis, (unsigned)((tiles + axis - 1) / axis));
  // 16-byte stores where every row of Y starts on a 16-byte boundary
  const int per16 = y_dt == TDQ_F32 ? 4 : 8;
  const int y_vec_ok = (reinterpret_cast<uintptr_t>(Y) % 16 == 0 && ld_y % per16 == 0) ? 1 : 0;
  if (y_dt == TDQ_F32)
    hipLaunchKernelGGL((k_w4a4_gemm_blocks_f6<float>), grid, dim3(BF6_THREADS), 0, st, A6, B6,
                       KB64, bscale, ld_s, M, K, N, w_scale, bias, static_cast<float*>(Y), ld_y, m_tiles,
                       n_tiles, y_vec_ok);
  else
    hipLaunchKernelGGL((k_w4a4_gemm_blocks_f6<_Float16>), grid, dim3(BF6_THREADS), 0, st, A6, B6,
                       KB64, bscale, ld_s, M, K, N, w_scale, bias, static_cast<_Float16*>(Y), ld_y,
                       m_tiles, n_tiles, y_vec_ok);
  return hipGetLastError();
}

}  // namespace tdq
