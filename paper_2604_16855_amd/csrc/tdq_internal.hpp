// Internal declarations shared by the translation units of libtdq (host side
// launch wrappers, workspace layout).  Nothing here is part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "tdq.h"

namespace tdq {

constexpr int kQMax = 7;
constexpr int kQMin = -8;
constexpr int kOctaveFloor = 24;       // assignment: keys > 24 octaves below the top share set 0
constexpr int kMaxLevels = 7;          // radix-select levels: a 31-bit key at >= 5 bits per level
                                       // (256 sets x 2^5 bins fill the LDS histogram)
constexpr int kHistLdsWords = 8192;    // 32 KiB of LDS histogram per workgroup
constexpr int kMaxLevelBits = 11;

// Per-(image, token set) working record of the calibration, kept in the workspace.
struct GroupWork {
  long long n;          // elements = tokens * C
  long long k_rem;      // rank still to be resolved below the current prefix
  unsigned prefix;      // radix levels: magnitude-key bits fixed so far (high bits of thr);
                        // sampled interval, binary32: keys collected of the set's bin
  unsigned tokens;      // tokens in the set
  float c_base;         // max |x|
  float sigma;          // population std + eps_std
};

// Key interval that a sample says holds the k-th smallest magnitude key of an (image, token
// set), and what the sweep counted for it: `width` bins of 2^shift keys from lo on (binary16: of one
// key), or (binary32, bit 8 of shift) `width` keys cut into cells of 2^(shift & 63) keys.
struct Bracket {
  unsigned lo;       // first key of the interval, at least 1
  unsigned width;    // bins or keys of the interval, 0 = nothing to count
  unsigned below;    // elements of the set with key < lo
  unsigned shift;
};
constexpr int kBracketLdsWords = 16384;   // 64 KiB of LDS histogram per workgroup (128 KiB, one
                                          // workgroup per CU, made the sweep 30 % slower)
// Fewest one-key bins per set worth sampling for: with fewer the interval (half-width
// bins / 2 keys, 1024 keys per octave) misses too often, and the multi-level radix
// select over all sets at once is the cheaper route from the start.
constexpr int kBracketMinBins = 256;
constexpr int kListMax = 1024;            // most words of a set's list of collected keys

// Bins per set of the interval histogram, at most 2048: the LDS budget shared out to G sets,
// rounded down to a power of two (0 = too many sets: use the multi-level radix select
// instead).  For the zr quantile most sets use bracket_bins_zr(G) of them, no more than half the
// budget where that leaves 512 -- every workgroup of the sweep clears and flushes all its bins
// ([8, 7744, 512] with 16 sets calibrates in 52.4 us with 1024 of them, 47.2 with 512), and 512, a
// quarter of an octave to either side, are six standard deviations of the sample's estimate in a
// set of similar tokens; a set whose sample says that its keys are sparse there uses all.  With
// few sets a set mixes tokens of very different ranges and the sample's error is that of its few
// hundred tokens, and a percentile base radius lies where keys are sparse: those get more bins and
// twice the sample.
int bracket_bins(int G);
int bracket_bins_zr(int G);

// How the magnitude key (15 bits for fp16, 31 for fp32) is split into radix levels.
struct LevelPlan {
  int n_levels;
  int bits[kMaxLevels];
  int shift[kMaxLevels];   // key >> shift gives this level's digit in the low `bits`
  int key_bits;
};

LevelPlan make_level_plan(tdq_dtype dt, int G);

// Byte offsets of the pieces of the calibration workspace (all 256-aligned).
struct WorkspaceLayout {
  size_t status;     // uint32[64]; word 0 = device status word, words 1 and 2 = sets whose
                     // rank the last calibration's sampled key interval missed in pass kPassZr
                     // and pass kPassBase (searched for in the set's own rows)
  size_t img_flag;   // uint32[B]     per-image non-finite flag
  size_t r;          // float[M]      per-token range
  size_t mean;       // double[M]     per-token mean
  size_t m2;         // double[M]     per-token sum (x - mean)^2
  size_t part;       // per-workgroup partial set records of the assignment
  size_t grp;        // GroupWork[B*G]
  size_t hist;       // uint32 [levels][B*G][1 << bits[level]]
  size_t hist_level[kMaxLevels];   // offset of each level inside the workspace
  size_t br;         // Bracket[B*G]
  size_t bhist;      // uint32 [B*G][bracket_bins(G)]
  size_t total;
};

WorkspaceLayout make_layout(int B, int T, int G, const LevelPlan& lp);

struct Scalars {   // fp32 constants of the projection, rounded once on the host
  float qmax_tau;  // 7 * tau
  float two_qmax;  // 14
  float qmax;      // 7
  float eps_scale;
  double eps_std;
  double zr;
  double base_pct;   // 0 = base radius is the set's maximum; (0,1) = rank quantile Q_p (Eq. DSTG_clip)
  unsigned flags;
  double inv_groups; // 1 / n_groups
};

// The rank select runs once per rank wanted of every set: pass kPassBase finds the
// base radius Q_p(|x|) (only when a percentile is asked for) and leaves it in
// GroupWork::c_base; pass kPassZr finds Q_zr(|x|) and applies the projection.
constexpr int kPassZr = 0;
constexpr int kPassBase = 1;

// What a statistics kernel clears for the kernels after it: the status words, and words that
// workgroups of the rank select add into.
struct SelectClear {
  unsigned* status;        // nullptr: nothing to clear
  unsigned* ctl;
  unsigned n_ctl;
  unsigned* hist;          // n_hist words, a multiple of 4, 16-byte aligned
  unsigned n_hist;
};

// ---- launch wrappers (each returns the hipError_t of its launch) -------------
hipError_t launch_token_stats(const void* X, tdq_dtype dt, int M, int C, long long ld,
                              float* r, double* mean, double* m2, const SelectClear& cl, hipStream_t st);
// Token-set assignment.  An image is shared by assign_split(T) workgroups, each of
// which leaves one partial record per set in `part`; the records are merged into
// GroupWork by launch_finalize_groups.  (The sampled rank select of either type assigns the sets
// in its own first kernel, launch_sets.)
constexpr int kAssignSplitMax = 8;
int assign_split(int T);
size_t assign_partial_bytes(int B, int G);
hipError_t launch_assign(const float* r, const double* mean, const double* m2, int B, int T, int C,
                         int G, int* gid, void* part, unsigned* img_flag, unsigned* status,
                         hipStream_t st);
// Arms the radix levels for one pass: working record of every set (rank of this pass;
// keep_base = keep the base radius an earlier pass left) and cleared level histograms.
hipError_t launch_finalize_groups(const void* part, int B, int T, int C, int G, const Scalars& sc,
                                  int pass, bool keep_base, GroupWork* grp, unsigned* hist,
                                  const LevelPlan& lp, hipStream_t st);
// The last level of pass kPassZr projects, that of pass kPassBase stores the base radius.
hipError_t launch_hist(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                       const int* gid, const GroupWork* grp, unsigned* hist_level, int shift,
                       int bits, hipStream_t st);
hipError_t launch_select(unsigned* hist_level, int B, int G, int shift, int bits, bool last,
                         tdq_dtype dt, const Scalars& sc, GroupWork* grp, float* clip,
                         float* scale, tdq_group_stats* stats, const unsigned* img_flag,
                         unsigned* status, int pass, hipStream_t st);
// Rank select guided by a sample: binary16 input in one sweep, binary32 input in two (the
// second, launch_bracket_gather, collects the keys of one bin per set into `lists`, cap words
// per set).  Of the W bins of a set's interval histogram most binary16 sets use the first Wfew;
// binary32: the interval is cut into `cells` cells and those into W bins.
hipError_t launch_sets(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                       int Wfew, int W, int cells, const float* r, const double* mean, const double* m2, int* gid,
                       const Scalars& sc, int pass, bool keep_base, GroupWork* grp, Bracket* br,
                       unsigned* bhist, unsigned* lists, int cap, unsigned* img_flag,
                       unsigned* status, hipStream_t st);
// The same for images of up to kWholeTokens tokens, seen through to the radii: the G + extra workgroups of
// an image are shared out to its sets and read their rows; ranks = 2: the percentile base radius as well.
// bhist (W words per set, for both ranks) and ctl (kSetCtl words per set) are cleared by the statistics kernel if
// extra > 0.
constexpr int kWholeTokens = 8192;     // (the list of tokens and the rest fit 64 KiB of LDS)
constexpr int kListTokens = 16384;     // most tokens of an image listed by rank in LDS
constexpr int kSetCtl = 8;
// binary32 sets that several workgroups share: how long, in ticks of 10 ns, one waits for the others before it claims
// another share of the rows, and before it counts on them no more.
struct Waits {
  unsigned patience, limit;
};
constexpr Waits kWaits = {2000, 2000000};
hipError_t launch_sets_whole(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G, int ranks,
                             int extra, int Wfew, int W, const float* r, const double* mean, const double* m2,
                             int* gid, const Scalars& sc, unsigned* bhist, void* ctl, unsigned* img_flag,
                             unsigned* status, float* clip, float* scale, tdq_group_stats* stats,
                             const Waits& waits, hipStream_t st);
hipError_t launch_bracket_hist(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                               int Wfew, int W, int cells, unsigned* lists, int cap, const int* gid,
                               Bracket* br, unsigned* bhist, hipStream_t st);
hipError_t launch_bracket_gather(const void* X, int B, int T, int C, long long ld, int G, int W,
                                 int cells, const int* gid, const Bracket* br, const unsigned* bhist,
                                 GroupWork* grp, unsigned* lists, int cap, hipStream_t st);
hipError_t launch_bracket_finish(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                                 int Wfew, int W, int cells, const int* gid, const unsigned* bhist,
                                 const unsigned* lists, int cap, bool force_miss, const Scalars& sc, int pass, GroupWork* grp,
                                 const Bracket* br, float* clip, float* scale, tdq_group_stats* stats,
                                 const unsigned* img_flag, unsigned* status, hipStream_t st);
hipError_t launch_quantize(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                           const int* gid, const float* clip, const float* scale, uint8_t* Q,
                           long long ld_q, hipStream_t st);
hipError_t launch_quantize_blocks(const void* X, tdq_dtype dt, long long M, int C, long long ld,
                                  int kq, int kp, const Scalars& sc, uint8_t* Q, long long ld_q,
                                  float* bscale, float* bclip, long long ld_s, hipStream_t st);
hipError_t launch_w4a4_gemm_blocks(const uint8_t* Qx, long long ld_q, const float* bscale,
                                   long long ld_s, int M, int K, int N, const uint8_t* Qw,
                                   long long ld_w, const float* w_scale, const float* bias, void* Y,
                                   tdq_dtype y_dt, long long ld_y, hipStream_t st);
hipError_t launch_quantize_blocks_f6(const void* X, tdq_dtype dt, long long M, int C, long long ld,
                                     int kq, int kp, const Scalars& sc, uint8_t* F, float* bscale,
                                     float* bclip, long long ld_s, hipStream_t st);
hipError_t launch_quantize_blocks_chw(const void* X, tdq_dtype dt, int B, int C, int T, long long ld_c,
                                      long long ld_b, int kq, int kp, const Scalars& sc, uint8_t* Q,
                                      long long ld_q, float* bscale, float* bclip, long long ld_s,
                                      hipStream_t st);
hipError_t launch_fused_small(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                              const Scalars& sc, float* r, double* mean, double* m2, int* gid,
                              float* clip, float* scale, tdq_group_stats* stats,
                              unsigned* image_flags, uint8_t* Q, long long ld_q, hipStream_t st);
hipError_t launch_range_disparity(const void* X, tdq_dtype dt, int B, int T, int C, long long ld,
                                  float* token_median, float* token_max, float* disparity,
                                  float* max_abs, hipStream_t st);
hipError_t launch_tokenize_stats_chw(const void* X, tdq_dtype dt, int B, int C, int T, long long ld_c,
                                     long long ld_b, void* Xt, long long ld_xt, float* r, double* mean,
                                     double* m2, const SelectClear& cl, hipStream_t st);
hipError_t launch_quantize_f6(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                              const int* gid, const float* clip, const float* scale, uint8_t* F,
                              hipStream_t st);
hipError_t launch_pack_f6(const uint8_t* Q, long long ld, int R, int K, uint8_t* F, hipStream_t st);
hipError_t launch_w4a4_gemm_f6(const uint8_t* A6, const uint8_t* B6, int K, const int* gid,
                               const float* scale, int M, int T, int N, int G, const float* w_scale,
                               const float* bias, void* Y, tdq_dtype y_dt, long long ld_y,
                               int* acc_dump, hipStream_t st);
hipError_t launch_w4a4_gemm_blocks_f6(const uint8_t* A6, const uint8_t* B6, const float* bscale,
                                      long long ld_s, int M, int K, int N, const float* w_scale,
                                      const float* bias, void* Y, tdq_dtype y_dt, long long ld_y,
                                      hipStream_t st);
hipError_t launch_tokenize_chw(const void* X, tdq_dtype dt, int B, int C, int T, long long ld_c,
                               long long ld_b, void* Xt, long long ld_xt, hipStream_t st);
hipError_t launch_group_diag(const void* X, tdq_dtype dt, int B, int T, int C, long long ld, int G,
                             const int* gid, const float* clip, const float* scale,
                             unsigned long long* zero_count, unsigned long long* clipped_count,
                             hipStream_t st);
hipError_t launch_quantize_weight(const float* W, int N, int K, long long ld_in, uint8_t* Qw,
                                  long long ld_w, float* w_scale, hipStream_t st);
hipError_t launch_w4a4_gemm(const uint8_t* Qx, long long ld_q, const int* gid, const float* scale,
                            int M, int T, int K, int N, int G, const uint8_t* Qw, long long ld_w,
                            const float* w_scale, const float* bias, void* Y, tdq_dtype y_dt,
                            long long ld_y, int* acc_dump, hipStream_t st);

}  // namespace tdq
