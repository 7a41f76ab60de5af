// C ABI of the fault-injection campaign engine (see include/fi.h): argument
// checking, plan construction and kernel launches.  No device work happens
// anywhere else.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdarg>
#include <cstddef>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <unordered_set>
#include <vector>

#include "affected.hpp"
#include "aux_kernels.hpp"
#include "fi.h"
#include "gemm_fi.hpp"
#include "gemm_fi_multi.hpp"
#include "gemm_fi_small.hpp"
#include "tile_cfg.hpp"

namespace {

thread_local char g_err[512] = "";

fi_status fail(fi_status code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

#define FI_HIP(call)                                                                        \
  do {                                                                                      \
    hipError_t e_ = (call);                                                                 \
    if (e_ != hipSuccess)                                                                   \
      return fail(e_ == hipErrorOutOfMemory ? FI_OOM : FI_DEVICE, "%s failed: %s", #call,   \
                  hipGetErrorString(e_));                                                   \
  } while (0)

constexpr int PAD = 512;                       // row/column vectors are zero padded to this multiple
size_t padded(uint32_t n) { return ((size_t)n + PAD - 1) / PAD * PAD; }
// elements of the fault-free result's allocation: whole tiles of rows plus one tile width
size_t golden_elems(const fi_plan_desc& d) { return padded((uint32_t)d.M) * (size_t)d.N + PAD; }

using fi::kCfg;
using fi::kMulti;
using fi::kNumCfg;
using fi::kNumMulti;
using fi::TileCfg;
using fi::MultiCfg;

}  // namespace

// Counts and descriptors of one batch of the multi-trial kernel.  One set per stream a
// plan's batches have been enqueued on: batches on the same stream follow each other, batches
// on different streams may be in flight together and must not share this state.
struct BatchScratch {
  hipStream_t stream = nullptr;
  uint32_t* words = nullptr;  // [scratch_words(cap)], see TrialScratch
  uint32_t cap = 0;
  bool own = false;           // an allocation of its own, else part of the plan's
  // For the affected-only campaign, in words; only fi_plan_reserve makes them: behind scratch_words(cap) in the same allocation
  // where that is made with them, else an allocation of their own, as a graph may hold the addresses of the words.
  uint32_t* parts = nullptr;
  size_t parts_cap = 0;
  bool parts_own = false;
};

struct fi_plan {
  fi_plan_desc d = {};
  const uint16_t* A = nullptr;
  const uint16_t* B = nullptr;       // effective [N][ldb] K-contiguous matrix
  uint32_t ldb = 0;
  void* memory = nullptr;            // one allocation for everything below that the plan owns
  size_t memory_bytes = 0;
  uint16_t* Bt = nullptr;            // plan-owned transposed copy (b_layout 1) or NULL
  // K not a multiple of 64: copies of A and B ([M][K + kshift], [N][K + kshift]) with kshift zeros
  // in front of every row, for the kernels that want whole 64-wide k-tiles; else NULL and 0
  uint16_t* Apad = nullptr;
  uint16_t* Bpad = nullptr;
  uint32_t kshift = 0;
  float* c_star = nullptr;           // [M][N]
  float* s_abs = nullptr;            // [M][N]
  float* kra = nullptr;              // [pad(M)]
  float* cb = nullptr;               // [pad(N)]
  float* scratch = nullptr;          // 4 floats + 4 words: maxima, what plan_stats_kernel found, clean flags; GemmArgs::clear_word
  uint32_t epoch = 0;                // the last value that went into that word, by calls on this stream
  hipStream_t clear_stream = nullptr;
  float t_global = 0.0f;
  uint32_t n_clean_flagged = 0;      // elements of C* the plan's own detector flags
  bool factors_normal = false;       // see GemmArgs::normal
  bool plain_ok = false;             // the affected-only campaign's short comparison holds, see fi::kTinyFactor
  int cfg = 0;                       // index into kCfg
  int cfg_affected = 0;              // index into kCfg: the tiles that the affected-only campaign's batch limit counts
  int mcfg = -1;                     // index into kMulti, or -1: every trial through the single-trial kernel
  int prop_cfg = -1;                 // index into kMulti for the next-layer batch, or -1: single-trial kernel
  int group = 32;                    // trials sharing a tile back to back
  bool auto_cfg = true;              // no fi_plan_tune has chosen a tile configuration
  int device = 0;
  uint32_t* first_scratch = nullptr; // for kFirstTrials trials on the first stream that asks
  size_t first_parts = 0;            // words of parts behind it, see BatchScratch
  std::vector<BatchScratch> batch;   // per stream, see BatchScratch
  int n_cus = 8;                     // compute units of the device: grid of the persistent kernel
  int product_check = FI_PCHECK_NONE;
  unsigned long long* clocks = nullptr;   // caller's [12] counter sink, or NULL (fi_plan_set_clock_sink)
};

namespace {

// Where one wave per (trial, 32 x 32 tile) stops paying, in its MFMA steps per SIMD: K = 576, 3136 x 64, 46
// trials (317 steps) 29 : 31 us against the multi-trial kernel.
constexpr double kSmallSteps = 320.0;
// Beyond, for K > 64, while steps + 15 * tiles per SIMD <= 550: few long tiles, which it has the registers and the room to
// hide less of than those of many short ones.  Of 632 random batches of 280 to 1200 steps, this kernel : four trials per
// item, up to four tiles per SIMD 0.80 at 280 to 550 steps, four to eight tiles 0.84 up to 400, 0.93 up to 550, 1.0 and
// more beyond; by this line 1.035 over those of more than 320 steps, 1.8 % of them over 5 % slower.
constexpr double kSmallLong = 550.0, kSmallLongTile = 15.0;
// With short K a tile's fixed part - first loads, detector, counters - is most of it, which the eight trials
// of the multi-trial kernel share, on 64 x 64 tiles.  Small while
//   tiles per SIMD <= first + share * (that kernel's, in units of 32 x 32) + 5 per 1000 trials (partition):
// `first` is what its two more launches cost, without outputs 15 (K = 64, 1000 x 1003, accumulator faults: 15
// tiles 23 : 25 us, 27 tiles 30 : 26; K = 128, 1024^2: 22 tiles 31 : 26); its tiles cost 0.4 as much, and more with
// outputs (K = 16, 2000^2, FP32: 39 tiles 68 : 131 us, 140 tiles 190 : 199).  Chosen on 14149 random batches of up
// to 320 steps, all kinds and outputs, both kernels timed: the choice costs 0.3 % against the better of the two
// on average (always small 1.0 %, 3.2 % of the batches over 5 % slower, the worst 2.9 times; now 0.9 % of
// them).  The host does not know the kinds: with operand faults, two launches there, the lines lie higher.
constexpr double kSmallTiles = 15.0, kSmallTilesOut = 25.0, kSmallShare = 0.4, kSmallShareC = 0.5, kSmallShareH = 0.75;
// MFMA steps of one trial up to which its workgroup, on one CU, does not take longer than the launch it
// saves: 64 trials of 128^3 (128 steps) 8.8 : 10.6 us, of 128 x 128 x 512 13.3 : 10.8; with outputs to
// store 33 x 59 x 48 (12 steps) 9.4 : 10.7, 128^3 11.6 : 11.1.  Not beyond a trial per CU: 256 of 33 x 59 x
// 48 7.6 : 10.6, 512 12.0 : 10.5.
constexpr uint32_t kTrialSteps = 128, kTrialStepsOut = 16;
// The same for the next layer's batches, whose trials share nothing but B: a workgroup per strip of 32 rows x
// 128 columns, two resident per CU.  Up to 160 steps per SIMD, counted in whole strips, while
//   rounds of resident workgroups <= first + weight * (the other kernel's tiles, in 128 x 128, per two on a CU).
// Persistent kernel: first = 1 (K = 768, 512 x 768: 4 trials, 0.8 rounds, 17 : 23 us, 6 trials, 1.1 rounds, 27 : 24), 5
// where it also stores outputs (K = 576, 64 x 3136, 20 trials: 44 : 49), weight 2 (K = 256, 512^2: 15 trials 15 : 20, 27
// trials 36 : 23).  One-trial kernel, K not a multiple of 64: 1 and 4 (K = 16, 3648 x 31, 330 trials 348 : 134).  Chosen on
// 9850 random batches: over 5 % slower than the other kernel 2.4 % of them, 7.3 % without the second line.
// Against the persistent kernel without outputs the line is 0.8 and 1 from K = 640 on: its items have lost most of what
// they cost between two k-loops.  From K = 384 on it is 0.8 and 1.25, while that kernel takes one round: where a wave's
// elements all differ (a B fault in the layer before) it waits sixteen times for magnitude sums, which a short k-loop does
// not outweigh (K = 384, 57 x 61, 521 trials in a second round 31 : 45 us).  Of 11146 random batches small by the line above 2862
// are not by this one: with one row changed in each trial, every row, or one row of Inf they are 1.35, 1.54 and 1.21x faster,
// 0.1, 4.5 and 2.9 % of them over 4 % slower (K = 768, 203 x 623, 15 trials, one row 24 : 19 us).
// Not beyond K = 8192, a chain of k-tiles (16 x 16 x 4096 38 : 44, x 16384 127 : 113).
constexpr double kSmallPropagate = 160.0;
// The same for the plan's fault-free pass, which has two results (see compute_golden).
constexpr double kSmallSums = 768.0;
// Exponent field >= 144 <=> NOT (|c| <= largest binary32 below 2^17)
constexpr float kExponentBound = 131071.9921875f;

using fi::GemmArgs;

// Each (format, configuration) pair has its launcher in a translation unit of its own.
hipError_t launch_gemm(int mode, int dtype, int cfg, const GemmArgs& a, int n_blocks, hipStream_t s) {
#define FI_CASE(DT, CFG) \
  if (dtype == DT && cfg == CFG) return fi::launch_single_d##DT##_c##CFG(mode, a, n_blocks, s)
  FI_CASE(0, 0); FI_CASE(0, 1); FI_CASE(0, 2);
  FI_CASE(1, 0); FI_CASE(1, 1); FI_CASE(1, 2);
#undef FI_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_multi(int dtype, int mcfg, const GemmArgs& a, int n_blocks, hipStream_t s) {
#define FI_CASE(DT, MC) \
  if (dtype == DT && mcfg == MC) return fi::launch_multi_d##DT##_c##MC(a, n_blocks, s)
  FI_CASE(0, 0); FI_CASE(0, 1); FI_CASE(0, 2); FI_CASE(0, 3); FI_CASE(0, 4); FI_CASE(0, 5);
  FI_CASE(1, 0); FI_CASE(1, 1); FI_CASE(1, 2); FI_CASE(1, 3); FI_CASE(1, 4); FI_CASE(1, 5);
  FI_CASE(0, 6); FI_CASE(1, 6);
#undef FI_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_prop(int dtype, int mcfg, const GemmArgs& a, int n_blocks, hipStream_t s) {
#define FI_CASE(DT, MC) \
  if (dtype == DT && mcfg == MC) return fi::launch_prop_d##DT##_c##MC(a, n_blocks, s)
  FI_CASE(0, 4); FI_CASE(0, 5); FI_CASE(1, 4); FI_CASE(1, 5);
#undef FI_CASE
  return hipErrorInvalidValue;
}

// Eight trials per tile carry the least operand traffic per flop.  On the largest problems one eight-wave workgroup per CU on a
// 128 x 64 tile measured fastest (less traffic into LDS per flop); below that two four-wave
// workgroups on 64 x 64 tiles win, because the barriers and the per-item epilogue of one run
// under the MFMAs of the other (+2 .. 16 % on 1024^3, 512 x 3072 x 768 and 3136 x 64 x 576).
int pick_multi(const fi_plan_desc& d) {
  const double work = (double)d.M * (double)d.N * (double)d.K;
  return work >= 34359738368.0 /* 2^35 */ ? 2 : 3;
}

int pick_cfg(const fi_plan_desc& d) {
  if (d.N <= 64) return 2;
  if (d.M >= 512 && d.N >= 512) return 0;
  return 1;
}

// Matrix steps per SIMD if every (trial, 32 x 32 tile) were a wave of gemm_fi_small_kernel.
double small_steps(const fi_plan* p, uint32_t n_trials) {
  const fi_plan_desc& d = p->d;
  return (double)n_trials * ((d.M + 31) / 32) * ((d.N + 31) / 32) * (d.K / 16) / (4.0 * p->n_cus);
}

// And its tiles per SIMD, four trials to a workgroup.
double small_tiles(const fi_plan* p, uint32_t n_trials) {
  const fi_plan_desc& d = p->d;
  return (double)((d.M + 31) / 32) * ((d.N + 31) / 32) * ((n_trials + 3) / 4 * 4) / (4.0 * p->n_cus);
}

// Batches that gemm_fi_small_kernel serves, unless the caller has chosen a tile configuration.
bool use_small(const fi_plan* p, uint32_t n_trials, bool c_out, bool h_out) {
  const fi_plan_desc& d = p->d;
  const double steps = small_steps(p, n_trials);
  if (!p->auto_cfg || (steps > kSmallSteps && (d.K <= 64 || steps + kSmallLongTile * small_tiles(p, n_trials) > kSmallLong))) return false;
  if (n_trials <= 2) return true;                        // they fill a quarter of a group of eight at most
  const double simds = 4.0 * p->n_cus, n = (double)n_trials;
  const double tiles = small_tiles(p, n_trials);
  const double theirs = 4.0 * ((d.M + 63) / 64) * ((d.N + 63) / 64) * ((n_trials + 7) / 8 * 8) / simds;
  return tiles <= (c_out || h_out ? kSmallTilesOut : kSmallTiles) +
                      (h_out ? kSmallShareH : c_out ? kSmallShareC : kSmallShare) * theirs + 0.005 * n;
}

// The same for the next layer; persistent: the other kernel is the persistent one.
bool use_small_propagate(const fi_plan* p, uint32_t n_trials, bool c_out, bool persistent) {
  const fi_plan_desc& d = p->d;
  const double strips = (double)((d.N + 127) / 128 * 4) / ((d.N + 31) / 32);
  if (!p->auto_cfg || small_steps(p, n_trials) * strips > kSmallPropagate || d.K > 8192) return false;
  const double rounds = (double)n_trials * ((d.M + 31) / 32) * ((d.N + 127) / 128) / (2.0 * p->n_cus);
  const int bm = persistent ? kMulti[p->prop_cfg].bm : kCfg[p->cfg].bm, bn = persistent ? kMulti[p->prop_cfg].bn : kCfg[p->cfg].bn;
  const double theirs = (double)n_trials * ((d.M + bm - 1) / bm) * ((d.N + bn - 1) / bn) * (bm * bn / 16384.0) / (2.0 * p->n_cus);
  if (persistent && !c_out && (d.K >= 640 || (d.K >= 384 && theirs <= 1.0)))
    return rounds <= 0.8 + (d.K >= 640 ? 1.0 : 1.25) * theirs;
  return rounds <= (persistent && c_out ? 5.0 : 1.0) + (persistent ? 2.0 : 4.0) * theirs;
}

// Tile shape of a next-layer batch.  Below 2^35 multiply-adds the plan has the 128 x 128 shape, two workgroups
// per CU, one's epilogue under the other's MFMAs.  256 x 256 tiles read a third less from LDS per MFMA and half
// as much from L2, but nothing hides an item's epilogue, so they take long items in whole rounds
// that fill nine tenths of the chip, on shapes that they pad no more.  128 : 256, shapes of 256 to 1024 a side, in the mean of
// 9 to 12 each, whole tiles (250 to 1010 a side, ragged ones): K = 1024 0.94 .. 0.98; K = 1536 and 2048 two rounds 1.03 (1.01, the
// least 0.96), three rounds 1.05 (1.04, 0.99), six 1.07 and 1.11 (1.05 and 1.09); K = 2560 two rounds 1.14, six 1.18; K = 3072 1.12
// (1.11) and 1.17 (1.16).  512 x 768 x 3072, 256 trials (6 rounds) 535 us; 90 trials (2.1 rounds, a third empty) 264 : 243 the
// other way, 64 trials (1.5) 177 : 145, and 384^2 x 4096, which the larger tiles pad more, 260 : 214.  All of
// K a multiple of 128: an odd number of k-tiles runs without the early loads, its line is that of before, K >= 3072 and
// whole tiles.
constexpr uint32_t kPropLongK = 1536, kPropLongestK = 2560, kPropOddK = 3072;
int pick_prop(const fi_plan* p, uint32_t n_trials) {
  const fi_plan_desc& d = p->d;
  const uint32_t tm = (d.M + 255) / 256, tn = (d.N + 255) / 256;
  if (!p->auto_cfg || d.K < kPropLongK || (d.M + 127) / 128 != 2 * tm || (d.N + 127) / 128 != 2 * tn) return p->prop_cfg;
  const uint64_t items = (uint64_t)tm * tn * n_trials, cus = (uint64_t)p->n_cus;
  const uint64_t rounds = (items + cus - 1) / cus;
  if (d.K % 128 != 0 && (d.K < kPropOddK || d.M % 256 != 0 || d.N % 256 != 0)) return p->prop_cfg;
  return rounds >= (d.K >= kPropLongestK ? 2u : 3u) && 10 * items >= 9 * rounds * cus ? fi::kMultiOneTrial[0] : p->prop_cfg;
}

// Items of four trials, both parts of the batch in one launch, in the place of the 64 x 64 shape's eight trials and two
// launches.  Four share less, eight leave more of the chip without work at the end and take a launch more (some 4 us).
// Stores of outputs are hidden better by three workgroups per CU than by two.  With outputs four while
//   rounds of that shape's resident workgroups * k-tiles <= 100,
// without them while there are no more than six rounds as well.  From random batches, all kinds, eight : four in the mean
// and the share over 3 % slower with four: FP32 outputs (500 batches) 1.21, 1.8 %, 16-bit ones (500) 1.24, 2.4 %; beyond 100,
// up to 500 (300 each), 1.10, 2.0 %, and 1.14, 2.3 %, not taken.  Without outputs (3326) up to 100: one round 1.21, 5 %; two 1.15,
// 11 %; four 1.10, 11 %.  Further (700) by kind - accumulator and product, A, B faults, mixed: four to six rounds 0.99, 1.04, 1.06,
// 1.10; six to ten 0.97, 1.04, 1.06, 1.09; ten to twenty 0.96, 1.02, 1.03, 1.03; up to fifty 0.92, 1.06, 1.02, 0.92 (59 x 1012 x 256,
// 5056 mixed trials 282 : 347 us).  Beyond six rounds, up to 100, the operand faults alone therefore, whose accounting three
// workgroups per CU hide better as well, the others in eights; against eights for both 1.00, 1.02, 1.03, 1.03 in the mean of
// these batches.
// 512 x 3072 x 768, 8 trials with outputs 43.9 : 34.7 us, 3136 x 64 x 576, 128 trials with outputs 56.4 : 47.9.  Not
// for K <= 64, whose items are handed out in turn: operand faults, 142 x 167 x 64, 7802 trials 190 : 294.
constexpr uint64_t kFourWork = 100, kFourRounds = 6;
bool use_four(const fi_plan* p, uint32_t n_trials, bool outputs) {
  const fi_plan_desc& d = p->d;
  if (!p->auto_cfg || p->mcfg != 3 || d.K <= 64) return false;
  const MultiCfg& m = kMulti[3];
  const uint64_t items = (uint64_t)((d.M + m.bm - 1) / m.bm) * ((d.N + m.bn - 1) / m.bn) * (((uint64_t)n_trials + m.r - 1) / m.r);
  const uint64_t round = (uint64_t)m.wgs * (uint64_t)p->n_cus;
  return items * ((d.K + 63) / 64) <= kFourWork * round && (outputs || items <= kFourRounds * round);
}
// The second part alone.
bool use_four_apart(const fi_plan* p, uint32_t n_trials, bool outputs) { return !use_four(p, n_trials, outputs) && use_four(p, n_trials, true); }

// Batches that gemm_fi_trial_kernel serves.
bool use_trial(const fi_plan* p, uint32_t n_trials, bool c_out, bool h_out) {
  const fi_plan_desc& d = p->d;
  if (!use_small(p, n_trials, c_out, h_out) || n_trials > (uint32_t)p->n_cus || d.M > 512 || d.N > 512) return false;
  const uint32_t tiles = ((d.M + 31) / 32) * ((d.N + 31) / 32);
  return tiles <= 16 && tiles * (d.K / 16) <= (c_out || h_out ? kTrialStepsOut : kTrialSteps);
}

GemmArgs base_args(const fi_plan* p, int cfg = -1) {
  GemmArgs a;
  memset(&a, 0, sizeof(a));
  const TileCfg c = kCfg[cfg >= 0 ? cfg : p->cfg];
  a.A = p->A; a.B = p->B; a.lda = (uint32_t)p->d.lda; a.ldb = p->ldb;
  a.M = (int)p->d.M; a.N = (int)p->d.N; a.K = (int)p->d.K; a.kb = (int)p->d.k_block;
  a.tiles_m = (a.M + c.bm - 1) / c.bm;
  a.tiles_n = (a.N + c.bn - 1) / c.bn;
  a.kra = p->kra; a.cb = p->cb; a.gamma = p->d.gamma;
  a.bound_global = p->d.bound_mode != FI_BOUND_ROWCOL;
  a.t_global = p->t_global;
  a.normal = p->factors_normal;
  a.c_star = p->c_star; a.s_abs = p->s_abs;
  const size_t gold_bytes = golden_elems(p->d) * sizeof(float);
  a.c_star_bytes = gold_bytes < (1ull << 32) ? (uint32_t)gold_bytes : 0u;
  a.clocks = p->clocks;
  return a;
}

// Workgroups of the affected-only campaign's row / column kernel per (chunk of trials, item): one per tile of the other
// operand while that stays within some 2048 workgroups; beyond, each walks several tiles, and the workgroups that
// find no item (all of them in a batch of accumulator faults) stay few.
struct RowsGrid { uint32_t items, x_slots; };
RowsGrid rows_grid(const fi_plan_desc& d, uint32_t n_trials) {
  const int64_t items = ((int64_t)n_trials + fi::kRowsChunk - 1) / fi::kRowsChunk * fi::kRowsSlots;
  const int64_t tiles = ((int64_t)(d.M > d.N ? d.M : d.N) + fi::kRowsX - 1) / fi::kRowsX;
  int64_t per_slot = (tiles * items + 2047) / 2048;
  if (per_slot > tiles) per_slot = tiles;
  return {(uint32_t)items, (uint32_t)((tiles + per_slot - 1) / per_slot)};
}
// The affected-only campaign: the operand faults' rows and columns, and every record by the element kernel, which
// comes last where `parts` holds what the others have counted.
template <int DT>
fi_status launch_affected(const GemmArgs& a, const RowsGrid& rows, int n_cus, bool plain_ok, uint32_t* parts, hipStream_t s) {
  auto elements = [&]() {
    // A piece is one load instruction per row (512 k) up to K = 512, two beyond.  Three pieces in
    // flight cover the memory latency of a wave that has its CU to itself; from two waves per CU on
    // they take each other's LDS, and one piece in flight per wave is the better use of it.
    const unsigned waves = ((unsigned)a.n_trials + fi::kElemTrials - 1) / fi::kElemTrials;
    const bool wide = a.K > 512, deep = waves <= 2u * (unsigned)n_cus;
    const int pieces = wide ? (a.K + 1023) / 1024 : 1;
    const int bufs = pieces < (deep ? 4 : 2) ? pieces : deep ? 4 : 2;
    const size_t lds = (size_t)2 * fi::kElemTrials * (wide ? 2080 : 1056) * bufs;
#define FI_ELEMENTS(IPR, NBUF)                                                                                        \
  if (parts)                                                                                                         \
    hipLaunchKernelGGL((fi::affected_element_kernel<DT, IPR, NBUF, true>), dim3(waves), dim3(64), lds, s, a, parts,   \
                       (int)rows.x_slots);                                                                           \
  else                                                                                                               \
    hipLaunchKernelGGL((fi::affected_element_kernel<DT, IPR, NBUF, false>), dim3(waves), dim3(64), lds, s, a, parts, \
                       (int)rows.x_slots)
    if (!wide) { FI_ELEMENTS(1, 2); } else if (deep) { FI_ELEMENTS(2, 4); } else { FI_ELEMENTS(2, 2); }
#undef FI_ELEMENTS
  };
  if (!parts) elements();
  if (a.c_star_bytes != 0)
    hipLaunchKernelGGL((fi::affected_rows_kernel<DT, false>), dim3(rows.items * rows.x_slots), dim3(256), 0, s, a, (int)rows.x_slots, (int)plain_ok, parts);
  else
    hipLaunchKernelGGL((fi::affected_rows_kernel<DT, true>), dim3(rows.items * rows.x_slots), dim3(256), 0, s, a, (int)rows.x_slots, (int)plain_ok, parts);
  FI_HIP(hipGetLastError());
  if (parts) elements();
  FI_HIP(hipGetLastError());
  return FI_OK;
}

// C*, the magnitude sums S and the number of elements of C* that the plan's own detector flags, with
// the campaigns' sequence of matrix steps (so that a fault-free tile of a trial is bit-identical).
// Up to kSmallSums steps per SIMD one wave per 32 x 32 tile feeds both results from the same
// fragments, beyond that the 256 x 256 tiles run twice, the second time with the signs cleared.
// Whole plan creations, waves : tiles: 512 x 3072 x 768 64 : 122 us (24 workgroups of 256 x 256), 2048^3
// (512 steps) 113 : 188, 4096 x 4096 x 1024 (1024 steps) 207 : 178, 4096^3 496 : 359.
fi_status compute_golden(fi_plan* p, hipStream_t s) {
  GemmArgs a = base_args(p);
  a.n_trials = 1; a.group = 1;
  a.c_out = p->c_star;
  a.n_clean = reinterpret_cast<uint32_t*>(p->scratch + 5);
  a.maxima = p->d.bound_mode == FI_BOUND_GLOBAL ? p->scratch : nullptr;
  a.t_global = kExponentBound;          // looked at under FI_BOUND_EXPONENT only
  if (small_steps(p, 1) <= kSmallSums) {
    a.s_out = p->s_abs;
    a.tiles_m = (a.M + 31) / 32;
    a.tiles_n = (a.N + 31) / 32;
    const dim3 grid((unsigned)a.tiles_m * (((unsigned)a.tiles_n + 3) / 4));
    if (p->d.dtype == FI_BF16)
      hipLaunchKernelGGL((fi::gemm_fi_small_kernel<FI_BF16, 1, fi::SMALL_SUMS>), grid, dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL((fi::gemm_fi_small_kernel<FI_FP16, 1, fi::SMALL_SUMS>), grid, dim3(256), 0, s, a);
    FI_HIP(hipGetLastError());
    return FI_OK;
  }
  a.word_mask = 0xFFFFFFFFu;
  FI_HIP(launch_gemm(fi::MODE_GOLDEN, (int)p->d.dtype, p->cfg, a, a.tiles_m * a.tiles_n, s));
  a.word_mask = 0x7FFF7FFFu;
  a.c_out = p->s_abs;
  a.n_clean = nullptr;
  FI_HIP(launch_gemm(fi::MODE_GOLDEN, (int)p->d.dtype, p->cfg, a, a.tiles_m * a.tiles_n, s));
  return FI_OK;
}

// The architecture of a device does not change: asked once per device (the properties take some
// hundred microseconds).
fi_status check_device() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(FI_STATE, "no HIP device: %s", hipGetErrorString(e));
  static std::atomic<uint64_t> known{0};               // bit d: device d is a gfx950
  const uint64_t bit = dev < 64 ? 1ull << dev : 0ull;
  if (known.load(std::memory_order_relaxed) & bit) return FI_OK;
  hipDeviceProp_t prop;
  e = hipGetDeviceProperties(&prop, dev);
  if (e != hipSuccess) return fail(FI_STATE, "hipGetDeviceProperties: %s", hipGetErrorString(e));
  if (strncmp(prop.gcnArchName, "gfx950", 6) != 0)
    return fail(FI_STATE, "device %d is %s; this library is built for gfx950 only", dev, prop.gcnArchName);
  known.fetch_or(bit, std::memory_order_relaxed);
  return FI_OK;
}

fi_status check_desc(const fi_plan_desc* d, float* gamma_out) {
  if (!d) return fail(FI_INVALID_ARG, "desc is NULL");
  if (d->M == 0 || d->N == 0 || d->K == 0) return fail(FI_INVALID_ARG, "M, N, K must be non-zero");
  if (d->k_block == 0 || d->k_block % 16 != 0)
    return fail(FI_INVALID_ARG, "k_block must be a non-zero multiple of 16 (got %u)", d->k_block);
  if (d->K % d->k_block != 0)
    return fail(FI_INVALID_ARG, "K (%u) must be a multiple of k_block (%u)", d->K, d->k_block);
  if (d->dtype != FI_FP16 && d->dtype != FI_BF16)
    return fail(FI_UNSUPPORTED, "dtype %u: only FP16 (0) and BF16 (1) operands", d->dtype);
  if (d->b_layout > 1) return fail(FI_INVALID_ARG, "b_layout must be 0 or 1");
  if (d->bound_mode > FI_BOUND_EXPONENT) return fail(FI_INVALID_ARG, "bound_mode must be 0, 1 or 2");
  // Default slack: 1 + 2^-11 for K <= 4096, growing in proportion beyond (a K-term FP32
  // accumulation inflates a sum by at most (1 + 2^-24)^(K-1); twice that, in units of 4096 terms).
  float g = d->gamma == 0.0f ? 1.0f + (float)((d->K + 4095u) / 4096u) / 2048.0f : d->gamma;
  if (!(g >= 1.0f) || !(g <= 3.0e38f)) return fail(FI_INVALID_ARG, "gamma must be finite and >= 1");
  if (d->K > 65536u) return fail(FI_UNSUPPORTED, "K > 65536");
  if (d->M > (1u << 24) || d->N > (1u << 24)) return fail(FI_UNSUPPORTED, "M or N > 2^24");
  if (gamma_out) *gamma_out = g;
  return FI_OK;
}

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

// Live plans.  A handle is looked up here before it is dereferenced, so a destroyed (or
// never created) plan is an error and not a read of freed memory.
std::mutex g_live_mu;
std::unordered_set<const fi_plan*> g_live;

fi_status check_plan(const fi_plan* p) {
  if (!p) return fail(FI_INVALID_ARG, "plan is NULL");
  std::lock_guard<std::mutex> lock(g_live_mu);
  if (g_live.find(p) == g_live.end()) return fail(FI_STATE, "plan is not live (destroyed or never created)");
  return FI_OK;
}

// Device memory of destroyed plans, for the plans that follow: a sweep over a model's layers makes and destroys one
// after the other.  A plan of 512 x 3072 x 768 (12 MB) took 55 us to make and 24 to destroy, 85 with eight trials between
// them 63; now 37, 1 and 37.  Plans below 2 MiB, whose memory the runtime keeps itself, 37 and 30 us to make.  At most
// kPoolBlocks blocks and kPoolBytes on each device; a block that kPoolAge further plans had no use for, the oldest
// where there is no room and all of them where the device is out of memory are given back.  fi_plan_destroy has waited for
// the device before a block comes here.
struct PoolBlock {
  void* ptr;
  size_t bytes;
  uint64_t born;              // plans made so far, on this device
};
constexpr int kMaxDevices = 64;
constexpr size_t kPoolBlocks = 4, kPoolBytes = 256u << 20;
constexpr uint64_t kPoolAge = 16;
std::mutex g_pool_mu;
std::vector<PoolBlock> g_pool[kMaxDevices];
uint64_t g_pool_plans[kMaxDevices] = {};

hipError_t pool_release(std::vector<PoolBlock>& blocks, size_t keep, uint64_t now) {
  hipError_t failed = hipSuccess;
  size_t kept = 0;
  std::vector<PoolBlock> stay;
  for (size_t i = blocks.size(); i-- > 0;) {              // youngest first
    if (stay.size() < kPoolBlocks && kept + blocks[i].bytes <= keep && now - blocks[i].born <= kPoolAge) {
      kept += blocks[i].bytes;
      stay.insert(stay.begin(), blocks[i]);
    } else {
      const hipError_t e = hipFree(blocks[i].ptr);
      if (e != hipSuccess) failed = e;
    }
  }
  blocks.swap(stay);
  return failed;
}

// An allocation on the current device; where there is no memory for it the pool's blocks are given back.
hipError_t device_alloc(int device, void** ptr, size_t bytes) {
  hipError_t e = hipMalloc(ptr, bytes);
  if (e == hipErrorOutOfMemory && device >= 0 && device < kMaxDevices) {
    (void)hipGetLastError();
    std::lock_guard<std::mutex> lock(g_pool_mu);
    (void)pool_release(g_pool[device], 0, 0);
    e = hipMalloc(ptr, bytes);
  }
  return e;
}

// A block of at least `bytes` on the current device, not more than twice as large; *got is its size.
hipError_t pool_take(int device, size_t bytes, void** ptr, size_t* got) {
  if (device >= 0 && device < kMaxDevices) {
    std::lock_guard<std::mutex> lock(g_pool_mu);
    std::vector<PoolBlock>& blocks = g_pool[device];
    const uint64_t now = ++g_pool_plans[device];
    size_t best = blocks.size();
    for (size_t i = 0; i < blocks.size(); ++i)
      if (blocks[i].bytes >= bytes && blocks[i].bytes / 2 <= bytes && (best == blocks.size() || blocks[i].bytes < blocks[best].bytes))
        best = i;
    if (best != blocks.size()) {
      *ptr = blocks[best].ptr;
      *got = blocks[best].bytes;
      blocks.erase(blocks.begin() + best);
      return hipSuccess;
    }
    (void)pool_release(blocks, kPoolBytes, now);
  }
  *got = bytes;
  return device_alloc(device, ptr, bytes);
}

// Back from a plan on `device`; nothing on it reads or writes the block any more.
void pool_give(int device, void* ptr, size_t bytes) {
  if (device < 0 || device >= kMaxDevices || bytes > kPoolBytes) {
    (void)hipFree(ptr);
    return;
  }
  std::lock_guard<std::mutex> lock(g_pool_mu);
  g_pool[device].push_back({ptr, bytes, g_pool_plans[device]});
  (void)pool_release(g_pool[device], kPoolBytes, g_pool_plans[device]);
}

// Pinned host words into which a plan's creation reads back eight of the device's, in slots of one cache line, made once
// and held (4 KB): into pageable memory the copy is staged, some 8 us.  (A kernel that
// writes them and a mark to wait for took 3 us less here and 20 us more in the next synchronisation.)
constexpr int kHostSlots = 64, kHostSlotWords = 16;
std::mutex g_host_mu;
uint32_t* g_host_words = nullptr;
uint64_t g_host_used = 0;              // bit: slot in use

// A slot, or -1: none free, or no pinned memory.
int host_slot_take() {
  std::lock_guard<std::mutex> lock(g_host_mu);
  if (!g_host_words &&
      hipHostMalloc(reinterpret_cast<void**>(&g_host_words), kHostSlots * kHostSlotWords * sizeof(uint32_t), hipHostMallocPortable) != hipSuccess) {
    g_host_words = nullptr;
    (void)hipGetLastError();
    return -1;
  }
  for (int i = 0; i < kHostSlots; ++i)
    if (!(g_host_used >> i & 1)) {
      g_host_used |= 1ull << i;
      return i;
    }
  return -1;
}
void host_slot_give(int slot) {
  std::lock_guard<std::mutex> lock(g_host_mu);
  g_host_used &= ~(1ull << slot);
}
hipError_t host_slots_release() {
  std::lock_guard<std::mutex> lock(g_host_mu);
  if (!g_host_words || g_host_used != 0) return hipSuccess;
  uint32_t* const words = g_host_words;
  g_host_words = nullptr;
  return hipHostFree(words);
}

// Eight words of the device, once everything on the stream has run.
fi_status read_back(const uint32_t* d_words, uint32_t* out, hipStream_t s) {
  const int slot = host_slot_take();
  uint32_t* const host = slot >= 0 ? g_host_words + slot * kHostSlotWords : out;
  hipError_t e = hipMemcpyAsync(host, d_words, 8 * sizeof(uint32_t), hipMemcpyDeviceToHost, s);
  const hipError_t es = hipStreamSynchronize(s);          // in any case before the slot goes back
  if (e == hipSuccess) e = es;
  if (slot >= 0) {
    memcpy(out, host, 8 * sizeof(uint32_t));
    host_slot_give(slot);
  }
  return e == hipSuccess ? FI_OK : fail(FI_DEVICE, "plan kernels failed: %s", hipGetErrorString(e));
}

// idle: the plan's device has been waited for.  Where that failed (a thread captures in the global mode, say), or the device
// could not be selected, the memory serves no other plan.
void free_plan_buffers(fi_plan* p, bool idle) {
  if (p->memory && idle) pool_give(p->device, p->memory, p->memory_bytes);
  else if (p->memory) (void)hipFree(p->memory);
  p->memory = nullptr;
  for (BatchScratch& b : p->batch) {
    if (b.own) (void)hipFree(b.words);
    if (b.parts_own) (void)hipFree(b.parts);
  }
  p->batch.clear();
}

// Trials that the scratch inside the plan's own allocation holds (8 KB).  Not more: an allocation that it
// takes past 2 MiB costs 27 us more to make and give back (a layer of 1010 x 161 x 272 with 58 KB 75 -> 102 us).
constexpr uint32_t kFirstTrials = 256;
// words: part counts, work counters, descriptors, each 256-byte aligned
constexpr size_t kScratchQueue = 64, kScratchDesc = kScratchQueue + 2 * fi::kQueueWords;
constexpr size_t scratch_words(uint32_t n) { return (kScratchDesc + ((size_t)n + 16) * fi::kMultiDescWords + 63) / 64 * 64; }

// Slots from which workgroups leave their counts in scratch.  Added to the record : left, K = 256, A faults: 4 slots
// (512^2) 3000 trials 16.5 : 15.6 us, 400 trials 14.7 : 14.9; 8 (1000^2) 19.2 : 17.6, 15.4 : 15.7; 16 (2048^2) 26.5 : 21.2,
// 16.3 : 15.8; 32 (4096^2) 49.4 : 38.9, 18.1 : 16.3, 8 trials 16.2 : 14.2.  The slots are those of the longer side; where
// the faults lie along the other, of one to four slots, it costs up to half a microsecond (3072 x 512, 400 trials 15.1 : 15.7).
constexpr uint32_t kPartSlots = 8;
// Words of those workgroups' parts, for this number of trials and any smaller one: x_slots <= min(tiles, 2048 / items + 1).
// It falls below kPartSlots beyond kPartChunks chunks (16384 trials), so that no more are ever used: 4.3 MB.
constexpr size_t kPartChunks = 2048 / ((kPartSlots - 1) * fi::kRowsSlots);
size_t parts_words(const fi_plan_desc& d, uint32_t n_trials) {
  size_t chunks = ((size_t)n_trials + fi::kRowsChunk - 1) / fi::kRowsChunk;
  if (chunks > kPartChunks) chunks = kPartChunks;
  const size_t tiles = ((size_t)(d.M > d.N ? d.M : d.N) + fi::kRowsX - 1) / fi::kRowsX;
  const size_t bound = 2048 / fi::kRowsSlots + 1 + chunks;   // of chunks * x_slots
  if (tiles < kPartSlots) return 0;
  return (chunks * tiles < bound ? chunks * tiles : bound) * (n_trials < fi::kRowsChunk ? n_trials : fi::kRowsChunk) * fi::kPartWords;
}

// What only makes a call faster is allocated without a word to captures of other threads, which a plain allocation would
// break, and not at all where `s` itself is capturing.
struct BesideCaptures {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  BesideCaptures() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  ~BesideCaptures() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};
bool capturing(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

// The batch scratch of `stream`, holding at least n trials.  Allocates on the first batch of a
// stream and when a batch is larger than any before on it (the replaced buffers are freed,
// which waits for device work that may still read them), and replaces them then alone; not for up to kFirstTrials trials on the
// plan's first stream.  Batches of the small kernels do not use it but size it all the same: a tile
// configuration chosen later sends the same batch to the multi-trial kernel, which must not allocate then.
// want_parts: with the affected-only campaign's parts, if there is memory for them; once there they stay, also where a
// larger batch replaces the scratch.
fi_status batch_scratch(fi_plan* p, hipStream_t stream, uint32_t n, BatchScratch** out, bool want_parts = false) {
  BatchScratch* b = nullptr;
  for (BatchScratch& x : p->batch)
    if (x.stream == stream) b = &x;
  if (!b) {
    if (p->batch.size() >= 64) return fail(FI_STATE, "a plan serves at most 64 distinct streams");
    p->batch.emplace_back();
    b = &p->batch.back();
    b->stream = stream;
    if (p->batch.size() == 1) {
      b->words = p->first_scratch;
      b->cap = kFirstTrials;
      b->parts = b->words + scratch_words(kFirstTrials);
      b->parts_cap = p->first_parts;
    }
  }
  auto alloc = [&](uint32_t** words, size_t n_words) { return device_alloc(p->device, reinterpret_cast<void**>(words), n_words * sizeof(uint32_t)); };
  size_t parts = want_parts ? parts_words(p->d, n) : 0;
  if (b->cap < n) {
    if (b->own) {
      if (!b->parts_own && b->parts == b->words + scratch_words(b->cap)) {   // in that allocation: what was reserved stays so
        if (parts < b->parts_cap) parts = b->parts_cap;
        b->parts = nullptr; b->parts_cap = 0;
      }
      (void)hipFree(b->words);
    }
    b->words = nullptr; b->cap = 0; b->own = false;
    if (b->parts_cap < parts) {
      if (alloc(&b->words, scratch_words(n) + parts) == hipSuccess) {
        if (b->parts_own) (void)hipFree(b->parts);
        b->parts = b->words + scratch_words(n);
        b->parts_cap = parts;
        b->parts_own = false;
      } else {
        b->words = nullptr;
        (void)hipGetLastError();
      }
    }
    if (!b->words) FI_HIP(alloc(&b->words, scratch_words(n)));
    b->cap = n;
    b->own = true;
  } else if (b->parts_cap < parts && !capturing(stream)) {
    const BesideCaptures beside;
    uint32_t* more = nullptr;
    if (alloc(&more, parts) == hipSuccess) {
      if (b->parts_own) (void)hipFree(b->parts);
      b->parts = more;
      b->parts_cap = parts;
      b->parts_own = true;
    } else {
      (void)hipGetLastError();
    }
  }
  *out = b;
  return FI_OK;
}

// Two chunks or more per workgroup, the same number for all of them, only beyond 16384 chunks: 8192 and 32768
// workgroups measured within 3 % of it, 2048 up to 20 % slower on rows that no chunk fits, a workgroup
// per chunk 18 % slower on 100 x 1000 x 1003 (84 : 71 us); neighbouring chunks instead of strided ones 2 %.
constexpr size_t kDetectGrid = 16384;
// Rows from which the waves of a workgroup hand over what they have flagged together.  With every element
// flagged 4 x 4096 x 4096 took 755 us wave by wave and 202 together, 2048 x 2048 191 and 53 (with a
// workgroup per row, before the flat walk, 392 and 98); with none flagged it costs up to 1 us where many
// workgroups follow each other on a CU (128 x 3136 x 64 17.3 : 18.4), and short rows gained most from the flat
// walk anyway (flagged throughout 1241 -> 130 us).
constexpr uint32_t kDetectTogether = 1024;

// The detector / corrector on [batch][M][N] outputs: whole vectors where the outputs (and flags)
// are aligned for them and a vector spans two rows at most, else element by element.
hipError_t launch_detect(const fi_plan* p, float* d_c, uint32_t batch, uint32_t policy, uint8_t* d_flags,
                         uint32_t* d_n_flagged, uint32_t* clear_word, uint32_t epoch, hipStream_t s) {
  const fi_plan_desc& d = p->d;
  const bool vec = d.N >= 4 && (reinterpret_cast<uintptr_t>(d_c) & 15u) == 0 &&
                   (reinterpret_cast<uintptr_t>(d_flags) & 3u) == 0;
  // four vectors in flight per lane once that leaves eight workgroups for every CU, else one: small
  // outputs are a matter of latency, and more lanes share it
  const size_t total = (size_t)batch * d.M * d.N, one = (size_t)256 * (vec ? 4 : 1);
  const bool deep = total >= one * 4 * 8 * (size_t)p->n_cus;
  const size_t chunk = one * (deep ? 4 : 1);
  const size_t chunks = (total + chunk - 1) / chunk;
  const size_t rounds = (chunks + kDetectGrid - 1) / kDetectGrid;   // the same for every workgroup, or one less
  const dim3 grid((unsigned)((chunks + rounds - 1) / rounds)), block(256);
  fi::DetectStep step;
  step.elems = grid.x * chunk;
  const size_t rows = step.elems / d.N;
  step.col = (uint32_t)(step.elems % d.N);
  step.row = (uint32_t)(rows % d.M);
  step.trial = (uint32_t)(rows / d.M);
  step.together = vec && d.N % 4 == 0 && d.N >= kDetectTogether;
  const int global = d.bound_mode != FI_BOUND_ROWCOL;
#define FI_DETECT(VEC, ROW4, UNROLL)                                                                               \
  hipLaunchKernelGGL((fi::detect_correct_kernel<VEC, ROW4, UNROLL>), grid, block, 0, s, d_c, batch, d.M, d.N, p->kra, \
                     p->cb, d.gamma, global, p->t_global, (int)policy, p->c_star, d_flags, d_n_flagged, step, clear_word, epoch)
  if (!vec) {
    if (deep) FI_DETECT(1, false, 4); else FI_DETECT(1, false, 1);
  } else if (d.N % 4 == 0) {
    if (deep) FI_DETECT(4, true, 4); else FI_DETECT(4, true, 1);
  } else {
    if (deep) FI_DETECT(4, false, 4); else FI_DETECT(4, false, 1);
  }
#undef FI_DETECT
  return hipGetLastError();
}

fi_status build_plan(fi_plan* p, const void* d_A, const void* d_B, hipStream_t s) {
  const fi_plan_desc& d = p->d;
  const size_t mn = (size_t)d.M * d.N;
  // C* is padded to whole 256-row tiles plus one tile width (zeros): the next layer's kernel
  // reads the tile-shaped neighbourhood of its outputs without clamping rows or columns, and so
  // does the affected-only campaign (its loads of the sums end at the last one: for one row of 2^18
  // columns padding both would take 1 GiB instead of 0.5).
  const size_t mn_pad = golden_elems(d);
  p->A = static_cast<const uint16_t*>(d_A);
  p->kshift = d.K % 64 ? 64 - d.K % 64 : 0;
  const uint32_t kp = d.K + p->kshift;
  // One allocation: C* with its padding and the scratch words behind it (zeroed together), S, the
  // statistics, the operand copies that this problem needs, and a first batch scratch.
  size_t bytes = 0;
  auto place = [&](size_t n) {
    const size_t at = bytes;
    bytes += (n + 255) / 256 * 256;
    return at;
  };
  const size_t at_c = place((mn_pad + 9) * sizeof(float)), at_s = place(mn * sizeof(float));
  const size_t at_kra = place(padded(d.M) * sizeof(float)), at_cb = place(padded(d.N) * sizeof(float));
  const size_t at_bt = place(d.b_layout ? (size_t)d.N * d.K * sizeof(uint16_t) : 0);
  const size_t at_ap = place(p->kshift ? (size_t)d.M * kp * sizeof(uint16_t) : 0);
  const size_t at_bp = place(p->kshift ? (size_t)d.N * kp * sizeof(uint16_t) : 0);
  const size_t at_scratch = place(scratch_words(kFirstTrials) * sizeof(uint32_t));
  // parts as well, unless they take the allocation past 2 MiB
  p->first_parts = parts_words(d, kFirstTrials);
  if (bytes <= (2u << 20) && bytes + p->first_parts * sizeof(uint32_t) > (2u << 20)) p->first_parts = 0;
  place(p->first_parts * sizeof(uint32_t));
  FI_HIP(pool_take(p->device, bytes, &p->memory, &p->memory_bytes));
  uint8_t* const base = static_cast<uint8_t*>(p->memory);
  p->c_star = reinterpret_cast<float*>(base + at_c);
  p->scratch = p->c_star + mn_pad;
  p->s_abs = reinterpret_cast<float*>(base + at_s);
  p->kra = reinterpret_cast<float*>(base + at_kra);
  p->cb = reinterpret_cast<float*>(base + at_cb);
  p->first_scratch = reinterpret_cast<uint32_t*>(base + at_scratch);
  const size_t zeros = mn_pad + 9 - mn;
  hipLaunchKernelGGL(fi::fill_u32_kernel, dim3((unsigned)(zeros < 262144 ? (zeros + 255) / 256 : 1024)), dim3(256), 0, s,
                     reinterpret_cast<uint32_t*>(p->c_star + mn), zeros, 0u);
  FI_HIP(hipGetLastError());
  if (d.b_layout == 0) {
    p->B = static_cast<const uint16_t*>(d_B);
    p->ldb = (uint32_t)d.ldb;
  } else {
    p->Bt = reinterpret_cast<uint16_t*>(base + at_bt);
    dim3 grid((d.N + 31) / 32, (d.K + 31) / 32);
    hipLaunchKernelGGL(fi::transpose16_kernel, grid, dim3(256), 0, s,
                       static_cast<const uint16_t*>(d_B), (uint32_t)d.ldb, p->Bt, d.K, (int)d.K, (int)d.N);
    FI_HIP(hipGetLastError());
    p->B = p->Bt;
    p->ldb = d.K;
  }
  if (p->kshift) {
    p->Apad = reinterpret_cast<uint16_t*>(base + at_ap);
    p->Bpad = reinterpret_cast<uint16_t*>(base + at_bp);
    hipLaunchKernelGGL(fi::pad_front16_kernel, dim3(1024), dim3(256), 0, s, p->A, (uint32_t)d.lda, p->Apad, d.M, d.K,
                       p->kshift);
    hipLaunchKernelGGL(fi::pad_front16_kernel, dim3(1024), dim3(256), 0, s, p->B, p->ldb, p->Bpad, d.N, d.K,
                       p->kshift);
    FI_HIP(hipGetLastError());
  }
  uint32_t* const words = reinterpret_cast<uint32_t*>(p->scratch);   // maxima, -, -, found, clean flags
  const uint32_t rows_a = (uint32_t)padded(d.M), rows_b = (uint32_t)padded(d.N);
  const uint32_t stat_blocks = (rows_a + rows_b) / fi::kStatWaves;     // a multiple of 32: rows are padded to 512
  const dim3 stat_grid(stat_blocks < (uint32_t)p->n_cus ? stat_blocks : (uint32_t)p->n_cus), stat_block(fi::kStatWaves * 64);
  if (d.dtype == FI_FP16)
    hipLaunchKernelGGL(fi::plan_stats_kernel<FI_FP16>, stat_grid, stat_block, 0, s, p->A, (uint32_t)d.lda, d.M, rows_a,
                       p->B, p->ldb, d.N, rows_b, d.K, p->kra, p->cb, words, words + 4, fi::kTinyFactor);
  else
    hipLaunchKernelGGL(fi::plan_stats_kernel<FI_BF16>, stat_grid, stat_block, 0, s, p->A, (uint32_t)d.lda, d.M, rows_a,
                       p->B, p->ldb, d.N, rows_b, d.K, p->kra, p->cb, words, words + 4, fi::kTinyFactor);
  FI_HIP(hipGetLastError());
  fi_status st = compute_golden(p, s);
  if (st != FI_OK) return st;
  uint32_t host_words[8];
  st = read_back(reinterpret_cast<const uint32_t*>(p->scratch), host_words, s);
  if (st != FI_OK) return st;
  float host[8];
  memcpy(host, host_words, sizeof(host));
  uint32_t badw;
  memcpy(&badw, &host[4], 4);
  if (badw & 1u) return fail(FI_INVALID_ARG, "A or B holds an Inf or NaN: the magnitude bound is undefined");
  // T = fl32(fl32(fl32(K*ra_max) * cb_max) * gamma), one rounding per product
  volatile float t = host[0] * host[1];
  t = t * d.gamma;
  p->t_global = t;
  if (d.bound_mode == FI_BOUND_EXPONENT) p->t_global = kExponentBound;
  p->factors_normal = !(badw & 2u) && host[1] * d.gamma <= 3.4028234e38f && t < 1.7e38f;
  p->plain_ok = p->t_global < 1.7e38f && (d.bound_mode != FI_BOUND_ROWCOL || p->factors_normal);
  // How many elements of the fault-free result the plan's own detector flags (none under the
  // operand-derived bounds with gamma at or above the default; possible under the exponent-only
  // bound or a caller's smaller gamma).  The affected-only campaign relies on it being 0.
  memcpy(&p->n_clean_flagged, &host[5], 4);
  return FI_OK;
}

// One handle for the streams of all host threads: what calls on it have in flight need not follow each other, so nothing
// but what a multi-trial batch cannot do without is kept by it.
bool shared_handle(hipStream_t s) { return s == hipStreamPerThread; }

// The small kernels clear the records themselves, and the detector its counters, through a word of the plan (clear_once.hpp): on
// the first stream that a plan's such batch comes on, whose calls follow each other - for good, as nothing here tells when its last
// one has run - outside capture (a graph may be replayed beside them, and with the same number each time), and up to
// kClearTrials, which one workgroup clears in half a microsecond (512 trials on 64 x 64 x 128 by one wave 12.2 us, by four
// 10.5).  Else a launch in front does.
constexpr uint32_t kClearTrials = 512;
bool clear_in_kernel(fi_plan* p, uint32_t n_trials, hipStream_t s, GemmArgs* a) {
  if (n_trials > kClearTrials || shared_handle(s) || p->epoch >= 0xFFFFFFFEu) return false;
  if (p->epoch != 0 && p->clear_stream != s) return false;
  if (capturing(s)) return false;
  p->epoch += 2;                                          // even, see clear_once.hpp
  p->clear_stream = s;
  a->clear_word = reinterpret_cast<uint32_t*>(p->scratch + 8);
  a->epoch = p->epoch;
  return true;
}

// Where one batch of the multi-trial kernel keeps its two part counts, its work counters and the
// per-trial descriptors; all of it is rewritten by the partition kernel of every batch.
struct TrialScratch {
  uint32_t* counts = nullptr;   // [2]
  uint32_t* queue = nullptr;    // [2 * kQueueWords]
  uint32_t* desc = nullptr;     // [(n_trials + 16) * kMultiDescWords]
  explicit TrialScratch(uint32_t* words) : counts(words), queue(words + kScratchQueue), desc(words + kScratchDesc) {}
  TrialScratch() = default;
};

fi_status check_batch_args(const fi_plan* plan, const fi_fault* d_faults, uint32_t n_trials, uint32_t policy,
                           const fi_trial_result* d_results) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (!d_faults || !d_results) return fail(FI_INVALID_ARG, "d_faults and d_results must be non-NULL");
  if (n_trials == 0) return fail(FI_INVALID_ARG, "n_trials is 0");
  if (policy > FI_CORRECT_RECOMPUTE) return fail(FI_INVALID_ARG, "unknown correction policy %u", policy);
  return FI_OK;
}

// As many of a workgroup's four waves on trials of one tile as there are trials: they share most.
template <int DT>
void launch_small(const GemmArgs& a, hipStream_t s) {
  const unsigned n = (unsigned)a.n_trials;
  auto blocks = [&](unsigned tpw) {
    const unsigned tiles = 4 / tpw;
    return dim3((n + tpw - 1) / tpw * (unsigned)a.tiles_m * (((unsigned)a.tiles_n + tiles - 1) / tiles));
  };
  if (n >= 3)
    hipLaunchKernelGGL((fi::gemm_fi_small_kernel<DT, 4, fi::SMALL_CAMPAIGN>), blocks(4), dim3(256), 0, s, a);
  else if (n == 2)
    hipLaunchKernelGGL((fi::gemm_fi_small_kernel<DT, 2, fi::SMALL_CAMPAIGN>), blocks(2), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((fi::gemm_fi_small_kernel<DT, 1, fi::SMALL_CAMPAIGN>), blocks(1), dim3(256), 0, s, a);
}

// One campaign batch: record fill, then either the partition kernel and the two launches of
// the multi-trial kernel (scratch in `ts`), or one launch of the one-trial kernel.
fi_status inject_batch(fi_plan* plan, const fi_fault* d_faults, uint32_t n_trials, uint32_t policy,
                       fi_trial_result* d_results, float* d_c_out, hipStream_t s, const TrialScratch& ts,
                       bool may_clear, uint16_t* d_h_out = nullptr) {
  GemmArgs a = base_args(plan);
  const uint64_t blocks = (uint64_t)a.tiles_m * a.tiles_n * n_trials;
  if (blocks >= (1ull << 31)) return fail(FI_UNSUPPORTED, "tiles x trials exceeds 2^31 workgroups; split the batch");
  const bool four = use_four(plan, n_trials, d_c_out != nullptr || d_h_out != nullptr);
  const bool apart = use_four_apart(plan, n_trials, d_c_out != nullptr || d_h_out != nullptr);
  const MultiCfg mc = four ? fi::kMultiFour : kMulti[plan->mcfg >= 0 ? plan->mcfg : 0];
  GemmArgs m = a;
  uint64_t mblocks = 0;
  if (plan->mcfg >= 0) {
    m.tiles_m = (a.M + mc.bm - 1) / mc.bm;
    m.tiles_n = (a.N + mc.bn - 1) / mc.bn;
    if (plan->kshift) {
      // whole k-tiles: the front-padded copies (bit-identical results, see pad_front16_kernel)
      m.A = plan->Apad; m.B = plan->Bpad;
      m.K = a.K + (int)plan->kshift;
      m.lda = m.ldb = (uint32_t)m.K;
    }
    // Persistent workgroups, as many per CU as the configuration's register budget admits.  They
    // take their items from counters, one per XCD, or walk the work list with the grid as stride
    // (see gemm_fi_multi_kernel); for both the grid has to be a multiple of 8 where it is not the
    // work list's length.
    const uint64_t groups = ((uint64_t)n_trials + mc.r - 1) / mc.r + (four ? 1 : 0);   // either part may end in a partial one
    const uint64_t items = (uint64_t)m.tiles_m * m.tiles_n * groups;
    if (items >= (1ull << 31)) return fail(FI_UNSUPPORTED, "tiles x trials exceeds 2^31 work items; split the batch");
    const uint64_t cus = (uint64_t)(plan->n_cus / 8 * 8) * (uint64_t)mc.wgs;
    mblocks = items < cus ? items : cus;
  }
  for (GemmArgs* g : {&a, &m}) {
    g->n_trials = (int)n_trials;
    g->group = plan->group;
    g->faults = d_faults;
    g->results = d_results;
    g->c_out = d_c_out;
    g->h_out = d_h_out;
    g->policy = (int)policy;
    g->product_check = plan->product_check;
  }
  if (use_trial(plan, n_trials, d_c_out != nullptr, d_h_out != nullptr)) {
    a.tiles_m = (a.M + 31) / 32;
    a.tiles_n = (a.N + 31) / 32;
    const size_t lds = (size_t)2 * (a.tiles_m + a.tiles_n) * 32 * 128;
    if (plan->d.dtype == FI_BF16)
      hipLaunchKernelGGL((fi::gemm_fi_trial_kernel<FI_BF16>), dim3(n_trials), dim3(1024), lds, s, a);
    else
      hipLaunchKernelGGL((fi::gemm_fi_trial_kernel<FI_FP16>), dim3(n_trials), dim3(1024), lds, s, a);
    FI_HIP(hipGetLastError());
    return FI_OK;
  }
  const bool small = use_small(plan, n_trials, d_c_out != nullptr, d_h_out != nullptr);
  const bool one_step = !small && plan->mcfg >= 0 && n_trials <= 1024u;   // the partition kernel clears the records
  if (!one_step && !(small && may_clear && clear_in_kernel(plan, n_trials, s, &a))) {
    const size_t words = (size_t)n_trials * (sizeof(fi_trial_result) / 4);
    hipLaunchKernelGGL(fi::fill_u32_kernel, dim3((unsigned)((words + 255) / 256 > 1024 ? 1024 : (words + 255) / 256)),
                       dim3(256), 0, s, reinterpret_cast<uint32_t*>(d_results), words, 0u);
    FI_HIP(hipGetLastError());
  }
  if (small) {
    a.tiles_m = (a.M + 31) / 32;
    a.tiles_n = (a.N + 31) / 32;
    if (plan->d.dtype == FI_BF16) launch_small<FI_BF16>(a, s); else launch_small<FI_FP16>(a, s);
    FI_HIP(hipGetLastError());
    return FI_OK;
  }
  if (plan->mcfg < 0) {
    FI_HIP(launch_gemm(fi::MODE_CAMPAIGN, (int)plan->d.dtype, plan->cfg, a, (int)blocks, s));
    return FI_OK;
  }
  // R trials at a time share staged operands.  The batch is split on the device into the trials
  // whose fault leaves the operands alone and the operand-fault trials; each part has its own
  // instantiation of the kernel.
#define FI_PARTITION(DT, STEPS)                                                                                           \
  hipLaunchKernelGGL((fi::partition_trials_kernel<DT, STEPS>), dim3(1), dim3(1024), 0, s, d_faults, n_trials, plan->d.M,  \
                     plan->d.N, plan->d.K, plan->d.k_block, a.A, a.B, a.lda, a.ldb, plan->product_check, (uint32_t)mc.bm, \
                     (uint32_t)mc.bn, plan->kshift, ts.counts, ts.desc, ts.queue, 2u * fi::kQueueWords, d_results)
  if (plan->d.dtype == FI_BF16) {
    if (one_step) FI_PARTITION(FI_BF16, 1); else FI_PARTITION(FI_BF16, fi::kPartitionSteps);
  } else {
    if (one_step) FI_PARTITION(FI_FP16, 1); else FI_PARTITION(FI_FP16, fi::kPartitionSteps);
  }
#undef FI_PARTITION
  FI_HIP(hipGetLastError());
  m.part_counts = ts.counts;
  m.desc = ts.desc;
  if (m.K >= 128) m.queue = ts.queue;
  m.operands_apart = apart;
  FI_HIP(launch_multi((int)plan->d.dtype, four ? fi::kMultiFourInst : plan->mcfg, m, (int)mblocks, s));
  if (!apart) return FI_OK;
  if (m.queue) m.queue += fi::kQueueWords;
  if (m.clocks) m.clocks += 4;
  const int fours = plan->n_cus / 8 * 8 * fi::kMultiFour.wgs;
  FI_HIP(launch_multi((int)plan->d.dtype, fi::kMultiFourInst, m, fours, s));
  return FI_OK;
}

// ---- scratch of fi_gemm_inject_batch_noalloc: one array per GPU, held until the process ends.
constexpr uint32_t kNoAllocMaxTrials = 16384;
constexpr size_t kNoAllocWords = scratch_words(kNoAllocMaxTrials);
static __device__ __align__(256) uint32_t scratch[kNoAllocWords];

// The array's address on each device (the name above is only a host-side handle for the
// symbol: every use from host code goes through the looked-up pointer).
std::mutex g_scratch_mu;
uint32_t* g_scratch_ptr[kMaxDevices] = {};

// Looks the address up once per device, with that device current.  Called from
// fi_plan_create (set-up), so that the entry point itself only reads the table.
fi_status resolve_static_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return fail(FI_UNSUPPORTED, "device index %d beyond %d", device, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return FI_OK;
  uint32_t* ptr = nullptr;
  FI_HIP(hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(scratch)));
  if (!ptr) return fail(FI_DEVICE, "hipGetSymbolAddress returned a NULL address for the static scratch");
  g_scratch_ptr[device] = ptr;
  return FI_OK;
}

uint64_t splitmix64(uint64_t* state) {
  uint64_t z = (*state += 0x9E3779B97F4A7C15ull);
  z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull;
  z ^= z >> 27; z *= 0x94D049BB133111EBull;
  z ^= z >> 31;
  return z;
}

inline uint32_t scale_to(uint32_t n, uint64_t u) { return (uint32_t)(((u >> 32) * (uint64_t)n) >> 32); }

}  // namespace

extern "C" {

const char* fi_last_error(void) { return g_err; }

#ifndef FI_SOURCES_SHA256
#define FI_SOURCES_SHA256 "unknown"
#endif
const char* fi_build_info(void) { return FI_SOURCES_SHA256; }

fi_status fi_plan_create(const fi_plan_desc* desc, const void* d_A, const void* d_B, void* stream,
                         fi_plan** out) {
  float gamma = 0.f;
  fi_status st = check_desc(desc, &gamma);
  if (st != FI_OK) return st;
  if (!d_A || !d_B || !out) return fail(FI_INVALID_ARG, "d_A, d_B and out must be non-NULL");
  const fi_plan_desc& d = *desc;
  const int64_t min_ldb = d.b_layout == 0 ? (int64_t)d.K : (int64_t)d.N;
  if (d.lda < (int64_t)d.K || d.ldb < min_ldb)
    return fail(FI_INVALID_ARG, "leading dimension smaller than the row length");
  if ((reinterpret_cast<uintptr_t>(d_A) & 15u) || (d.lda & 7))
    return fail(FI_UNSUPPORTED, "A must be 16-byte aligned with lda a multiple of 8");
  if (d.b_layout == 0 && ((reinterpret_cast<uintptr_t>(d_B) & 15u) || (d.ldb & 7)))
    return fail(FI_UNSUPPORTED, "B must be 16-byte aligned with ldb a multiple of 8");
  if ((uint64_t)d.M * (uint64_t)d.lda >= (1ull << 31) ||
      (uint64_t)d.N * (uint64_t)(d.b_layout == 0 ? d.ldb : (int64_t)d.K) >= (1ull << 31))
    return fail(FI_UNSUPPORTED, "an operand spans 2^31 elements or more");
  if ((uint64_t)d.M * (uint64_t)d.N >= (1ull << 40)) return fail(FI_UNSUPPORTED, "M*N too large");
  st = check_device();
  if (st != FI_OK) return st;

  fi_plan* p = new (std::nothrow) fi_plan();
  if (!p) return fail(FI_OOM, "host allocation failed");
  p->d = d;
  p->d.gamma = gamma;
  p->cfg = pick_cfg(d);
  p->cfg_affected = d.N <= 64 ? 2 : 1;
  p->mcfg = pick_multi(d);
  // Next-layer launches: on problems below 2^35 multiply-adds the 128 x 128 shape with two workgroups
  // per CU (one's epilogue runs under the other's MFMAs) but for the batches that pick_prop sends to the
  // 256 x 256 shape, above it that one always (less LDS traffic per flop).
  p->prop_cfg = (double)d.M * (double)d.N * (double)d.K >= 34359738368.0 ? fi::kMultiOneTrial[0]
                                                                         : fi::kMultiOneTrial[1];
  p->group = 32;
  (void)hipGetDevice(&p->device);
  if (hipDeviceGetAttribute(&p->n_cus, hipDeviceAttributeMultiprocessorCount, p->device) != hipSuccess ||
      p->n_cus < 8)
    p->n_cus = 8;
  st = build_plan(p, d_A, d_B, as_stream(stream));
  if (st != FI_OK) {
    free_plan_buffers(p, hipStreamSynchronize(as_stream(stream)) == hipSuccess);
    delete p;
    return st;
  }
  st = resolve_static_scratch(p->device);
  if (st != FI_OK) {
    free_plan_buffers(p, true);                           // its creation has read back from the stream
    delete p;
    return st;
  }
  {
    std::lock_guard<std::mutex> lock(g_live_mu);
    g_live.insert(p);
  }
  *out = p;
  return FI_OK;
}

fi_status fi_plan_destroy(fi_plan* plan) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  {
    std::lock_guard<std::mutex> lock(g_live_mu);
    g_live.erase(plan);
  }
  // work that still reads the plan's buffers, on the plan's device, which need not be the current one
  int current = plan->device;
  bool there = hipGetDevice(&current) == hipSuccess;
  const bool other = there && current != plan->device;
  if (other) there = hipSetDevice(plan->device) == hipSuccess;
  const bool waited = hipDeviceSynchronize() == hipSuccess;
  free_plan_buffers(plan, there && waited);
  if (other) (void)hipSetDevice(current);
  delete plan;
  return FI_OK;
}

fi_status fi_release_memory(void) {
  hipError_t failed = hipSuccess;
  {
    std::lock_guard<std::mutex> lock(g_pool_mu);
    for (std::vector<PoolBlock>& blocks : g_pool) {
      const hipError_t e = pool_release(blocks, 0, 0);
      if (e != hipSuccess) failed = e;
    }
  }
  const hipError_t e = host_slots_release();
  if (e != hipSuccess) failed = e;
  FI_HIP(failed);
  return FI_OK;
}

fi_status fi_plan_buffer(const fi_plan* plan, uint32_t which, const void** d_ptr) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (!d_ptr) return fail(FI_INVALID_ARG, "d_ptr is NULL");
  switch (which) {
    case 0: *d_ptr = plan->c_star; break;
    case 1: *d_ptr = plan->s_abs; break;
    case 2: *d_ptr = plan->kra; break;
    case 3: *d_ptr = plan->cb; break;
    default: return fail(FI_INVALID_ARG, "which must be 0..3");
  }
  return FI_OK;
}

fi_status fi_plan_tune(fi_plan* plan, int32_t tile_config, int32_t trial_group, void* stream) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (tile_config >= kNumCfg + kNumMulti)
    return fail(FI_INVALID_ARG, "tile_config must be < %d", kNumCfg + kNumMulti);
  if (trial_group == 0 || trial_group > 4096) return fail(FI_INVALID_ARG, "trial_group must be in 1..4096");
  if (trial_group > 0) plan->group = trial_group;
  // C* does not depend on the tile shape: every shape feeds each output element the same
  // sequence of 16-wide MFMA steps in ascending k.
  if (tile_config >= 0) plan->auto_cfg = false;
  if (tile_config >= kNumCfg) {
    plan->mcfg = tile_config - kNumCfg;
    if (kMulti[plan->mcfg].r == 1) plan->prop_cfg = plan->mcfg;
  } else if (tile_config >= 0) {
    plan->cfg = tile_config; plan->cfg_affected = tile_config;
    // One trial per work item.  The 256x256 and 128x128 shapes run as persistent workgroups (the
    // multi-trial kernel's item loop with one trial per item).
    const bool persistent = tile_config < 2;
    plan->mcfg = persistent ? fi::kMultiOneTrial[tile_config] : -1;
    plan->prop_cfg = persistent ? fi::kMultiOneTrial[tile_config] : -1;
  }
  (void)stream;
  return FI_OK;
}

fi_status fi_plan_reserve(fi_plan* plan, uint32_t max_trials, void* stream) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (max_trials == 0) return fail(FI_INVALID_ARG, "max_trials is 0");
  BatchScratch* bs = nullptr;
  return batch_scratch(plan, as_stream(stream), max_trials, &bs, true);
}

fi_status fi_plan_set_clock_sink(fi_plan* plan, uint64_t* d_clocks) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (reinterpret_cast<uintptr_t>(d_clocks) & 7u) return fail(FI_INVALID_ARG, "d_clocks must be 8-byte aligned");
  plan->clocks = reinterpret_cast<unsigned long long*>(d_clocks);
  return FI_OK;
}

fi_status fi_probe_mfma_loop(uint32_t dtype, uint32_t random_data, uint32_t iters, uint32_t n_workgroups,
                             float* d_sink, uint64_t* d_clocks, void* stream) {
  if (dtype != FI_FP16 && dtype != FI_BF16) return fail(FI_UNSUPPORTED, "dtype %u: only FP16 (0) and BF16 (1)", dtype);
  if (!d_sink) return fail(FI_INVALID_ARG, "d_sink is NULL");
  if (iters == 0 || n_workgroups == 0 || n_workgroups > 65536u || iters > (1u << 24))
    return fail(FI_INVALID_ARG, "iters must be in 1..2^24 and n_workgroups in 1..65536");
  fi_status st = check_device();
  if (st != FI_OK) return st;
  unsigned long long* clk = reinterpret_cast<unsigned long long*>(d_clocks);
  if (dtype == FI_BF16)
    hipLaunchKernelGGL(fi::mfma_loop_probe_kernel<FI_BF16>, dim3(n_workgroups), dim3(512), 0, as_stream(stream),
                       (int)random_data, (int)iters, d_sink, clk);
  else
    hipLaunchKernelGGL(fi::mfma_loop_probe_kernel<FI_FP16>, dim3(n_workgroups), dim3(512), 0, as_stream(stream),
                       (int)random_data, (int)iters, d_sink, clk);
  FI_HIP(hipGetLastError());
  return FI_OK;
}

fi_status fi_plan_set_product_check(fi_plan* plan, uint32_t mode) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (mode > FI_PCHECK_RANGE_FLIP) return fail(FI_INVALID_ARG, "unknown product check %u", mode);
  plan->product_check = (int)mode;
  return FI_OK;
}

fi_status fi_plan_describe(const fi_plan* plan, char* h_buf, uint64_t n) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (!h_buf || n == 0) return fail(FI_INVALID_ARG, "h_buf is NULL or n is 0");
  const TileCfg c = kCfg[plan->cfg];
  const char* dt = plan->d.dtype == FI_BF16 ? "bf16" : "fp16";
  char small[256] = "";
  if (use_small(plan, 1, false, false)) {
    const double each = small_steps(plan, 1), long_each = each + kSmallLongTile * small_tiles(plan, 4) / 4.0;
    const unsigned most = (unsigned)(plan->d.K > 64 && kSmallLong / long_each > kSmallSteps / each ? kSmallLong / long_each : kSmallSteps / each), cus = (unsigned)plan->n_cus;
    char trial[128] = "";
    if (use_trial(plan, 1, false, false))
      snprintf(trial, sizeof(trial), ", without outputs and at most %u trials: gemm_fi_trial_kernel<%s, one workgroup per trial>",
               most < cus ? most : cus, dt);
    snprintf(small, sizeof(small), "; small batches, at most %u trials: gemm_fi_small_kernel<%s, one trial per wave, 32x32>%s",
             most, dt, trial);
  }
  if (plan->mcfg >= 0) {
    const MultiCfg m = kMulti[plan->mcfg];
    if (m.r == 1)
      snprintf(h_buf, n, "gemm_fi_multi_kernel<%s, one trial per item, %dx%d, %d threads, persistent x%d per CU>%s", dt,
               m.bm, m.bn, m.wm * m.wn * 64, m.wgs, small);
    else {
      char four[224] = "";
      if (use_four(plan, 1, true)) {
        const uint64_t tiles = (uint64_t)((plan->d.M + m.bm - 1) / m.bm) * ((plan->d.N + m.bn - 1) / m.bn), round = (uint64_t)m.wgs * (uint64_t)plan->n_cus;
        const uint64_t with = kFourWork * round / (tiles * ((plan->d.K + 63) / 64)), without = kFourRounds * round / tiles;
        const MultiCfg f = fi::kMultiFour;
        snprintf(four, sizeof(four), "; at most %llu trials, operand faults and batches with outputs %llu: gemm_fi_four_kernel<R=%d, x%d per CU>",
                 (unsigned long long)((without < with ? without : with) * (uint64_t)m.r), (unsigned long long)(with * (uint64_t)m.r), f.r, f.wgs);
      }
      snprintf(h_buf, n, "gemm_fi_multi_kernel<%s, R=%d, %dx%d, %d threads, persistent x%d per CU> (a second, "
               "operand-patching instantiation for operand faults)%s%s", dt, m.r, m.bm, m.bn, m.wm * m.wn * 64, m.wgs, four, small);
    }
  } else {
    snprintf(h_buf, n, "gemm_fi_kernel<%s, %dx%d, %d threads>", dt, c.bm, c.bn, c.wm * c.wn * 64);
  }
  return FI_OK;
}

fi_status fi_gemm_inject_batch(fi_plan* plan, const fi_fault* d_faults, uint32_t n_trials, uint32_t policy,
                               fi_trial_result* d_results, float* d_c_out, void* stream) {
  fi_status st = check_batch_args(plan, d_faults, n_trials, policy, d_results);
  if (st != FI_OK) return st;
  TrialScratch ts;
  if (plan->mcfg >= 0) {
    BatchScratch* bs = nullptr;
    st = batch_scratch(plan, as_stream(stream), n_trials, &bs);
    if (st != FI_OK) return st;
    ts = TrialScratch(bs->words);
  }
  return inject_batch(plan, d_faults, n_trials, policy, d_results, d_c_out, as_stream(stream), ts, true);
}

fi_status fi_gemm_inject_batch_act(fi_plan* plan, const fi_fault* d_faults, uint32_t n_trials, uint32_t policy,
                                   fi_trial_result* d_results, void* d_h_out, void* stream) {
  fi_status st = check_batch_args(plan, d_faults, n_trials, policy, d_results);
  if (st != FI_OK) return st;
  if (!d_h_out) return fail(FI_INVALID_ARG, "d_h_out is NULL");
  if (reinterpret_cast<uintptr_t>(d_h_out) & 1u) return fail(FI_UNSUPPORTED, "d_h_out must be 2-byte aligned");
  if (plan->mcfg < 0)
    return fail(FI_UNSUPPORTED, "the fused hand-over is not available with tile_config 2; use fi_gemm_inject_batch "
                "with d_c_out and fi_activation_round");
  BatchScratch* bs = nullptr;
  st = batch_scratch(plan, as_stream(stream), n_trials, &bs);
  if (st != FI_OK) return st;
  const TrialScratch ts(bs->words);
  return inject_batch(plan, d_faults, n_trials, policy, d_results, nullptr, as_stream(stream), ts, true,
                      static_cast<uint16_t*>(d_h_out));
}

fi_status fi_gemm_inject_batch_noalloc(fi_plan* plan, const fi_fault* d_faults, uint32_t n_trials, uint32_t policy,
                                       fi_trial_result* d_results, float* d_c_out, void* stream) {
  fi_status st = check_batch_args(plan, d_faults, n_trials, policy, d_results);
  if (st != FI_OK) return st;
  if (n_trials > kNoAllocMaxTrials)
    return fail(FI_UNSUPPORTED, "n_trials %u exceeds the %u trials the static scratch holds; split the batch or use "
                "fi_gemm_inject_batch", n_trials, kNoAllocMaxTrials);
  uint32_t* base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    base = g_scratch_ptr[plan->device];
  }
  if (!base) return fail(FI_STATE, "the static scratch of device %d was not resolved at plan creation", plan->device);
  const TrialScratch ts(base);
  return inject_batch(plan, d_faults, n_trials, policy, d_results, d_c_out, as_stream(stream), ts, false);
}

fi_status fi_gemm_inject_batch_affected(fi_plan* plan, const fi_fault* d_faults, uint32_t n_trials,
                                        uint32_t policy, fi_trial_result* d_results, void* stream) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (!d_faults || !d_results) return fail(FI_INVALID_ARG, "d_faults and d_results must be non-NULL");
  if (n_trials == 0) return fail(FI_INVALID_ARG, "n_trials is 0");
  if (policy > FI_CORRECT_RECOMPUTE) return fail(FI_INVALID_ARG, "unknown correction policy %u", policy);
  if (plan->n_clean_flagged != 0)
    return fail(FI_UNSUPPORTED, "the plan's detector flags %u element(s) of the fault-free result itself, which the "
                "affected-only campaign would not count; use fi_gemm_inject_batch", plan->n_clean_flagged);
  // The largest batch is what it was when an operand fault took a workgroup per tile of its row or column:
  // callers split their batches by it.  The kernels here take more.
  GemmArgs a = base_args(plan, plan->cfg_affected);
  const uint64_t slots = (uint64_t)(a.tiles_m > a.tiles_n ? a.tiles_m : a.tiles_n);
  if (slots * n_trials >= (1ull << 31))
    return fail(FI_UNSUPPORTED, "%llu (a row or column in output tiles) x %u trials exceeds 2^31; split the batch",
                (unsigned long long)slots, n_trials);
  hipStream_t s = as_stream(stream);
  a.n_trials = (int)n_trials;
  a.faults = d_faults;
  a.results = d_results;
  a.policy = (int)policy;
  a.product_check = plan->product_check;
  const RowsGrid rows = rows_grid(plan->d, n_trials);
  // Not under capture: a graph may be replayed beside calls on this stream, and outlive the buffer.
  uint32_t* parts = nullptr;
  for (const BatchScratch& b : plan->batch) {
    if (rows.x_slots < kPartSlots || shared_handle(s) || b.stream != s || b.parts_cap < (size_t)rows.x_slots * n_trials * fi::kPartWords) continue;
    if (!capturing(s)) parts = b.parts;
  }
  if (plan->d.dtype == FI_BF16) return launch_affected<FI_BF16>(a, rows, plan->n_cus, plan->plain_ok, parts, s);
  return launch_affected<FI_FP16>(a, rows, plan->n_cus, plan->plain_ok, parts, s);
}

fi_status fi_activation_round(uint32_t dtype, const float* d_c, uint64_t n, uint16_t* d_h, void* stream) {
  if (dtype != FI_FP16 && dtype != FI_BF16)
    return fail(FI_UNSUPPORTED, "dtype %u: only FP16 (0) and BF16 (1)", dtype);
  if (!d_c || !d_h) return fail(FI_INVALID_ARG, "d_c and d_h must be non-NULL");
  if (n == 0) return fail(FI_INVALID_ARG, "n is 0");
  if ((reinterpret_cast<uintptr_t>(d_c) & 15u) || (reinterpret_cast<uintptr_t>(d_h) & 15u))
    return fail(FI_UNSUPPORTED, "d_c and d_h must be 16-byte aligned");
  uint64_t blocks = (n / 8 + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  if (blocks == 0) blocks = 1;
  if (dtype == FI_BF16)
    hipLaunchKernelGGL(fi::activation_round_kernel<FI_BF16>, dim3((unsigned)blocks), dim3(256), 0, as_stream(stream),
                       d_c, (size_t)n, d_h);
  else
    hipLaunchKernelGGL(fi::activation_round_kernel<FI_FP16>, dim3((unsigned)blocks), dim3(256), 0, as_stream(stream),
                       d_c, (size_t)n, d_h);
  FI_HIP(hipGetLastError());
  return FI_OK;
}

fi_status fi_gemm_propagate_batch(fi_plan* plan, const void* d_a_stack, uint64_t trial_stride, uint32_t n_trials,
                                  uint32_t policy, fi_trial_result* d_results, float* d_c_out, void* stream) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (!d_a_stack || !d_results) return fail(FI_INVALID_ARG, "d_a_stack and d_results must be non-NULL");
  if (n_trials == 0) return fail(FI_INVALID_ARG, "n_trials is 0");
  if (policy > FI_CORRECT_RECOMPUTE) return fail(FI_INVALID_ARG, "unknown correction policy %u", policy);
  if ((reinterpret_cast<uintptr_t>(d_a_stack) & 15u) || (trial_stride & 7u))
    return fail(FI_UNSUPPORTED, "d_a_stack must be 16-byte aligned with trial_stride a multiple of 8");
  if (trial_stride != 0 && trial_stride < ((uint64_t)plan->d.M - 1) * (uint64_t)plan->d.lda + plan->d.K)
    return fail(FI_INVALID_ARG, "trial_stride %llu is smaller than one operand ((M-1)*lda + K elements)",
                (unsigned long long)trial_stride);
  GemmArgs a = base_args(plan);
  // C* is addressed with 32 bits; the trials' operands are the caller's, so K must hold whole k-tiles
  bool persistent = plan->prop_cfg >= 0 && a.c_star_bytes != 0 && plan->kshift == 0;
  const bool small = use_small_propagate(plan, n_trials, d_c_out != nullptr, persistent);
  persistent = persistent && !small;
  auto tile = [&](int prop_cfg) {
    const MultiCfg mc = kMulti[prop_cfg];
    a.tiles_m = (a.M + mc.bm - 1) / mc.bm;
    a.tiles_n = (a.N + mc.bn - 1) / mc.bn;
    return (uint64_t)a.tiles_m * a.tiles_n * n_trials;
  };
  // The largest batch is that of the plan's own tile shape, whichever shape serves this one.
  uint64_t blocks = persistent ? tile(plan->prop_cfg) : (uint64_t)a.tiles_m * a.tiles_n * n_trials;
  if (blocks >= (1ull << 31)) return fail(FI_UNSUPPORTED, "tiles x trials exceeds 2^31 workgroups; split the batch");
  const int prop_cfg = pick_prop(plan, n_trials);
  if (persistent) blocks = tile(prop_cfg);
  hipStream_t s = as_stream(stream);
  if (!(small && clear_in_kernel(plan, n_trials, s, &a))) {
    const size_t words = (size_t)n_trials * (sizeof(fi_trial_result) / 4);
    hipLaunchKernelGGL(fi::fill_u32_kernel, dim3((unsigned)((words + 255) / 256 > 1024 ? 1024 : (words + 255) / 256)),
                       dim3(256), 0, s, reinterpret_cast<uint32_t*>(d_results), words, 0u);
    FI_HIP(hipGetLastError());
  }
  a.A = static_cast<const uint16_t*>(d_a_stack);
  a.a_trial_stride = trial_stride;
  a.n_trials = (int)n_trials;
  // Trials share B but not A: a trial's tiles follow each other in the work list, so the column
  // tiles of one A panel run at the same time on one XCD and the panel comes from HBM once
  // (measured on 512 x 768 x 3072, 256 trials: 0.72 ms against 0.83 ms with three trials per tile).
  a.group = 1;
  a.results = d_results;
  a.c_out = d_c_out;
  a.policy = (int)policy;
  if (small) {
    a.tiles_m = (a.M + 31) / 32;
    a.tiles_n = (a.N + 31) / 32;
    const dim3 grid((unsigned)a.tiles_m * (((unsigned)a.tiles_n + 3) / 4) * n_trials);
    if (plan->d.dtype == FI_BF16)
      hipLaunchKernelGGL((fi::gemm_fi_small_kernel<FI_BF16, 1, fi::SMALL_PROPAGATE>), grid, dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL((fi::gemm_fi_small_kernel<FI_FP16, 1, fi::SMALL_PROPAGATE>), grid, dim3(256), 0, s, a);
    FI_HIP(hipGetLastError());
    return FI_OK;
  }
  if (persistent) {
    // persistent workgroups walking (tile, trial) items
    static_assert(offsetof(fi_trial_result, site_word_after) == offsetof(fi_trial_result, site_word_before) + 4,
                  "the word behind the first counter counts the workgroups that are done");
    if (n_trials >= (uint32_t)fi::kQueueXcds && plan->d.K >= 128) a.queue = &d_results->site_word_before;
    const MultiCfg mc = kMulti[prop_cfg];
    const uint64_t cus = (uint64_t)(plan->n_cus / 8 * 8) * (uint64_t)mc.wgs;
    FI_HIP(launch_prop((int)plan->d.dtype, prop_cfg, a, (int)(blocks < cus ? blocks : cus), s));
    return FI_OK;
  }
  FI_HIP(launch_gemm(fi::MODE_PROPAGATE, (int)plan->d.dtype, plan->cfg, a, (int)blocks, s));
  return FI_OK;
}

fi_status fi_detect_correct(fi_plan* plan, float* d_c, uint32_t batch, uint32_t policy, uint8_t* d_flags,
                            uint32_t* d_n_flagged, void* stream) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (!d_c) return fail(FI_INVALID_ARG, "d_c is NULL");
  if (batch == 0 || batch > 65535u) return fail(FI_INVALID_ARG, "batch must be in 1..65535");
  if (policy > FI_CORRECT_RECOMPUTE) return fail(FI_INVALID_ARG, "unknown correction policy %u", policy);
  hipStream_t s = as_stream(stream);
  const fi_plan_desc& d = plan->d;
  GemmArgs a = {};
  if (d_n_flagged && !clear_in_kernel(plan, batch, s, &a)) {
    hipLaunchKernelGGL(fi::fill_u32_kernel, dim3((batch + 255) / 256), dim3(256), 0, s, d_n_flagged,
                       (size_t)batch, 0u);
    FI_HIP(hipGetLastError());
  }
  FI_HIP(launch_detect(plan, d_c, batch, policy, d_flags, d_n_flagged, a.clear_word, a.epoch, s));
  return FI_OK;
}

fi_status fi_classify(fi_plan* plan, const fi_trial_result* d_results, uint32_t n_trials, uint8_t* d_class,
                      uint64_t* d_counts, void* stream) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (!d_results || !d_counts) return fail(FI_INVALID_ARG, "d_results and d_counts must be non-NULL");
  if (n_trials == 0) return fail(FI_INVALID_ARG, "n_trials is 0");
  hipLaunchKernelGGL(fi::classify_kernel, dim3(1), dim3(1024), 0, as_stream(stream), d_results, n_trials,
                     d_class, d_counts);
  FI_HIP(hipGetLastError());
  return FI_OK;
}

fi_status fi_deviation_histogram(fi_plan* plan, const fi_fault* d_faults, const fi_trial_result* d_results,
                                 uint32_t n_trials, uint32_t which, uint64_t* d_hist, void* stream) {
  fi_status st = check_plan(plan);
  if (st != FI_OK) return st;
  if (!d_faults || !d_results || !d_hist) return fail(FI_INVALID_ARG, "d_faults, d_results and d_hist must be non-NULL");
  if (n_trials == 0) return fail(FI_INVALID_ARG, "n_trials is 0");
  if (which > FI_HIST_DEV_POST) return fail(FI_INVALID_ARG, "unknown histogram quantity %u", which);
  hipLaunchKernelGGL(fi::deviation_histogram_kernel, dim3(1), dim3(1024), 0, as_stream(stream), d_faults, d_results,
                     n_trials, (int)which, reinterpret_cast<unsigned long long*>(d_hist));
  FI_HIP(hipGetLastError());
  return FI_OK;
}

fi_status fi_sample_faults(uint64_t seed, uint32_t first_trial, uint32_t n_trials, const fi_plan_desc* desc,
                           uint32_t kind_mode, uint32_t nbits, fi_fault* h_out) {
  fi_status st = check_desc(desc, nullptr);
  if (st != FI_OK) return st;
  if (!h_out) return fail(FI_INVALID_ARG, "h_out is NULL");
  if (kind_mode > FI_KIND_ALL_PRODUCT) return fail(FI_INVALID_ARG, "unknown kind_mode %u", kind_mode);
  if (nbits < 1 || nbits > 16) return fail(FI_INVALID_ARG, "nbits must be in 1..16");
  const uint32_t nblocks = desc->K / desc->k_block;
  for (uint32_t n = 0; n < n_trials; ++n) {
    const uint64_t t = (uint64_t)first_trial + n;
    uint64_t state = seed + (t << 32);
    uint64_t u[4];
    for (int q = 0; q < 4; ++q) u[q] = splitmix64(&state);
    fi_fault f;
    uint32_t kind = kind_mode == FI_KIND_ALL_ACC ? FI_SITE_ACC
                  : kind_mode == FI_KIND_ALL_A   ? FI_SITE_A
                  : kind_mode == FI_KIND_ALL_B   ? FI_SITE_B
                  : kind_mode == FI_KIND_ALL_PRODUCT ? FI_SITE_PRODUCT
                  : ((t & 1) ? FI_SITE_A : FI_SITE_ACC);
    f.kind = kind;
    uint32_t width = 16;
    if (kind == FI_SITE_ACC) {
      f.row = scale_to(desc->M, u[0]);
      f.col = scale_to(desc->N, u[1]);
      f.kblock = scale_to(nblocks, u[2]);
      width = 32;
    } else if (kind == FI_SITE_PRODUCT) {
      f.row = scale_to(desc->M, u[0]);
      f.col = scale_to(desc->N, u[1]);
      f.kblock = scale_to(desc->K, u[2]);          // the term: k, uniform over all MMA steps and terms
    } else {
      const uint32_t s = scale_to(nblocks, u[1]);
      const uint32_t k = s * desc->k_block + scale_to(desc->k_block, u[2]);
      f.kblock = s;
      if (kind == FI_SITE_A) { f.row = scale_to(desc->M, u[0]); f.col = k; }
      else                   { f.row = k; f.col = scale_to(desc->N, u[0]); }
    }
    const uint32_t pos = scale_to(width - nbits + 1, u[3]);
    f.xor_mask = (uint32_t)(((1ull << nbits) - 1ull) << pos);
    h_out[n] = f;
  }
  return FI_OK;
}

}  // extern "C"
