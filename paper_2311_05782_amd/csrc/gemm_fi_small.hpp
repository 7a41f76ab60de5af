// Fault-injecting GEMM for batches too small to fill the chip, gfx950: one wave per (trial, 32 x 32
// output tile).
//
// The multi-trial kernel's unit is eight trials of a 64 x 64 tile by four waves; a batch of a few
// dozen trials on a small problem gives it a handful of units, most of them padded, each behind a
// partition launch and a code path of tens of kilobytes that is cold on every launch.  Here four
// waves take TPW trials x 4 / TPW neighbouring tiles, share the staged operands, and read the fault
// from the list itself: no partition, no second launch for the operand faults, one trial per wave.
//
// Bound: launches and latency - a chain of K/64 k-tiles, each a load, a barrier and four MFMAs - so
// k-tiles are loaded NBUF - 1 ahead; on larger batches the LDS (two 1 KB fragments per MFMA, where
// eight trials per wave read a quarter of one).
//
// Measured, record fill included, multi-trial kernel -> this one: 24 trials on 300 x 203 x 176 22 -> 10 us
// (A faults 27 -> 10 us, with outputs 48 -> 12 us), 32 on 3136 x 64 x 576 27 -> 22 us, 16 on 64 x 64 x
// 4096 63 -> 32 us (40 us with the loads of a k-tile in loops, see issue_tile); without LDS, fragments
// straight from global memory, the last two took 72 and 62 us (a fragment's 32 rows are 32 cache lines).
//
// The per-element arithmetic is that of gemm_fi_kernel: the same sequence of 16-wide MFMA steps in
// ascending k, hence bit-identical results.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "clear_once.hpp"
#include "fi.h"
#include "gemm_fi.hpp"

namespace fi {

// A trial's fault (uniform in its wave): its coordinates, the 16-wide step that consumes the faulted
// operand word (its k is fk) or at whose end the accumulator changes, and a product-term fault's terms.
struct TrialFault {
  uint32_t kind, row, col, mask;
  int event, fk;
  bool valid;
  float re, re_err;
  bool fired;
  __device__ __forceinline__ bool operand() const { return kind == FI_SITE_A || kind == FI_SITE_B; }
  __device__ __forceinline__ bool isA() const { return kind == FI_SITE_A; }
  // the fault reaches an element of the 32 x 32 tile at (m0, n0)
  __device__ __forceinline__ bool reaches(int m0, int n0) const {
    const bool in_rows = (int)row >= m0 && (int)row < m0 + 32, in_cols = (int)col >= n0 && (int)col < n0 + 32;
    return kind == FI_SITE_NONE ? false : kind == FI_SITE_A ? in_rows : kind == FI_SITE_B ? in_cols : in_rows && in_cols;
  }
};

__device__ __forceinline__ TrialFault decode_fault(const GemmArgs& p, int trial) {
  const fi_fault f = p.faults[trial];
  TrialFault t;
  t.kind = f.kind; t.row = f.row; t.col = f.col; t.mask = f.xor_mask;
  t.valid = true; t.event = -1; t.fk = 0; t.re = t.re_err = 0.0f; t.fired = false;
  if (f.kind == FI_SITE_ACC) {
    t.valid = f.row < (uint32_t)p.M && f.col < (uint32_t)p.N && f.kblock < (uint32_t)(p.K / p.kb);
    t.event = (int)((f.kblock + 1) * (uint32_t)p.kb) / 16 - 1;
  } else if (f.kind == FI_SITE_PRODUCT) {
    t.valid = f.row < (uint32_t)p.M && f.col < (uint32_t)p.N && f.kblock < (uint32_t)p.K;
    t.fk = (int)f.kblock;
  } else if (f.kind == FI_SITE_A) {
    t.valid = f.row < (uint32_t)p.M && f.col < (uint32_t)p.K;
    t.fk = (int)f.col;
  } else if (f.kind == FI_SITE_B) {
    t.valid = f.row < (uint32_t)p.K && f.col < (uint32_t)p.N;
    t.fk = (int)f.row;
  } else {
    t.valid = f.kind == FI_SITE_NONE;
  }
  if (f.kind != FI_SITE_ACC) t.event = t.fk / 16;
  if (!t.valid) t.kind = FI_SITE_NONE;
  if (t.kind == FI_SITE_NONE) t.event = -1;
  return t;
}

// The terms of a product-term fault, by a wave that owns its element.
template <int DT>
__device__ __forceinline__ void fetch_product_terms(TrialFault& t, const GemmArgs& p) {
  product_fault_terms<DT>(p.A[(size_t)t.row * p.lda + t.fk], p.B[(size_t)t.col * p.ldb + t.fk], t.mask, p.product_check,
                          t.re, t.re_err, t.fired);
}

// One 16-wide step at whose operands or end the fault strikes, in a tile that it reaches.
template <int DT>
__device__ __forceinline__ f32x16 faulty_step(const TrialFault& t, u32x4 a, u32x4 b, f32x16 acc, int m0, int n0, int lane,
                                              uint32_t& before, uint32_t& after) {
  if (t.operand()) {
    // the lane that holds the word (row or column l % 32, k half l / 32), two words per register
    const int l = (int)((t.isA() ? t.row - (uint32_t)m0 : t.col - (uint32_t)n0) & 31u) + 32 * ((t.fk >> 3) & 1);
    const uint32_t x = lane == l ? (t.mask & 0xFFFFu) << (16 * (t.fk & 1)) : 0u;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t xr = r == ((t.fk & 7) >> 1) ? x : 0u;
      a[r] ^= t.isA() ? xr : 0u;
      b[r] ^= t.isA() ? 0u : xr;
    }
    return mfma_32x32x16<DT>(a, b, acc);
  }
  acc = mfma_32x32x16<DT>(a, b, acc);
  const int ri = (int)t.row - m0, rj = (int)t.col - n0;   // inside the tile
  const int sel_v = 4 * (ri >> 3) + (ri & 3), sel_lane = rj + 32 * ((ri >> 2) & 1);
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const uint32_t word = __float_as_uint(acc[v]);
    const uint32_t nw = t.kind == FI_SITE_PRODUCT ? __float_as_uint(write_back(acc[v], t.re, t.re_err)) : (word ^ t.mask);
    before = v == sel_v ? word : before;                  // meaningful in lane sel_lane
    after = v == sel_v ? nw : after;
    acc[v] = __uint_as_float((v == sel_v && lane == sel_lane) ? nw : word);
  }
  return acc;
}

// Counts of what a fault changed in one tile that it reaches: one element, one row (it lies in one
// register and half-wave) or one column (gathered into lanes 0 .. 31, row k to lane k).  Counters are
// uniform, maxima per lane.
struct TileDeviation {
  uint32_t n_bit, n_pre, n_post, n_bT, n_btau;
  float mx_pre, mx_post;
};
__device__ __forceinline__ TileDeviation tile_deviation(const TrialFault& t, const GemmArgs& p, const f32x16& acc,
                                                        const f32x16& T, int m0, int n0, int lane) {
  const int l32 = lane & 31, lhi = lane >> 5, col = n0 + l32;
  float c = acc[0], th = T[0];
  int row, cc_col;
  bool act;
  if (t.kind != FI_SITE_B) {
    const int ri = ((int)t.row - m0) & 31;
    const int sel_v = 4 * (ri >> 3) + (ri & 3), sel_hi = (ri >> 2) & 1;
#pragma unroll
    for (int v = 1; v < 16; ++v) {
      c = v == sel_v ? acc[v] : c;
      th = v == sel_v ? T[v] : th;
    }
    row = (int)t.row;
    cc_col = min(col, p.N - 1);
    act = lhi == sel_hi && col < p.N && (t.isA() || col == (int)t.col);
  } else {
    const int sel = (int)t.col - n0;
    int x = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int word = (int)__float_as_uint(acc[v]);
      const int k0 = 8 * (v >> 2) + (v & 3);
      // read with all lanes active, outside the selects
      const int lo = __builtin_amdgcn_readlane(word, sel), hi = __builtin_amdgcn_readlane(word, sel + 32);
      x = lane == k0 ? lo : x;
      x = lane == k0 + 4 ? hi : x;
    }
    c = __uint_as_float((uint32_t)x);
    act = lane < 32 && m0 + lane < p.M;
    row = min(m0 + l32, p.M - 1);
    cc_col = (int)t.col;
    th = p.bound_global ? p.t_global : __fmul_rn(__fmul_rn(p.kra[row], p.cb[t.col]), p.gamma);
  }
  const size_t idx = (size_t)row * (size_t)p.N + (size_t)cc_col;
  const float cs = p.c_star[idx], tau = p.s_abs[idx] * 0.000244140625f;   // 2^-12, exact scaling
  const bool flag = !(fabsf(c) <= th);
  float fixed = c;
  if (flag && p.policy == FI_CORRECT_ZERO) fixed = 0.0f;
  if (flag && p.policy == FI_CORRECT_RECOMPUTE) fixed = cs;
  const float dpre = finite_or_inf(fabsf(c - cs)), dpost = finite_or_inf(fabsf(fixed - cs));
  const float band = fmaxf(2.0f * tau, th * 0.015625f), mag = fabsf(c);
  const uint64_t am = __ballot(act), changed = __ballot(__float_as_uint(c) != __float_as_uint(cs)) & am;
  TileDeviation d;
  d.n_bit = (uint32_t)__builtin_popcountll(changed);
  d.n_pre = (uint32_t)__builtin_popcountll(__ballot(!(dpre <= tau)) & am);
  d.n_post = (uint32_t)__builtin_popcountll(__ballot(!(dpost <= tau)) & am);
  d.n_bT = (uint32_t)__builtin_popcountll(changed & __ballot(mag <= 3.4028234e38f) & __ballot(fabsf(mag - th) <= band));
  d.n_btau = (uint32_t)__builtin_popcountll(changed & __ballot(tau > 0.0f) & __ballot(dpre >= 0.5f * tau) &
                                            __ballot(dpre <= 2.0f * tau));
  d.mx_pre = act ? dpre : 0.0f;
  d.mx_post = act ? dpost : 0.0f;
  return d;
}

// Detector on a tile's elements (those outside the problem, copies of the last row or column, get
// T = +Inf and the value 0) and its outputs, corrected where flagged, in FP32 or in the operand
// format.  Returns the number of flagged elements (uniform).
template <int DT>
__device__ __forceinline__ uint32_t detect_tile(const GemmArgs& p, f32x16& acc, f32x16& T, const f32x4* kra4, float cbj,
                                                int trial, int m0, int n0, int lane) {
  const int row_base = m0 + 4 * (lane >> 5), col = n0 + (lane & 31);
  const bool ragged = m0 + 32 > p.M || n0 + 32 > p.N;
#pragma unroll
  for (int v = 0; v < 16; ++v)
    T[v] = p.bound_global ? p.t_global : __fmul_rn(__fmul_rn(kra4[v >> 2][v & 3], cbj), p.gamma);
  if (ragged) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const bool in = row_base + 8 * (v >> 2) + (v & 3) < p.M && col < p.N;
      T[v] = in ? T[v] : __builtin_inff();
      acc[v] = in ? acc[v] : 0.0f;
    }
  }
  uint64_t any = 0;
#pragma unroll
  for (int v = 0; v < 16; ++v) any |= __ballot(!(fabsf(acc[v]) <= T[v]));
  uint32_t n_flag = 0;
  if (any != 0) {
#pragma unroll
    for (int v = 0; v < 16; ++v) n_flag += (uint32_t)__builtin_popcountll(__ballot(!(fabsf(acc[v]) <= T[v])));
  }
  if (p.c_out || p.h_out) {
    f32x16 out = acc;
    if (any != 0 && p.policy != FI_CORRECT_NONE) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (!(fabsf(out[v]) <= T[v]))
          out[v] = p.policy == FI_CORRECT_ZERO ? 0.0f : p.c_star[(size_t)(row_base + 8 * (v >> 2) + (v & 3)) * p.N + col];
    }
    const size_t out0 = (size_t)trial * (size_t)p.M * (size_t)p.N + col;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = row_base + 8 * (v >> 2) + (v & 3);
      if (!ragged || (row < p.M && col < p.N)) {
        if (p.c_out) __builtin_nontemporal_store(out[v], p.c_out + out0 + (size_t)row * p.N);
        if (p.h_out) __builtin_nontemporal_store((uint16_t)relu_round16<DT>(out[v]), p.h_out + out0 + (size_t)row * p.N);
      }
    }
  }
  return n_flag;
}

// CAMPAIGN: trials with faults.  SUMS: the plan's fault-free pass; C* to p.c_out and the magnitude
// sums, from the same fragments with the sign bits cleared, to p.s_out.  PROPAGATE: the next layer;
// trial t multiplies its own A operand, nothing is injected, every element is compared with C*.
// p.tiles_m and p.tiles_n count 32 x 32 tiles.
enum { SMALL_CAMPAIGN = 0, SMALL_SUMS = 1, SMALL_PROPAGATE = 2 };
template <int DT, int TPW, int MODE>
__global__ void __launch_bounds__(256) gemm_fi_small_kernel(const GemmArgs p) {
  constexpr bool SUMS = MODE == SMALL_SUMS, PROP = MODE == SMALL_PROPAGATE;
  static_assert(TPW == 1 || MODE == SMALL_CAMPAIGN, "only campaign trials share operands");
  static_assert(TPW == 1 || TPW == 2 || TPW == 4, "four waves: trials x tiles");
  constexpr int TILES = 4 / TPW;                          // neighbouring 32-column tiles
  constexpr int NBUF = TPW == 1 ? 3 : 4;                  // 60, 48 or 32 KB of LDS
  constexpr int BK = 64, ROWS = 32 + 32 * TILES, STAGE = ROWS * 128;
  constexpr int GROUPS = ROWS / 8, G_W = (GROUPS + 3) / 4;   // 8-row groups; loads per wave and k-tile
  __shared__ __attribute__((aligned(16))) uint8_t smem[NBUF * STAGE];
  typedef __attribute__((address_space(3))) void lds_void;
  const int lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t n_trials = SUMS ? 1u : (uint32_t)p.n_trials;
  const uint32_t n_groups = (n_trials + TPW - 1) / TPW;   // trials that share a workgroup
  const uint32_t wide = (uint32_t)(p.tiles_n + TILES - 1) / TILES;
  const uint32_t strip = blockIdx.x / n_groups;           // 32 rows x 32 * TILES columns
  const int m0 = (int)(strip / wide) * 32, strip_n0 = (int)(strip % wide) * (32 * TILES);
  // Waves of a padded trial or tile stage and keep the barriers, nothing else.
  const int trial = (int)min(blockIdx.x % n_groups * TPW + (uint32_t)(wave % TPW), n_trials - 1u);
  const int n0 = strip_n0 + wave / TPW * 32;
  const bool works = blockIdx.x % n_groups * TPW + (uint32_t)(wave % TPW) < n_trials && n0 < p.N;
  auto clock = [&](int at) __attribute__((always_inline)) {   // see GemmArgs::clocks
    if (!SUMS && p.clocks && blockIdx.x == 0 && threadIdx.x == 0) {
      at += PROP ? 8 : 0;
      p.clocks[at] = __builtin_readcyclecounter();
      p.clocks[at + 1] = __builtin_amdgcn_s_memrealtime();
    }
  };
  clock(0);

  // ---- records: cleared here where no launch in front has done it (for a few hundred trials a launch is the larger
  // part of the time: 24 product-term trials on 300 x 203 x 176, with classes and histogram, 16.3 -> 14.0 us), see
  // clear_once.hpp.  A wave that owns a fault looks at the word now and needs it behind its k-loop, the others (thousands,
  // and one word) only when they have something to write.
  [[maybe_unused]] uint32_t seen = 0;                     // not looked at
  const bool clearing = !SUMS && p.clear_word != nullptr;    // uniform in the launch
  uint32_t* const records = reinterpret_cast<uint32_t*>(p.results);
  const uint32_t record_words = n_trials * (uint32_t)(sizeof(fi_trial_result) / 4);
  if (clearing && blockIdx.x == 0) {
    uint32_t* const taken = reinterpret_cast<uint32_t*>(smem);   // nothing is staged yet
    if (wave == 0) {
      const bool mine = take_clearing(p.clear_word, p.epoch, lane);
      if (lane == 0) *taken = mine ? 1u : 0u;
    }
    __syncthreads();
    const bool ours = __builtin_amdgcn_readfirstlane((int)*taken) != 0;
    if (ours) clear_words(records, record_words, threadIdx.x, 256);
    __syncthreads();
    if (ours) clearing_done(p.clear_word, p.epoch, threadIdx.x);
  }
  // In front of every write into a record.
  auto wait_cleared = [&]() __attribute__((always_inline)) {
    if (clearing) cleared(records, record_words, p.clear_word, p.epoch, seen, lane, 64);
  };

  // ---- this wave's fault
  TrialFault f = {};
  f.kind = FI_SITE_NONE; f.event = -1;
  bool owns = false;                                      // it reaches an element of this tile
  if constexpr (MODE == SMALL_CAMPAIGN) {
    f = decode_fault(p, trial);
    owns = works && f.reaches(m0, n0);
    if (clearing && owns) seen = __hip_atomic_load(p.clear_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (owns && f.kind == FI_SITE_PRODUCT) fetch_product_terms<DT>(f, p);
  }
  const int event = owns ? f.event : -1;

  // the epilogue's inputs, requested before anything is waited for
  const int row_base = m0 + 4 * lhi, col = n0 + l32;      // rows + 8*q + e; the vectors are zero padded
  f32x4 kra4[4] = {};
  float cbj = 0.0f;
  if (works) {
#pragma unroll
    for (int q = 0; q < 4; ++q) kra4[q] = *reinterpret_cast<const f32x4*>(p.kra + row_base + 8 * q);
    cbj = p.cb[col];
  }

  // ---- staging, as in gemm_fi_multi_kernel: rows 0 .. 31 the A tile, then the B tiles.  Wave w
  // loads row groups w, w + 4, ...; every wave issues G_W loads per k-tile (one group may come twice).
  const int lrow = lane >> 3, lslot = lane & 7;
  const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(PROP ? p.A + (size_t)trial * p.a_trial_stride : p.A), 0, (int)(uint32_t)(((size_t)(p.M - 1) * p.lda + (size_t)p.K) * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.B), 0, (int)(uint32_t)(((size_t)(p.N - 1) * p.ldb + (size_t)p.K) * 2), 0x00020000);
  static_assert(GROUPS % 4 == 0, "every wave loads its own row groups");
  uint32_t goff[G_W];                                     // byte offset of this lane's chunk at k = 0
  static_for<G_W>([&](auto cc) {
    constexpr int c = cc;
    const int r = (c * 4 + wave) * 8 + lrow;
    const uint32_t chunk = (uint32_t)((lslot ^ lds_swizzle(r)) * 8);
    if constexpr (c == 0) goff[c] = ((uint32_t)min(m0 + r, p.M - 1) * p.lda + chunk) * 2u;       // 4 groups of A
    else goff[c] = ((uint32_t)min(strip_n0 + r - 32, p.N - 1) * p.ldb + chunk) * 2u;
  });
  auto issue_tile = [&](int kt, int buf) __attribute__((always_inline)) {
    const int k0 = kt * BK;
    uint8_t* const s = smem + buf * STAGE + wave * 1024;
    // Two copies behind a uniform branch: with the lane's and the scalar offset chosen by one condition in
    // one copy, the scalar one landed in a vector register and every load in a loop over its values.
    if (k0 + BK <= p.K) {
      static_for<G_W>([&](auto cc) {
        constexpr int c = cc;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(c == 0 ? rsrc_a : rsrc_b, (lds_void*)(s + c * 4096), 16, (int)goff[c], k0 * 2, 0, 0);
      });
    } else {
      // a ragged last tile: chunks past K are fetched from the start of their row and never used
      static_for<G_W>([&](auto cc) {
        constexpr int c = cc;
        const int ch = (lslot ^ lds_swizzle((c * 4 + wave) * 8 + lrow)) * 8;
        const uint32_t off = k0 + ch < p.K ? goff[c] + 2u * (uint32_t)k0 : goff[c] - 2u * (uint32_t)ch;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(c == 0 ? rsrc_a : rsrc_b, (lds_void*)(s + c * 4096), 16, (int)off, 0, 0, 0);
      });
    }
  };
  const int nkt = (p.K + BK - 1) / BK, n_steps = p.K / 16;
  for (int kt = 0; kt < min(NBUF - 1, nkt); ++kt) issue_tile(kt, kt);

  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 acc = zero;
  [[maybe_unused]] f32x16 sum = zero;
  uint32_t before = 0, after = 0;
  const int sw = lds_swizzle(l32);
  const int a_rd = l32 * 128, b_rd = (32 + wave / TPW * 32 + l32) * 128;
  int buf = 0;
  for (int kt = 0; kt < nkt; ++kt) {
    // this wave's loads of tile kt have landed once only those of the tiles after it are in flight
    static_assert(NBUF <= 4 && 2 * G_W < 64, "tiles after it: up to two");
    const int later = min(NBUF - 2, nkt - 1 - kt);
    if (NBUF == 4 && later == 2) __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * G_W & 15) | (2 * G_W >> 4 << 14));
    else if (later >= 1) __builtin_amdgcn_s_waitcnt(0x0F70 | G_W);
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    __builtin_amdgcn_s_waitcnt(0xC07F);                   // lgkmcnt(0): no read of the tile before is in flight
    // after the barrier the tile is there for all, and nobody reads the tile before it any more
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (kt + NBUF - 1 < nkt) issue_tile(kt + NBUF - 1, buf == 0 ? NBUF - 1 : buf - 1);
    const uint8_t* const s = smem + buf * STAGE;
    buf = buf == NBUF - 1 ? 0 : buf + 1;
    if (!works) continue;
    const int g = 4 * kt;
    auto fragment = [&](int rd, int u) __attribute__((always_inline)) {
      return *reinterpret_cast<const u32x4*>(s + rd + (((2 * u + lhi) ^ sw) << 4));
    };
    if (__builtin_expect(g + 4 <= n_steps && (MODE != SMALL_CAMPAIGN || (event >> 2) != kt), 1)) {
      u32x4 a[4], b[4];
      static_for<4>([&](auto uu) {
        a[uu] = fragment(a_rd, uu);
        b[uu] = fragment(b_rd, uu);
      });
      static_for<4>([&](auto uu) {
        acc = mfma_32x32x16<DT>(a[uu], b[uu], acc);
        if constexpr (SUMS) sum = mfma_32x32x16<DT>(a[uu] & 0x7FFF7FFFu, b[uu] & 0x7FFF7FFFu, sum);
      });
    } else {
      // a ragged last tile, or one with this wave's event: a loop, so that the event's code exists once
#pragma unroll 1
      for (int u = 0; u < min(4, n_steps - g); ++u) {
        u32x4 a = fragment(a_rd, u), b = fragment(b_rd, u);
        if (MODE == SMALL_CAMPAIGN && g + u == event) {
          acc = faulty_step<DT>(f, a, b, acc, m0, n0, lane, before, after);
        } else {
          acc = mfma_32x32x16<DT>(a, b, acc);
          if constexpr (SUMS) sum = mfma_32x32x16<DT>(a & 0x7FFF7FFFu, b & 0x7FFF7FFFu, sum);
        }
      }
    }
  }
  if (!works) return;

  if constexpr (SUMS) {
    // the elements of the fault-free result that the plan's own detector flags are counted
    uint32_t n_clean = 0;
    const float t_all = golden_t_global(p);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = row_base + 8 * (v >> 2) + (v & 3);
      const bool in = row < p.M && col < p.N;
      const float th = p.bound_global ? t_all : __fmul_rn(__fmul_rn(kra4[v >> 2][v & 3], cbj), p.gamma);
      if (in) {
        p.c_out[(size_t)row * p.N + col] = acc[v];
        p.s_out[(size_t)row * p.N + col] = sum[v];
      }
      n_clean += (uint32_t)__builtin_popcountll(__ballot(in && !(fabsf(acc[v]) <= th)));
    }
    if (n_clean != 0 && lane == 0) atomicAdd(p.n_clean, n_clean);
    return;
  } else {
    f32x16 T;
    const uint32_t n_flag = detect_tile<DT>(p, acc, T, kra4, cbj, trial, m0, n0, lane);
    fi_trial_result* const r = p.results + trial;
    const bool invalid = MODE == SMALL_CAMPAIGN && !f.valid && m0 == 0 && n0 == 0;
    if (n_flag != 0 || owns || invalid) wait_cleared();
    if (invalid && lane == 0) r->status = 1;
    if (n_flag != 0 && lane == 0) atomicAdd(&r->n_flagged, n_flag);
    if constexpr (PROP) {
      // most tiles equal the fault-free result bit for bit and hold nothing that is flagged (a corrected
      // element deviates whatever it was compared with) or not finite: nothing to count
      float cs[16];
      bool differs = n_flag != 0;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = row_base + 8 * (v >> 2) + (v & 3);
        cs[v] = p.c_star[(size_t)min(row, p.M - 1) * p.N + min(col, p.N - 1)];
        differs |= row < p.M && col < p.N && (__float_as_uint(acc[v]) != __float_as_uint(cs[v]) || not_finite(acc[v]));
      }
      if (__ballot(differs) != 0) {
        Deviations d;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = row_base + 8 * (v >> 2) + (v & 3);
          const float sa = p.s_abs[(size_t)min(row, p.M - 1) * p.N + min(col, p.N - 1)];
          d.account(row < p.M && col < p.N, acc[v], T[v], cs[v], sa, p.policy);
        }
        const uint32_t n_bit = wave_sum(d.n_bit), n_pre = wave_sum(d.n_pre), n_post = wave_sum(d.n_post);
        const uint32_t n_bT = wave_sum(d.n_bT), n_btau = wave_sum(d.n_btau);
        const uint32_t mp = wave_max(__float_as_uint(d.mx_pre)), mq = wave_max(__float_as_uint(d.mx_post));
        wait_cleared();
        if (lane == 0) {
          if (n_bit) atomicAdd(&r->n_bitdiff, n_bit);
          if (n_pre) atomicAdd(&r->n_dev_pre, n_pre);
          if (n_post) atomicAdd(&r->n_dev_post, n_post);
          if (n_bT) atomicAdd(&r->n_border_T, n_bT);
          if (n_btau) atomicAdd(&r->n_border_tau, n_btau);
          if (mp) atomicMax(reinterpret_cast<uint32_t*>(&r->max_dev_pre), mp);
          if (mq) atomicMax(reinterpret_cast<uint32_t*>(&r->max_dev_post), mq);
        }
      }
    }
    if (owns) {
      const TileDeviation d = tile_deviation(f, p, acc, T, m0, n0, lane);
      // non-negative floats (and +Inf) order like their words
      const uint32_t mp = wave_max(__float_as_uint(d.mx_pre)), mq = wave_max(__float_as_uint(d.mx_post));
      if (lane == 0) {
        if (d.n_bit) atomicAdd(&r->n_bitdiff, d.n_bit);
        if (d.n_pre) atomicAdd(&r->n_dev_pre, d.n_pre);
        if (d.n_post) atomicAdd(&r->n_dev_post, d.n_post);
        if (d.n_bT) atomicAdd(&r->n_border_T, d.n_bT);
        if (d.n_btau) atomicAdd(&r->n_border_tau, d.n_btau);
        if (mp) atomicMax(reinterpret_cast<uint32_t*>(&r->max_dev_pre), mp);
        if (mq) atomicMax(reinterpret_cast<uint32_t*>(&r->max_dev_post), mq);
        // the faulted operand word, once per trial
        if (f.operand() && (f.isA() ? n0 == 0 : m0 == 0)) {
          const uint32_t word = f.isA() ? p.A[(size_t)f.row * p.lda + f.col] : p.B[(size_t)f.col * p.ldb + f.row];
          r->site_word_before = word;
          r->site_word_after = word ^ (f.mask & 0xFFFFu);
        }
      }
      if (!f.operand() && lane == ((int)f.col - n0) + 32 * ((((int)f.row - m0) >> 2) & 1)) {
        r->site_word_before = before;
        r->site_word_after = after;
        if (f.fired) r->product_flag = 1;
      }
    }
    clock(2);
  }
}

// The smallest problems: one workgroup of 16 waves per trial, a wave for each of its (up to 16) 32 x 32
// tiles, all rows of A and B staged per k-tile.  A trial's record is put together in LDS and written
// once, so the call is this one launch: no records to clear, no atomics.  The host's launches are the
// bound there: 64 trials on 128^3 8.8 us against 10.6 us for fill and gemm_fi_small_kernel.  (Five tiles
// per wave, for problems up to 300 x 256, spilled 200 registers and took 49 us against 11.)
template <int DT>
__global__ void __launch_bounds__(1024) gemm_fi_trial_kernel(const GemmArgs p) {
  constexpr int BK = 64, LOADS = 5;                       // 8-row groups per wave: (tiles_m + tiles_n) * 4 <= 68
  extern __shared__ __attribute__((aligned(16))) uint8_t tsmem[];   // two stages
  __shared__ uint32_t part[16][8];
  __shared__ uint32_t site[3];                            // word before, after, product check fired
  typedef __attribute__((address_space(3))) void lds_void;
  const int lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int trial = (int)blockIdx.x;
  const int n_tiles = p.tiles_m * p.tiles_n, rows = 32 * (p.tiles_m + p.tiles_n), stage_bytes = rows * 128;
  if (p.clocks && trial == 0 && threadIdx.x == 0) {       // see GemmArgs::clocks
    p.clocks[0] = __builtin_readcyclecounter();
    p.clocks[1] = __builtin_amdgcn_s_memrealtime();
  }
  if (threadIdx.x < 3) site[threadIdx.x] = 0;
  TrialFault f = decode_fault(p, trial);

  // ---- staging: wave w loads row groups w, w + 16, ...
  const int lrow = lane >> 3, lslot = lane & 7;
  const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.A), 0, (int)(uint32_t)(((size_t)(p.M - 1) * p.lda + (size_t)p.K) * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.B), 0, (int)(uint32_t)(((size_t)(p.N - 1) * p.ldb + (size_t)p.K) * 2), 0x00020000);
  const int groups = rows / 8, groups_a = p.tiles_m * 4;
  uint32_t goff[LOADS];
  static_for<LOADS>([&](auto cc) {
    constexpr int c = cc;
    const int g = c * 16 + wave, r = g * 8 + lrow;        // row inside the stage
    const uint32_t chunk = (uint32_t)((lslot ^ lds_swizzle(r)) * 8);
    goff[c] = g < groups_a ? ((uint32_t)min(r, p.M - 1) * p.lda + chunk) * 2u
                           : ((uint32_t)min(r - 32 * p.tiles_m, p.N - 1) * p.ldb + chunk) * 2u;
  });
  auto issue_tile = [&](int kt, int stage) __attribute__((always_inline)) {
    const int k0 = kt * BK;
    const bool whole = k0 + BK <= p.K;                    // uniform
    static_for<LOADS>([&](auto cc) {
      constexpr int c = cc;
      const int g = c * 16 + wave;                        // uniform
      if (g < groups) {
        // in a ragged last tile, chunks past K are fetched from the start of their row and never used
        const int ch = (lslot ^ lds_swizzle(g * 8 + lrow)) * 8;
        const uint32_t off = whole ? goff[c] : k0 + ch < p.K ? goff[c] + 2u * (uint32_t)k0 : goff[c] - 2u * (uint32_t)ch;
        const int soff = whole ? k0 * 2 : 0;
        uint8_t* const s = tsmem + stage * stage_bytes + g * 1024;
        if (g < groups_a) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (lds_void*)s, 16, (int)off, soff, 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, (lds_void*)s, 16, (int)off, soff, 0, 0);
      }
    });
  };
  issue_tile(0, 0);

  const bool works = wave < n_tiles;                      // uniform; the others stage and keep the barriers
  const int m0 = wave / p.tiles_n * 32, n0 = wave % p.tiles_n * 32;
  const bool owns = works && f.reaches(m0, n0);
  if (owns && f.kind == FI_SITE_PRODUCT) fetch_product_terms<DT>(f, p);
  f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const int nkt = (p.K + BK - 1) / BK, n_steps = p.K / 16;
  const int sw = lds_swizzle(l32);
  uint32_t before = 0, after = 0;
  __builtin_amdgcn_s_waitcnt(0x0F70);                     // vmcnt(0)
  __syncthreads();
  for (int kt = 0; kt < nkt; ++kt) {
    if (kt + 1 < nkt) issue_tile(kt + 1, (kt + 1) & 1);
    const uint8_t* const s = tsmem + (kt & 1) * stage_bytes;
    const int g = 4 * kt;
    if (works) {
      auto fragment = [&](int row, int u) __attribute__((always_inline)) {
        return *reinterpret_cast<const u32x4*>(s + row * 128 + (((2 * u + lhi) ^ sw) << 4));
      };
      const int ra = m0 + l32, rb = 32 * p.tiles_m + n0 + l32;
      if (g + 4 <= n_steps && !(owns && (f.event >> 2) == kt)) {
        static_for<4>([&](auto u) { acc = mfma_32x32x16<DT>(fragment(ra, u), fragment(rb, u), acc); });
      } else {
#pragma unroll 1
        for (int u = 0; u < min(4, n_steps - g); ++u) {
          const u32x4 a = fragment(ra, u), b = fragment(rb, u);
          if (owns && g + u == f.event) acc = faulty_step<DT>(f, a, b, acc, m0, n0, lane, before, after);
          else acc = mfma_32x32x16<DT>(a, b, acc);
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                   // vmcnt(0): this wave's loads have landed
    __syncthreads();
  }

  // ---- detector, outputs and deviations
  uint32_t n[6] = {0, 0, 0, 0, 0, 0}, mp = 0, mq = 0;
  if (works) {
    f32x4 kra4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) kra4[q] = *reinterpret_cast<const f32x4*>(p.kra + m0 + 4 * lhi + 8 * q);   // zero padded
    const float cbj = p.cb[n0 + l32];
    f32x16 T;
    n[0] = detect_tile<DT>(p, acc, T, kra4, cbj, trial, m0, n0, lane);
    if (owns) {
      const TileDeviation d = tile_deviation(f, p, acc, T, m0, n0, lane);
      n[1] = d.n_bit; n[2] = d.n_pre; n[3] = d.n_post; n[4] = d.n_bT; n[5] = d.n_btau;
      mp = wave_max(__float_as_uint(d.mx_pre));           // non-negative floats (and +Inf) order like their words
      mq = wave_max(__float_as_uint(d.mx_post));
      if (!f.operand() && lane == ((int)f.col - n0) + 32 * ((((int)f.row - m0) >> 2) & 1)) {
        site[0] = before;
        site[1] = after;
        site[2] = f.fired ? 1u : 0u;
      }
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int q = 0; q < 6; ++q) part[wave][q] = n[q];
    part[wave][6] = mp;
    part[wave][7] = mq;
  }
  __syncthreads();
  if (threadIdx.x < 8) {
    uint32_t x = 0;
    for (int w = 0; w < 16; ++w) x = threadIdx.x < 6 ? x + part[w][threadIdx.x] : max(x, part[w][threadIdx.x]);
    // n_flagged, n_bitdiff, n_dev_pre, n_dev_post, n_border_T, n_border_tau, the two maxima
    constexpr uint32_t word_of = 0x54983210u;             // their words in a record, one hex digit each
    static_assert(offsetof(fi_trial_result, max_dev_pre) == 16 && offsetof(fi_trial_result, n_border_T) == 32, "record layout");
    reinterpret_cast<uint32_t*>(p.results + trial)[(word_of >> (4 * threadIdx.x)) & 15u] = x;
  } else if (threadIdx.x == 8) {
    fi_trial_result* const r = p.results + trial;
    uint32_t b = site[0], a = site[1];
    if (f.operand()) {
      b = f.isA() ? p.A[(size_t)f.row * p.lda + f.col] : p.B[(size_t)f.col * p.ldb + f.row];
      a = b ^ (f.mask & 0xFFFFu);
    }
    r->site_word_before = b;
    r->site_word_after = a;
    r->status = f.valid ? 0u : 1u;
    r->product_flag = site[2];
  }
  if (p.clocks && trial == 0 && threadIdx.x == 0) {
    p.clocks[2] = __builtin_readcyclecounter();
    p.clocks[3] = __builtin_amdgcn_s_memrealtime();
  }
}

}  // namespace fi
