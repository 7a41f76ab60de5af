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
// Measured, record fill included, multi-trial kernel -> this one: 64 trials on 128^3 25 -> 10 us, 24 on
// 300 x 203 x 176 23 -> 10 us (with operand faults 40 -> 10 us, with outputs 47 -> 11 us), 32 on 3136 x
// 64 x 576 27 -> 20 us, 16 on 64 x 64 x 4096 63 -> 40 us; without LDS, fragments straight from global
// memory, the last two took 72 and 62 us (a fragment's 32 rows are 32 cache lines).
//
// The per-element arithmetic is that of gemm_fi_kernel: the same sequence of 16-wide MFMA steps in
// ascending k, hence bit-identical results.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fi.h"
#include "gemm_fi.hpp"

namespace fi {

// SUMS: the plan's fault-free pass; C* to p.c_out and the magnitude sums, from the same fragments
// with the sign bits cleared, to p.s_out.  Else a campaign (p.tiles_m, p.tiles_n in 32 x 32 tiles).
template <int DT, int TPW, bool SUMS>
__global__ void __launch_bounds__(256) gemm_fi_small_kernel(const GemmArgs p) {
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
      p.clocks[at] = __builtin_readcyclecounter();
      p.clocks[at + 1] = __builtin_amdgcn_s_memrealtime();
    }
  };
  clock(0);

  // ---- this wave's fault (all uniform)
  uint32_t fkind = FI_SITE_NONE, frow = 0, fcol = 0, fmask = 0;
  int event = -1;                                         // step that consumes a faulted word, or ends at an accumulator fault
  int fk = 0;
  bool owns = false;                                      // the fault reaches an element of this tile
  float re = 0.0f, re_err = 0.0f;
  bool fired = false;
  if constexpr (!SUMS) {
    const fi_fault f = p.faults[trial];
    fkind = f.kind; frow = f.row; fcol = f.col; fmask = f.xor_mask;
    bool valid = true;
    if (fkind == FI_SITE_ACC) valid = frow < (uint32_t)p.M && fcol < (uint32_t)p.N && f.kblock < (uint32_t)(p.K / p.kb);
    else if (fkind == FI_SITE_PRODUCT) valid = frow < (uint32_t)p.M && fcol < (uint32_t)p.N && f.kblock < (uint32_t)p.K;
    else if (fkind == FI_SITE_A) valid = frow < (uint32_t)p.M && fcol < (uint32_t)p.K;
    else if (fkind == FI_SITE_B) valid = frow < (uint32_t)p.K && fcol < (uint32_t)p.N;
    else if (fkind != FI_SITE_NONE) valid = false;
    if (!valid) {
      if (works && m0 == 0 && n0 == 0 && lane == 0) p.results[trial].status = 1;
      fkind = FI_SITE_NONE;
    }
    const bool in_rows = (int)frow >= m0 && (int)frow < m0 + 32, in_cols = (int)fcol >= n0 && (int)fcol < n0 + 32;
    if (fkind == FI_SITE_ACC) {
      owns = in_rows && in_cols;
      event = (int)((f.kblock + 1) * (uint32_t)p.kb) / 16 - 1;
    } else if (fkind == FI_SITE_PRODUCT) {
      owns = in_rows && in_cols;
      fk = (int)f.kblock;
      event = fk / 16;
      if (owns)
        product_fault_terms<DT>(p.A[(size_t)frow * p.lda + fk], p.B[(size_t)fcol * p.ldb + fk], fmask, p.product_check,
                                re, re_err, fired);
    } else if (fkind == FI_SITE_A) {
      owns = in_rows;
      fk = (int)fcol;
      event = fk / 16;
    } else if (fkind == FI_SITE_B) {
      owns = in_cols;
      fk = (int)frow;
      event = fk / 16;
    }
    owns = owns && works;
    if (!owns) event = -1;
  }
  const bool operand = fkind == FI_SITE_A || fkind == FI_SITE_B, isA = fkind == FI_SITE_A;
  // an operand fault's word: the lane that holds it and the XOR in the fragment's register sel_w
  const int sel_w = (fk & 7) >> 1;
  const uint32_t x_mine = operand && lane == (int)((isA ? frow - (uint32_t)m0 : fcol - (uint32_t)n0) & 31u) + 32 * ((fk >> 3) & 1)
                              ? (fmask & 0xFFFFu) << (16 * (fk & 1)) : 0u;
  // the faulted element's row inside the tile as register and half-wave
  const int ri = (int)(frow - (uint32_t)m0) & 31;
  const int sel_v = 4 * (ri >> 3) + (ri & 3), sel_hi = (ri >> 2) & 1;

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
      const_cast<uint16_t*>(p.A), 0, (int)(uint32_t)(((size_t)(p.M - 1) * p.lda + (size_t)p.K) * 2), 0x00020000);
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
    static_for<G_W>([&](auto cc) {
      constexpr int c = cc;
      const int ch = (lslot ^ lds_swizzle((c * 4 + wave) * 8 + lrow)) * 8;
      // in a ragged last tile, chunks past K are fetched from the start of their row and never used
      const bool whole = k0 + BK <= p.K;                  // uniform
      const uint32_t off = whole ? goff[c] : k0 + ch < p.K ? goff[c] + 2u * (uint32_t)k0 : goff[c] - 2u * (uint32_t)ch;
      const int soff = whole ? k0 * 2 : 0;
      if constexpr (c == 0)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (lds_void*)(s + c * 4096), 16, (int)off, soff, 0, 0);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, (lds_void*)(s + c * 4096), 16, (int)off, soff, 0, 0);
    });
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
    if (__builtin_expect(g + 4 <= n_steps && (SUMS || (event >> 2) != kt), 1)) {
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
        const bool here = !SUMS && g + u == event;
        if (here && operand) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint32_t x = r == sel_w ? x_mine : 0u;
            a[r] ^= isA ? x : 0u;
            b[r] ^= isA ? 0u : x;
          }
        }
        acc = mfma_32x32x16<DT>(a, b, acc);
        if constexpr (SUMS) sum = mfma_32x32x16<DT>(a & 0x7FFF7FFFu, b & 0x7FFF7FFFu, sum);
        if (here && !operand) {
          const bool product = fkind == FI_SITE_PRODUCT;
          const bool mine = lhi == sel_hi && col == (int)fcol;
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const uint32_t word = __float_as_uint(acc[v]);
            const uint32_t nw = product ? __float_as_uint(write_back(acc[v], re, re_err)) : (word ^ fmask);
            before = v == sel_v ? word : before;
            after = v == sel_v ? nw : after;
            acc[v] = __uint_as_float((v == sel_v && mine) ? nw : word);
          }
        }
      }
    }
  }
  if (!works) return;
  if (!SUMS && event >= 0 && !operand && lhi == sel_hi && col == (int)fcol) {
    p.results[trial].site_word_before = before;
    p.results[trial].site_word_after = after;
    if (fired) p.results[trial].product_flag = 1;
  }

  const bool ragged = m0 + 32 > p.M || n0 + 32 > p.N;
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
    // ---- detector on every element; those outside the problem (copies of the last row or column)
    // get T = +Inf and the value 0: never flagged, stored or counted
    f32x16 T;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float th = p.bound_global ? p.t_global : __fmul_rn(__fmul_rn(kra4[v >> 2][v & 3], cbj), p.gamma);
      T[v] = th;
    }
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
    fi_trial_result* const r = p.results + trial;
    if (any != 0) {
      uint32_t n_flag = 0;
#pragma unroll
      for (int v = 0; v < 16; ++v) n_flag += (uint32_t)__builtin_popcountll(__ballot(!(fabsf(acc[v]) <= T[v])));
      if (lane == 0) atomicAdd(&r->n_flagged, n_flag);
    }
    // ---- outputs: corrected where flagged, in FP32 or handed on in the operand format
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
    // ---- deviation from the fault-free result, where the fault reaches: one element, one row (it
    // lies in one register and half-wave) or one column (gathered into lanes 0 .. 31, row k to lane k)
    if (!owns) {
      clock(2);
      return;
    }
    float c = acc[0], th = T[0];
    int row, cc_col;
    bool act;
    if (fkind != FI_SITE_B) {
#pragma unroll
      for (int v = 1; v < 16; ++v) {
        c = v == sel_v ? acc[v] : c;
        th = v == sel_v ? T[v] : th;
      }
      row = (int)frow;
      cc_col = min(col, p.N - 1);
      act = lhi == sel_hi && col < p.N && (isA || col == (int)fcol);
    } else {
      const int sel = (int)fcol - n0;
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
      cc_col = (int)fcol;
      th = p.bound_global ? p.t_global : __fmul_rn(__fmul_rn(p.kra[row], p.cb[fcol]), p.gamma);
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
    const uint32_t n_bit = (uint32_t)__builtin_popcountll(changed);
    const uint32_t n_pre = (uint32_t)__builtin_popcountll(__ballot(!(dpre <= tau)) & am);
    const uint32_t n_post = (uint32_t)__builtin_popcountll(__ballot(!(dpost <= tau)) & am);
    const uint32_t n_bT = (uint32_t)__builtin_popcountll(changed & __ballot(mag <= 3.4028234e38f) & __ballot(fabsf(mag - th) <= band));
    const uint32_t n_btau = (uint32_t)__builtin_popcountll(changed & __ballot(tau > 0.0f) & __ballot(dpre >= 0.5f * tau) &
                                                           __ballot(dpre <= 2.0f * tau));
    // non-negative floats (and +Inf) order like their words
    const uint32_t mp = wave_max(act ? __float_as_uint(dpre) : 0u), mq = wave_max(act ? __float_as_uint(dpost) : 0u);
    if (lane == 0) {
      if (n_bit) atomicAdd(&r->n_bitdiff, n_bit);
      if (n_pre) atomicAdd(&r->n_dev_pre, n_pre);
      if (n_post) atomicAdd(&r->n_dev_post, n_post);
      if (n_bT) atomicAdd(&r->n_border_T, n_bT);
      if (n_btau) atomicAdd(&r->n_border_tau, n_btau);
      if (mp) atomicMax(reinterpret_cast<uint32_t*>(&r->max_dev_pre), mp);
      if (mq) atomicMax(reinterpret_cast<uint32_t*>(&r->max_dev_post), mq);
      // the faulted operand word, once per trial
      if (operand && (isA ? n0 == 0 : m0 == 0)) {
        const uint32_t word = isA ? p.A[(size_t)frow * p.lda + fcol] : p.B[(size_t)fcol * p.ldb + frow];
        r->site_word_before = word;
        r->site_word_after = word ^ (fmask & 0xFFFFu);
      }
    }
    clock(2);
  }
}

}  // namespace fi
