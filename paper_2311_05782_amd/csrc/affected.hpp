// Campaigns restricted to what a fault can reach (fi_gemm_inject_batch_affected), gfx950.
//
// A trial's fault reaches one output element (accumulator flip, product-term fault), one output
// row (A-operand fault) or one output column (B-operand fault); everything else equals the
// fault-free result bit for bit.  An element of a 32x32x16 MFMA depends on its own row of the
// first operand and its own column of the second only, so rows and columns of DIFFERENT trials
// can share one instruction: nothing but the reached elements has to be computed, and each
// still passes the sequence of 16-wide steps in ascending k that the full campaign feeds it.
//   - elements: one wave takes four trials; lane l supplies A row and B column of trial l % 4, and
//     trial r's element is the diagonal one, register r of lane r;
//   - rows and columns: the faulted rows (columns) of 64 trials are gathered into one operand of
//     64 rows, multiplied with the whole other operand.
// Measured, a call among others: 1024 accumulator faults on 4096^3 14 us (195 .. 263 us with a 128 x 128
// tile around every element), 4096 trials on 512 x 3072 x 768, half of them A faults, 48 us (4195 us with
// a tile row of 128 rows per operand fault), all B faults 57 us (1088 us).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "fi.h"
#include "gemm_fi.hpp"

namespace fi {

constexpr int kElemTrials = 4;        // trials per wave of the element kernel
constexpr int kRowsChunk = 512;       // consecutive trials whose operand faults are gathered together
constexpr int kRowsTrials = 64;       // gathered rows per work item
constexpr int kRowsX = 128;           // rows of the other operand per work item
constexpr int kRowsBuf = 2;           // k-tile buffers: a third leaves room for two workgroups per CU, 38 -> 45 us
// A chunk of trials fills at most this many items of one kind after the other: the A and the B
// faults are gathered separately, so one more than kRowsChunk / kRowsTrials.
constexpr int kRowsSlots = kRowsChunk / kRowsTrials + 1;

// What a row / column workgroup has counted of a trial: {n_flagged, n_bitdiff, n_dev_pre, n_dev_post, n_border_T,
// n_border_tau, max_dev_pre, max_dev_post}.  With scratch for them (`parts`, [x slot][trial]) the row / column kernel
// comes first, each workgroup leaves its own and the element kernel adds up; without, the element kernel comes
// first and they are added to the record: updates of one 128-byte line come one after the other, and with 24 slots
// each takes some 290 of them (4096 trials on 512 x 3072 x 768, half of them A faults: 46.0 -> 38.6 us; without any record
// written 38.5).
constexpr uint32_t kPartWords = 8;

// What can be told from a fault's coordinates: 0 nothing to compute (no fault), 1 one element,
// 2 an A row, 3 a B column, 4 outside the problem.
__device__ __forceinline__ int affected_kind(const fi_fault& f, const GemmArgs& p) {
  if (f.kind == FI_SITE_ACC)
    return f.row < (uint32_t)p.M && f.col < (uint32_t)p.N && f.kblock < (uint32_t)(p.K / p.kb) ? 1 : 4;
  if (f.kind == FI_SITE_PRODUCT)
    return f.row < (uint32_t)p.M && f.col < (uint32_t)p.N && f.kblock < (uint32_t)p.K ? 1 : 4;
  if (f.kind == FI_SITE_A) return f.row < (uint32_t)p.M && f.col < (uint32_t)p.K ? 2 : 4;
  if (f.kind == FI_SITE_B) return f.row < (uint32_t)p.K && f.col < (uint32_t)p.N ? 3 : 4;
  return f.kind == FI_SITE_NONE ? 0 : 4;
}

// Element kernel: one wave per kElemTrials consecutive trials.  Writes every trial's whole record:
// the final one of element faults, fault-free trials and bad sites, and for operand faults the site
// words with zeroed counters, to which affected_rows_kernel adds.
//
// Bound: the chain of K/16 dependent MFMAs (32 cycles each: some 4 us of 12 us at K = 4096) and the
// memory latency in front of it, so the operands must not be waited for again.  1024 trials on
// 4096^3: 15.6 us with one piece in flight and the fragment reads of a group in one block, 12.4 us
// with three pieces and the reads between the MFMAs.  The 2 x 4 rows stream into LDS in pieces of 512 * IPR k, whole rows in
// 1 KB loads that need no registers, the next NBUF - 1 pieces in flight under the steps of this one.  Four
// trials per wave put 1024 trials on 256 CUs; more per wave would leave CUs idle, fewer would load
// the LDS pipe with reads of the same bytes.  Rows lie 32 bytes apart modulo the 256 bytes of the
// banks, so that the eight 16-byte words of a fragment read fall on different banks.
template <int DT, int IPR, int NBUF, bool PARTS>
__global__ void __launch_bounds__(64, 2) affected_element_kernel(const GemmArgs p, const uint32_t* parts, int n_x_slots) {
  constexpr int T = kElemTrials;
  constexpr int STRIDE = IPR * 1024 + 32, BUF = 2 * T * STRIDE;
  constexpr int STEPS = IPR * 32;                         // 16-wide steps in a piece
  extern __shared__ __attribute__((aligned(16))) uint8_t esmem[];   // min(NBUF, pieces of K) buffers
  typedef __attribute__((address_space(3))) void lds_void;
  typedef const __attribute__((address_space(1))) void glb_void;

  const int lane = threadIdx.x, l32 = lane & 31, lhi = lane >> 5, slot = lane & (T - 1);
  const uint32_t t_mine = blockIdx.x * T + slot;
  const bool have = t_mine < (uint32_t)p.n_trials;
  const fi_fault f = p.faults[have ? t_mine : 0];
  const int kind = have ? affected_kind(f, p) : 0;
  const bool element = kind == 1, product = element && f.kind == FI_SITE_PRODUCT;
  uint32_t before = 0, after = 0, product_flag = 0;
  Deviations dev;

  const bool operand = kind == 2 || kind == 3;
  if (operand) before = kind == 2 ? p.A[(size_t)f.row * p.lda + f.col] : p.B[(size_t)f.col * p.ldb + f.row];
  if (__ballot(element) != 0) {
    const uint32_t row = element ? f.row : 0u, col = element ? f.col : 0u;
    // what the accounting needs, requested before the operands
    const size_t idx = (size_t)row * (size_t)p.N + col;
    const float cs = p.c_star[idx], sabs = p.s_abs[idx], kra = p.kra[row], cb = p.cb[col];
    float re = 0.0f, re_err = 0.0f;
    if (product) {
      bool fired;
      product_fault_terms<DT>(p.A[(size_t)row * p.lda + f.kblock], p.B[(size_t)col * p.ldb + f.kblock], f.xor_mask,
                              p.product_check, re, re_err, fired);
      product_flag = fired ? 1u : 0u;
    }
    // the 16-wide step after which the accumulator changes
    const int step_mine = !element ? -1 : product ? (int)(f.kblock / 16) : (int)((f.kblock + 1) * (uint32_t)p.kb) / 16 - 1;
    int ev[T];
    const uint16_t* rows[2 * T];
    static_for<T>([&](auto rr) {
      constexpr int r = rr;
      ev[r] = __builtin_amdgcn_readlane(step_mine, r);
      rows[r] = p.A + (size_t)(uint32_t)__builtin_amdgcn_readlane((int)row, r) * p.lda;
      rows[T + r] = p.B + (size_t)(uint32_t)__builtin_amdgcn_readlane((int)col, r) * p.ldb;
    });
    const int n_chunks = p.K / 8;                         // 16-byte chunks of a row
    const int n_steps = p.K / 16, n_pieces = (n_steps + STEPS - 1) / STEPS;
    auto issue = [&](int piece, int buf) {
      // lanes past the end of a row fetch its last chunk again: never used
#pragma unroll
      for (int i = 0; i < IPR; ++i) {
        const int chunk = min((piece * IPR + i) * 64 + lane, n_chunks - 1);
        static_for<2 * T>([&](auto q) {
          __builtin_amdgcn_global_load_lds((glb_void*)(rows[q] + chunk * 8),
                                           (lds_void*)(esmem + buf * BUF + q * STRIDE + i * 1024), 16, 0, 0);
        });
      }
    };
    f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // A group of 8 steps; each MFMA is followed by the fragment reads of its step in the next group.
    constexpr int GRP = 8;
    struct Frags { u32x4 a[GRP], b[GRP]; };
    const int rd = slot * STRIDE + lhi * 16;
    auto read_step = [&](Frags& fr, auto uu, const uint8_t* s, int step) __attribute__((always_inline)) {
      constexpr int u = uu;
      fr.a[u] = *reinterpret_cast<const u32x4*>(s + rd + (step + u) * 32);
      fr.b[u] = *reinterpret_cast<const u32x4*>(s + T * STRIDE + rd + (step + u) * 32);
    };
    static_assert(T == 4, "the events of four trials are tested one by one");
    auto event_after = [&](int g) __attribute__((always_inline)) {
      static_for<T>([&](auto rr) {
        constexpr int r = rr;
        const bool hit = lane == r && step_mine == g;
        const uint32_t w = __float_as_uint(acc[r]);
        const uint32_t nw = product ? __float_as_uint(write_back(acc[r], re, re_err)) : w ^ f.xor_mask;
        before = hit ? w : before;
        after = hit ? nw : after;
        acc[r] = hit ? __uint_as_float(nw) : acc[r];
      });
    };
    int next_ev = -1;                                     // earliest event at or after the current group
    auto run_group = [&](const Frags& fr, Frags& fn, const uint8_t* s, int next_step, int g, int end)
                         __attribute__((always_inline)) {
      if (g > next_ev) {
        next_ev = 0x7fffffff;
        static_for<T>([&](auto r) { next_ev = ev[r] >= g && ev[r] < next_ev ? ev[r] : next_ev; });
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);                 // lgkmcnt(0): this group's fragments
      __builtin_amdgcn_sched_barrier(0);
      if (next_ev >= g + GRP && g + GRP <= end) {
        static_for<GRP>([&](auto uu) {
          constexpr int u = uu;
          acc = mfma_32x32x16<DT>(fr.a[u], fr.b[u], acc);
          __builtin_amdgcn_sched_barrier(0);
          read_step(fn, uu, s, next_step);
          __builtin_amdgcn_sched_barrier(0);
        });
      } else {
        static_for<GRP>([&](auto uu) { read_step(fn, uu, s, next_step); });
        static_for<GRP>([&](auto uu) {
          constexpr int u = uu;
          if (g + u < end) {
            acc = mfma_32x32x16<DT>(fr.a[u], fr.b[u], acc);
            if (ev[0] == g + u || ev[1] == g + u || ev[2] == g + u || ev[3] == g + u) event_after(g + u);
          }
        });
      }
    };
    // all loads but those of the `later` youngest pieces have landed
    auto wait_pieces = [&](int later) __attribute__((always_inline)) {
      constexpr int L = 2 * T * IPR;                      // loads of a piece
      static_assert((NBUF - 1) * L < 64, "the counter of loads in flight has six bits");
      if (NBUF > 3 && later == 3) __builtin_amdgcn_s_waitcnt(0x0F70 | (3 * L & 15) | (3 * L >> 4 << 14));
      else if (NBUF > 2 && later == 2) __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * L & 15) | (2 * L >> 4 << 14));
      else if (later == 1) __builtin_amdgcn_s_waitcnt(0x0F70 | (L & 15) | (L >> 4 << 14));
      else __builtin_amdgcn_s_waitcnt(0x0F70);
    };
    for (int piece = 0; piece < min(NBUF - 1, n_pieces); ++piece) issue(piece, piece);
    int buf = 0;
    for (int piece = 0; piece < n_pieces; ++piece) {
      // into the buffer of the piece before this one, every read of which has returned
      if (piece + NBUF - 1 < n_pieces) issue(piece + NBUF - 1, buf == 0 ? NBUF - 1 : buf - 1);
      wait_pieces(min(NBUF - 1, n_pieces - 1 - piece));
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const uint8_t* s = esmem + buf * BUF;
      const int base = piece * STEPS, ns = min(STEPS, n_steps - base);
      Frags f0, f1;
      static_for<GRP>([&](auto uu) { read_step(f0, uu, s, 0); });
      for (int g = 0; g < ns; g += 2 * GRP) {             // a piece holds whole pairs of groups
        run_group(f0, f1, s, g + GRP, base + g, base + ns);
        if (g + GRP >= ns) break;
        // the last group of the buffer reads its own first steps again: not used
        run_group(f1, f0, s, g + 2 * GRP < STEPS ? g + 2 * GRP : 0, base + g + GRP, base + ns);
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);                 // lgkmcnt(0): no read of this buffer is in flight
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      buf = buf == NBUF - 1 ? 0 : buf + 1;
    }
    float c = acc[0];
    static_for<T>([&](auto rr) {
      constexpr int r = rr;
      c = slot == r ? acc[r] : c;
    });
    const float th = p.bound_global ? p.t_global : __fmul_rn(__fmul_rn(kra, cb), p.gamma);
    dev.account(element, c, th, cs, sabs, p.policy);
  }
  if (PARTS && __ballot(operand) != 0) {
    // Operand faults: lane l adds up the slots l / 4, l / 4 + 16, ... of trial l % 4.
    static_assert(T == 4, "four trials' parts fill a line");
    const int filled = operand ? min(n_x_slots, ((kind == 2 ? p.N : p.M) + kRowsX - 1) / kRowsX) : 0;
    uint32_t sum[6] = {0, 0, 0, 0, 0, 0}, mp = 0, mq = 0;
    for (int s = lane >> 2; s < filled; s += 16) {
      const u32x4* const at = reinterpret_cast<const u32x4*>(parts + ((size_t)s * p.n_trials + t_mine) * kPartWords);
      const u32x4 lo = at[0], hi = at[1];
      sum[0] += lo[0]; sum[1] += lo[1]; sum[2] += lo[2]; sum[3] += lo[3]; sum[4] += hi[0]; sum[5] += hi[1];
      mp = max(mp, hi[2]); mq = max(mq, hi[3]);
    }
    for (int o = 4; o < 64 && __ballot(4 * filled > o) != 0; o <<= 1) {
#pragma unroll
      for (int q = 0; q < 6; ++q) sum[q] += (uint32_t)__shfl_xor((int)sum[q], o, 64);
      mp = max(mp, (uint32_t)__shfl_xor((int)mp, o, 64));
      mq = max(mq, (uint32_t)__shfl_xor((int)mq, o, 64));
    }
    if (filled != 0) {
      dev.n_flag = sum[0]; dev.n_bit = sum[1]; dev.n_pre = sum[2]; dev.n_post = sum[3]; dev.n_bT = sum[4]; dev.n_btau = sum[5];
      dev.mx_pre = __uint_as_float(mp); dev.mx_post = __uint_as_float(mq);
    }
  }
  if (operand) after = before ^ (f.xor_mask & 0xFFFFu);
  if (lane < T && have) {
    fi_trial_result r;
    r.n_flagged = dev.n_flag; r.n_bitdiff = dev.n_bit; r.n_dev_pre = dev.n_pre; r.n_dev_post = dev.n_post;
    r.max_dev_pre = dev.mx_pre; r.max_dev_post = dev.mx_post;
    r.site_word_before = before; r.site_word_after = after;
    r.n_border_T = dev.n_bT; r.n_border_tau = dev.n_btau;
    r.status = kind == 4 ? 1u : 0u;
    r.product_flag = product_flag;
    p.results[t_mine] = r;
  }
}

// Row / column kernel: the operand faults of kRowsChunk consecutive trials, the A faults and the B
// faults apart, in items of kRowsTrials gathered rows: G, trial t's row with its faulted word XORed
// in LDS by the lane that fetched it, times all rows of the other operand X.  Workgroup = (chunk,
// item, x slot), walking the x tiles with stride n_x_slots; a workgroup without an item leaves after
// one look at the chunk's kinds.
//
// Bound: the k-tiles' latency and LDS reads (1.5 KB per MFMA of a wave), then the accounting of every
// element and the record updates: 37 us for 2048 A faults x 3072 columns x K = 768, 56 us for 4096 B
// faults x 512 rows, whose accounting has no short form.  64 x 128 by four waves takes 48 KB of LDS, three
// workgroups per CU cover each other; the 170 registers that leaves a wave are 10 too few (20 with 64-bit
// addresses), spilled outside the k-loop.
// The lanes of a wave lie along the columns of C in both cases, so that C* and the magnitude sums are
// read in whole lines: A faults feed the MFMA G x X (a register is a trial, a lane an element of its
// row), B faults X x G (a lane is a trial, its registers the elements of its column).
struct RowsLists {
  uint32_t trial[kRowsTrials], row[kRowsTrials], k[kRowsTrials], mask[kRowsTrials];
};

// The row / column kernel compares most elements with kra * (cb * gamma) * 0.97 instead of the three roundings
// T = fl(fl(kra * cb) * gamma).  The two agree to a few ulps while neither leaves the normal range:
// every kra and cb that is not 0 at or above this (a product of two stays normal, a 0 makes the
// limit 0), cb * gamma finite and T below 1.7e38 everywhere.  Plans for which that does not hold take
// the whole rule for every element.
constexpr float kTinyFactor = 0x1p-60f;

// v[LANE] = x (uniform): v_writelane_b32 has no builtin.
template <int LANE>
__device__ __forceinline__ void set_lane(int& v, int x) {
  asm("v_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(x), "n"(LANE));
}

// One item, all its x tiles.  ISA: A faults.  BIG: C* spans 4 GiB or more (64-bit addresses).
template <int DT, bool BIG, bool ISA>
__device__ __forceinline__ void affected_rows_item(const GemmArgs& p, uint8_t* smem, const RowsLists& list, int n_act,
                                                   int x_slot, int n_x_slots, bool plain_holds, uint32_t* parts) {
  constexpr int BK = 64, BT = kRowsTrials, BX = kRowsX;
  constexpr int STAGE = (BT + BX) * 128;
  constexpr int G_G = BT / 8 / 4, X_G = BX / 8 / 4;       // 8-row groups staged per wave
  typedef __attribute__((address_space(3))) void lds_void;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int X = ISA ? p.N : p.M;                          // rows of the other operand
  const int x_tiles = (X + BX - 1) / BX;
  const uint16_t* const Gp = ISA ? p.A : p.B;
  const uint16_t* const Xp = ISA ? p.B : p.A;
  const uint32_t ldg = ISA ? p.lda : p.ldb, ldx = ISA ? p.ldb : p.lda;
  // buffer loads, as in gemm_fi_multi_kernel: scalar base and k offset, one 32-bit offset per lane
  const uint32_t g_bytes = (uint32_t)(((size_t)((ISA ? p.M : p.N) - 1) * ldg + (size_t)p.K) * 2);
  const uint32_t x_bytes = (uint32_t)(((size_t)(X - 1) * ldx + (size_t)p.K) * 2);
  const __amdgpu_buffer_rsrc_t rsrc_g = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(Gp), 0, (int)g_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(Xp), 0, (int)x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_c = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.c_star), 0, (int)p.c_star_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_s = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.s_abs), 0, (int)((uint32_t)p.M * (uint32_t)p.N * 4u), 0x00020000);
  // element (row, col) of C* and of the magnitude sums, as row part + column part in bytes.  C* is
  // padded to whole tiles, loads of the sums past their end give 0: neither is counted
  auto golden = [&](uint32_t row, uint32_t col, float& cs, float& sa) __attribute__((always_inline)) {
    if constexpr (!BIG) {
      const uint32_t at = (row * (uint32_t)p.N + col) * 4u;
      cs = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc_c, (int)at, 0, 0));
      sa = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc_s, (int)at, 0, 0));
    } else {
      const size_t at = (size_t)min(row, (uint32_t)p.M - 1u) * (size_t)p.N + min(col, (uint32_t)p.N - 1u);
      cs = p.c_star[at];
      sa = p.s_abs[at];
    }
  };

  // ---- staging, as in gemm_fi_kernel; the gathered rows' offsets and faults stay for all x tiles
  const int lrow = lane >> 3, lslot = lane & 7;
  uint32_t g_goff[G_G], g_k[G_G], g_mask[G_G];
#pragma unroll
  for (int c = 0; c < G_G; ++c) {
    const int r = (wave * G_G + c) * 8 + lrow;
    g_goff[c] = list.row[r] * ldg + (uint32_t)((lslot ^ lds_swizzle(r)) * 8);
    // the faulted word, if this lane fetches the chunk that holds it
    g_k[c] = ((list.k[r] >> 3) & 7u) == (uint32_t)(lslot ^ lds_swizzle(r)) ? list.k[r] : 0xFFFFFFFFu;
    g_mask[c] = list.mask[r];
  }
  const int wt = wave & 1, wx = wave >> 1;                // 32 trials x 64 rows of X per wave
  const int sw = lds_swizzle(l32);
  const int g_rd = (wt * 32 + l32) * 128, x_rd = (BT + wx * 64 + l32) * 128;
  const int nkt = (p.K + BK - 1) / BK;
  const int last_steps = ((p.K - 1) % BK) / 16 + 1;

  // ISA: counters of trial l32 in lanes 0 .. 31 (from lane masks), the maxima per register (trial)
  // and lane.  Else: lane = trial, everything in its own counters.
  [[maybe_unused]] int n_flag = 0, n_bit = 0, n_pre = 0, n_corr = 0, n_bT = 0, n_btau = 0;
  [[maybe_unused]] const uint64_t plain_ok = plain_holds ? ~0ull : 0ull;   // see kTinyFactor
  [[maybe_unused]] float mxp[ISA ? 16 : 1], mxq[ISA ? 16 : 1];
  [[maybe_unused]] Deviations dev;
  const int q_mine = wt * 32 + l32;                       // this lane's trial (ISA: as a counter)
  const bool act = q_mine < n_act;
  [[maybe_unused]] const uint32_t row_mine = list.row[q_mine];
  [[maybe_unused]] const float g_factor = ISA ? 0.0f : p.cb[row_mine];
  if constexpr (ISA) {
#pragma unroll
    for (int v = 0; v < 16; ++v) { mxp[v] = 0.0f; mxq[v] = 0.0f; }
  }

  for (int xt = x_slot; xt < x_tiles; xt += n_x_slots) {
    const int x0 = xt * BX;
    uint32_t x_goff[X_G];
#pragma unroll
    for (int c = 0; c < X_G; ++c) {
      const int r = (wave * X_G + c) * 8 + lrow;
      x_goff[c] = (uint32_t)min(x0 + r, X - 1) * ldx + (uint32_t)((lslot ^ lds_swizzle(r)) * 8);
    }
    auto issue_tile = [&](int kt, int stage) __attribute__((always_inline)) {
      const int k0 = kt * BK;
      uint8_t* sG = smem + stage * STAGE + wave * (G_G * 1024);
      uint8_t* sX = smem + stage * STAGE + BT * 128 + wave * (X_G * 1024);
      if (k0 + BK <= p.K) {
#pragma unroll
        for (int c = 0; c < G_G; ++c)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_g, (lds_void*)(sG + c * 1024), 16, (int)(g_goff[c] * 2u), k0 * 2, 0, 0);
#pragma unroll
        for (int c = 0; c < X_G; ++c)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_x, (lds_void*)(sX + c * 1024), 16, (int)(x_goff[c] * 2u), k0 * 2, 0, 0);
      } else {
        // chunks past K are fetched from the start of their row and never used
#pragma unroll
        for (int c = 0; c < G_G; ++c) {
          const int ch = (lslot ^ lds_swizzle((wave * G_G + c) * 8 + lrow)) * 8;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_g, (lds_void*)(sG + c * 1024), 16,
                                                   (int)((g_goff[c] + (uint32_t)(k0 + ch < p.K ? k0 : -ch)) * 2u), 0, 0, 0);
        }
#pragma unroll
        for (int c = 0; c < X_G; ++c) {
          const int ch = (lslot ^ lds_swizzle((wave * X_G + c) * 8 + lrow)) * 8;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_x, (lds_void*)(sX + c * 1024), 16,
                                                   (int)((x_goff[c] + (uint32_t)(k0 + ch < p.K ? k0 : -ch)) * 2u), 0, 0, 0);
        }
      }
    };
    // once this wave's loads of k-tile kt have landed, before the barrier that publishes them
    auto fault_tile = [&](int kt, int stage) {
      uint8_t* sG = smem + stage * STAGE + wave * (G_G * 1024) + lane * 16;
#pragma unroll
      for (int c = 0; c < G_G; ++c)
        if ((g_k[c] >> 6) == (uint32_t)kt) *(reinterpret_cast<uint16_t*>(sG + c * 1024) + (g_k[c] & 7u)) ^= (uint16_t)g_mask[c];
    };
    struct Frags { u32x4 g, x[2]; };
    auto read_frags = [&](Frags& fr, const uint8_t* s, int kk) __attribute__((always_inline)) {
      const int at = ((2 * kk + lhi) ^ sw) << 4;
      fr.g = *reinterpret_cast<const u32x4*>(s + g_rd + at);
      fr.x[0] = *reinterpret_cast<const u32x4*>(s + x_rd + at);
      fr.x[1] = *reinterpret_cast<const u32x4*>(s + x_rd + 4096 + at);
    };
    f32x16 acc[2];
    static_for<2>([&](auto i) {
      acc[i] = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    });
    // Tiles kt + 1 .. kt + kRowsBuf - 1 are in flight while tile kt is used; one barrier per k-tile
    // says that tile kt is there for all and that nobody reads the tile before it any more.
    for (int kt = 0; kt < min(kRowsBuf - 1, nkt); ++kt) issue_tile(kt, kt);
    int buf = 0;
    for (int kt = 0; kt < nkt; ++kt) {
      constexpr int L = G_G + X_G;                        // loads of a tile by this wave
      static_assert(kRowsBuf == 2 || kRowsBuf == 3, "waits for one or two tiles in flight");
      if (kRowsBuf == 3 && kt + 1 < nkt) __builtin_amdgcn_s_waitcnt(0x0F70 | L);   // all but the youngest tile's
      else __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0)
      fault_tile(kt, buf);
      __builtin_amdgcn_s_waitcnt(0xC07F);                 // lgkmcnt(0): the fault is in LDS
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (kt + kRowsBuf - 1 < nkt) issue_tile(kt + kRowsBuf - 1, buf == 0 ? kRowsBuf - 1 : buf - 1);
      const int steps = kt + 1 < nkt ? 4 : last_steps;
      const uint8_t* s = smem + buf * STAGE;
      buf = buf == kRowsBuf - 1 ? 0 : buf + 1;
      Frags fr[2];
      read_frags(fr[0], s, 0);
      static_for<4>([&](auto kk) {
        if constexpr (kk + 1 < 4) read_frags(fr[(kk + 1) % 2], s, kk + 1);
        if (kk < steps) {
          static_for<2>([&](auto i) {
            if constexpr (ISA) acc[i] = mfma_32x32x16<DT>(fr[kk % 2].g, fr[kk % 2].x[i], acc[i]);
            else acc[i] = mfma_32x32x16<DT>(fr[kk % 2].x[i], fr[kk % 2].g, acc[i]);
          });
        }
      });
    }
    // every wave is done with the last tiles before the next ones (or the maxima) go into the buffers
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    // ---- detector, corrector and counters
    const int xw = x0 + wx * 64;
    static_for<2>([&](auto ii) {
      constexpr int i = ii;
      __builtin_amdgcn_sched_barrier(0);
      const f32x16 t = acc[i];
      float cs[16], sa[16];
      if constexpr (ISA) {
        // register v: trial 8*(v/4) + 4*lhi + v%4 of the wave's 32, lane: column x of its row
        const int x = xw + 32 * i + l32;
        const bool in = x < X;
        float kra[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const u32x4 rows = *reinterpret_cast<const u32x4*>(list.row + wt * 32 + 8 * q + 4 * lhi);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            golden(rows[e], (uint32_t)x, cs[4 * q + e], sa[4 * q + e]);
            kra[4 * q + e] = p.kra[rows[e]];
          }
        }
        const float cb_x = p.cb[x];                       // zero padded to a multiple of 512
        // Some 30 instructions per register (two trials' 32 elements each): conditions are lane
        // masks in scalar registers, counted there and written to the trial's lane.
        int t_flag = 0, t_bit = 0, t_pre = 0, t_corr = 0, t_bT = 0, t_btau = 0;   // of this tile
        auto count = [&](int& to, auto vv, uint64_t m) __attribute__((always_inline)) {
          constexpr int lo = 8 * (vv >> 2) + (vv & 3);    // trial of lanes 0 .. 31; + 4 in lanes 32 .. 63
          set_lane<lo>(to, __builtin_popcount((uint32_t)m));
          set_lane<lo + 4>(to, __builtin_popcount((uint32_t)(m >> 32)));
        };
        const uint64_t in_mask = __ballot(in);
        // Plain: |c| below 0.97 T (T to a few ulps, see kTinyFactor) and 2 tau below T/64, hence below the
        // band around T, unflagged and finite: nothing is corrected and the deviation is the same before
        // and after.
        const float lim_x = p.bound_global ? 0.97f : cb_x * p.gamma * 0.97f;
        static_for<16>([&](auto vv) {
          constexpr int v = vv;
          const float c = t[v], cse = cs[v];
          const float lim = (p.bound_global ? p.t_global : kra[v]) * lim_x;
          const float tau = sa[v] * 0.000244140625f;      // 2^-12, exact scaling
          const uint64_t plain = __ballot(fabsf(c) < lim) & __ballot(tau * 130.0f <= lim) & plain_ok;
          const uint64_t changed = __ballot(__float_as_uint(c) != __float_as_uint(cse)) & in_mask;
          float dpre = fabsf(c - cse), dpost = dpre;
          uint64_t pre = __ballot(!(dpre <= tau)) & in_mask;
          if ((in_mask & ~plain) != 0) {
            // the whole rule, for both trials of the register
            const float T = p.bound_global ? p.t_global : __fmul_rn(__fmul_rn(kra[v], cb_x), p.gamma);
            const bool flag = !(fabsf(c) <= T);
            float cc = c;
            if (flag && p.policy == FI_CORRECT_ZERO) cc = 0.0f;
            if (flag && p.policy == FI_CORRECT_RECOMPUTE) cc = cse;
            dpre = finite_or_inf(dpre);
            dpost = finite_or_inf(fabsf(cc - cse));
            const float mag = fabsf(c), band = fmaxf(2.0f * tau, T * 0.015625f);
            pre = __ballot(!(dpre <= tau)) & in_mask;
            count(t_flag, vv, __ballot(flag) & in_mask);
            count(t_bT, vv, changed & __ballot(mag <= 3.4028234e38f) & __ballot(fabsf(mag - T) <= band));
            // deviating after correction, less those deviating before
            const uint64_t post = __ballot(!(dpost <= tau)) & in_mask;
            constexpr int lo = 8 * (v >> 2) + (v & 3);
            set_lane<lo>(t_corr, __builtin_popcount((uint32_t)post) - __builtin_popcount((uint32_t)pre));
            set_lane<lo + 4>(t_corr, __builtin_popcount((uint32_t)(post >> 32)) - __builtin_popcount((uint32_t)(pre >> 32)));
          }
          count(t_bit, vv, changed);
          count(t_pre, vv, pre);
          count(t_btau, vv, changed & __ballot(tau > 0.0f) & __ballot(dpre >= 0.5f * tau) & __ballot(dpre <= 2.0f * tau));
          mxp[v] = fmaxf(mxp[v], in ? dpre : 0.0f);
          mxq[v] = fmaxf(mxq[v], in ? dpost : 0.0f);
        });
        n_flag += t_flag; n_bit += t_bit; n_pre += t_pre; n_corr += t_corr; n_bT += t_bT; n_btau += t_btau;
      } else {
        const uint32_t xb = (uint32_t)(xw + 32 * i + 4 * lhi);   // + 8*q + e
#pragma unroll
        for (int v = 0; v < 16; ++v) golden(xb + 8 * (v >> 2) + (v & 3), row_mine, cs[v], sa[v]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 x4 = *reinterpret_cast<const f32x4*>(p.kra + xb + 8 * q);   // zero padded to a multiple of 512
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float T = p.bound_global ? p.t_global : __fmul_rn(__fmul_rn(x4[e], g_factor), p.gamma);
            dev.account(act && xb + 8 * q + e < (uint32_t)X, t[4 * q + e], T, cs[4 * q + e], sa[4 * q + e], p.policy);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    });
  }
  uint32_t n[6];
  float mp, mq;
  if constexpr (ISA) {
    n[0] = n_flag; n[1] = n_bit; n[2] = n_pre; n[3] = n_pre + n_corr; n[4] = n_bT; n[5] = n_btau;
    // Maxima: through this wave's part of the staging LDS (its last tile has been read), rows of 64
    // lanes padded by 16 bytes; lane t < 32 collects the 32 lanes that hold trial t's register.
    constexpr int ROWB = 64 * 4 + 16;
    static_assert(4 * 2 * 16 * ROWB <= 2 * STAGE, "the maxima of four waves fit the staging LDS");
    uint8_t* const scr = smem + wave * (2 * 16 * ROWB);
    static_for<16>([&](auto vv) {
      constexpr int v = vv;
      *reinterpret_cast<float*>(scr + v * ROWB + lane * 4) = mxp[v];
      *reinterpret_cast<float*>(scr + (16 + v) * ROWB + lane * 4) = mxq[v];
    });
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int v_mine = 4 * (l32 >> 3) + (l32 & 3), h_mine = (l32 >> 2) & 1;
    // lanes 0 .. 31 the maxima before, lanes 32 .. 63 those after correction
    const uint8_t* const at = scr + (16 * lhi + v_mine) * ROWB + h_mine * 128;
    float m = 0.0f;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const f32x4 w = *reinterpret_cast<const f32x4*>(at + u * 16);
      m = fmaxf(fmaxf(fmaxf(m, w[0]), fmaxf(w[1], w[2])), w[3]);
    }
    mp = m;
    mq = __shfl_xor(m, 32, 64);
  } else {
    // the two half-waves hold the same trials
    n[0] = dev.n_flag; n[1] = dev.n_bit; n[2] = dev.n_pre; n[3] = dev.n_post; n[4] = dev.n_bT; n[5] = dev.n_btau;
#pragma unroll
    for (int q = 0; q < 6; ++q) n[q] += __shfl_xor(n[q], 32, 64);
    mp = fmaxf(dev.mx_pre, __shfl_xor(dev.mx_pre, 32, 64));
    mq = fmaxf(dev.mx_post, __shfl_xor(dev.mx_post, 32, 64));
  }
  // One record update per item and trial: the waves of the other rows of X hand theirs over in LDS.
  // The updates leave the XCD (its L2 is not the point of coherence), so their number counts: six
  // 32-bit ones by every wave took 19 of 53 us on 2048 A faults x 3072 columns.
  constexpr int XCH = 40 * 1024;                          // behind the maxima
  static_assert(XCH + 2 * 8 * 32 * 4 <= 2 * STAGE && 4 * 2 * 16 * (64 * 4 + 16) <= XCH, "exchange inside the staging LDS");
  uint32_t* const xch = reinterpret_cast<uint32_t*>(smem + XCH) + wt * 256 + l32;
  if (wx == 1 && lhi == 0) {
#pragma unroll
    for (int q = 0; q < 6; ++q) xch[q * 32] = n[q];
    xch[6 * 32] = __float_as_uint(mp);
    xch[7 * 32] = __float_as_uint(mq);
  }
  __syncthreads();
  if (wx == 0 && act && lhi == 0) {
#pragma unroll
    for (int q = 0; q < 6; ++q) n[q] += xch[q * 32];
    // non-negative floats (and +Inf) order like their words
    const uint32_t wp = max(__float_as_uint(mp), xch[6 * 32]), wq = max(__float_as_uint(mq), xch[7 * 32]);
    fi_trial_result* r = p.results + list.trial[q_mine];
    if (parts != nullptr) {
      u32x4* const to = reinterpret_cast<u32x4*>(parts + ((size_t)x_slot * p.n_trials + list.trial[q_mine]) * kPartWords);
      to[0] = u32x4{n[0], n[1], n[2], n[3]};
      to[1] = u32x4{n[4], n[5], wp, wq};
      return;
    }
    if ((reinterpret_cast<uintptr_t>(p.results) & 7u) == 0) {
      // neighbouring counters in one 64-bit addition: no sum reaches 2^32
      auto add2 = [](uint32_t* at, uint32_t lo, uint32_t hi) __attribute__((always_inline)) {
        if (lo | hi) atomicAdd(reinterpret_cast<unsigned long long*>(at), (unsigned long long)hi << 32 | lo);
      };
      static_assert(offsetof(fi_trial_result, n_bitdiff) == 4 && offsetof(fi_trial_result, n_dev_pre) == 8 &&
                    offsetof(fi_trial_result, n_dev_post) == 12 && offsetof(fi_trial_result, n_border_T) == 32 &&
                    offsetof(fi_trial_result, n_border_tau) == 36 && sizeof(fi_trial_result) == 48, "pairs of counters");
      add2(&r->n_flagged, n[0], n[1]);
      add2(&r->n_dev_pre, n[2], n[3]);
      add2(&r->n_border_T, n[4], n[5]);
    } else {
      if (n[0]) atomicAdd(&r->n_flagged, n[0]);
      if (n[1]) atomicAdd(&r->n_bitdiff, n[1]);
      if (n[2]) atomicAdd(&r->n_dev_pre, n[2]);
      if (n[3]) atomicAdd(&r->n_dev_post, n[3]);
      if (n[4]) atomicAdd(&r->n_border_T, n[4]);
      if (n[5]) atomicAdd(&r->n_border_tau, n[5]);
    }
    if (wp) atomicMax(reinterpret_cast<uint32_t*>(&r->max_dev_pre), wp);
    if (wq) atomicMax(reinterpret_cast<uint32_t*>(&r->max_dev_post), wq);
  }
}

template <int DT, bool BIG>
__global__ void __launch_bounds__(256, 3) affected_rows_kernel(const GemmArgs p, int n_x_slots, int plain_holds, uint32_t* parts) {
  constexpr int BT = kRowsTrials;
  __shared__ __attribute__((aligned(16))) uint8_t smem[kRowsBuf * (kRowsTrials + kRowsX) * 128];
  __shared__ uint32_t cnt[2][8];
  __shared__ __attribute__((aligned(16))) RowsLists list;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int x_slot = (int)(blockIdx.x % (uint32_t)n_x_slots);
  const uint32_t item = blockIdx.x / (uint32_t)n_x_slots;
  // The first items of all chunks come first: the workgroups that find none start last and do not
  // hold up those that do (39 -> 37 us on the 4096 trials above, five ninths of whose items are empty).
  const uint32_t n_chunks = ((uint32_t)p.n_trials + kRowsChunk - 1) / kRowsChunk;
  const uint32_t sub = item / n_chunks, chunk0 = item % n_chunks * kRowsChunk;

  // ---- which trials: ranks of the chunk's A faults and of its B faults, in list order
  fi_fault f[2];
  int kind[2];
  unsigned long long mask[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t t = chunk0 + (uint32_t)(h * 256 + tid);
    f[h] = p.faults[t < (uint32_t)p.n_trials ? t : 0u];
    kind[h] = t < (uint32_t)p.n_trials ? affected_kind(f[h], p) : 0;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      mask[h][b] = __ballot(kind[h] == 2 + b);
      if (lane == 0) cnt[b][h * 4 + wave] = (uint32_t)__builtin_popcountll(mask[h][b]);
    }
  }
  if (tid < BT) { list.trial[tid] = 0; list.row[tid] = 0; list.k[tid] = 0xFFFFFFFFu; list.mask[tid] = 0; }
  __syncthreads();
  uint32_t n_kind[2] = {0, 0};
  uint32_t first[2][2] = {{0, 0}, {0, 0}};                // [h][b]: rank of this wave's first trial
#pragma unroll
  for (int w = 0; w < 8; ++w) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (w == wave) first[0][b] = n_kind[b];
      if (w == 4 + wave) first[1][b] = n_kind[b];
      n_kind[b] += cnt[b][w];
    }
  }
  const uint32_t items_a = (n_kind[0] + BT - 1) / BT, items_b = (n_kind[1] + BT - 1) / BT;
  if (sub >= items_a + items_b) return;                   // uniform
  const bool isA = sub < items_a;
  const uint32_t rank0 = (isA ? sub : sub - items_a) * BT;
  const int n_act = __builtin_amdgcn_readfirstlane((int)min((uint32_t)BT, (isA ? n_kind[0] : n_kind[1]) - rank0));
  if (x_slot * kRowsX >= (isA ? p.N : p.M)) return;       // uniform
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (kind[h] == (isA ? 2 : 3)) {
      const unsigned long long m = isA ? mask[h][0] : mask[h][1];
      const uint32_t rank = (isA ? first[h][0] : first[h][1]) + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull));
      if (rank >= rank0 && rank < rank0 + BT) {
        const uint32_t q = rank - rank0;
        list.trial[q] = chunk0 + (uint32_t)(h * 256 + tid);
        list.row[q] = isA ? f[h].row : f[h].col;
        list.k[q] = isA ? f[h].col : f[h].row;
        list.mask[q] = f[h].xor_mask & 0xFFFFu;
      }
    }
  }
  __syncthreads();
  if (isA) affected_rows_item<DT, BIG, true>(p, smem, list, n_act, x_slot, n_x_slots, plain_holds != 0, parts);
  else affected_rows_item<DT, BIG, false>(p, smem, list, n_act, x_slot, n_x_slots, false, parts);
}

}  // namespace fi
