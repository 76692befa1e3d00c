// Drafter evaluation with one read of every logit, in one launch: softmax statistics,
// alpha = sum_v min(p, q_i) for every drafter (Theorem 1), greedy argmax and agreement, and
// for hs_round the learner step.
//
// min(p_v, q_v) needs both rows' normalisers, which depend on the whole row, so the
// slices of a row have to meet before any min can be taken. Here they meet on chip: a
// work item is (row set, slice) = the target slice and the slices of up to D drafters of
// one (query, position) group, 256 16-byte vectors each, held in the registers of one
// 256-thread workgroup (thread t owns vector t of every row). The S items of a row set form
// a team that is resident at the same time:
//   1. every item takes its rows' exp2 sums (z c, c = log2(e) / T, less an integer-valued offset:
//      the thread's own, at or above its largest z c, or one common to the call) and, where
//      asked for, maxima and lowest argmaxes, and publishes them as tagged words, the offsets
//      beside the sums;
//   2. item s folds the S slice statistics of row s (rows s, s + S, ... when S is smaller
//      than the row count) into the row's log2 normaliser L = hi + lo and publishes it (sums
//      against different offsets rescale by powers of two, so exactly);
//   3. every item reads the normalisers and forms its slice's part of sum_v min(p_v, q_v)
//      for each drafter: from the e_v kept in registers when the workgroup holds one item
//      (one multiply, one min and one add per drafter logit), else from the logits again
//      (one fma, one min, one exp2 and one add); the partials are published;
//   4. slot d mod S sums drafter d's S slice partials in slice order into alpha.
// Within a workgroup every reduction over the slice goes through LDS: each thread stores its
// per-row value, then one 16-lane group per row reduces the row's 256 values and the result
// is known to the whole group, so no wave reduces all rows on its own.
// A workgroup with several items overlaps them: while item j's normalisers are exchanged it
// runs the statistics of item j + 1, and the loads of item j + 2 go out as soon as item j's
// min-sums have freed its registers.
//
// The grid holds as many teams as the device keeps resident at once, so all members of a
// team run together and waiting on one cannot deadlock. Words crossing workgroups carry the
// call's tag; the last team to finish advances the epoch the tag derives from. Every wait is
// bounded: a word that never arrives yields NaN (argmax -2), no hang, and everything computed
// from it carries a taint mark, so the learner step of such a round leaves the learner state
// unchanged.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>

#include "hs_exchange.h"
#include "hs_learner.h"

namespace hs {

constexpr int kCritPrio = 2;   // wave priority of the exchange-critical stages (s_setprio)
constexpr int kFoldPrio = 3;   // and of the pipelined kernel's row folds, which gate the team
// The wave that holds no row of the group reductions (16-lane group r reduces row r, so the at
// most kMaxSetDrafters + 1 rows sit in the other waves) takes a member's first fold duty and
// the normaliser wait: their load round trips then overlap the other waves' group reductions
// instead of following them, and wave 0 keeps thread 0's claims and counts.
constexpr int kDutyWave = kWaves - 1;
static_assert(kMaxSetDrafters + 1 <= 4 * kDutyWave, "the duty wave must hold no reduction row");

struct TeamArgs {
  // What every workgroup reads before its first loads comes first: the first 128 bytes of the
  // kernel arguments, two scalar-cache lines, requested together at entry. The row table
  // follows at the end.
  int B, N, K, nsub, S, items;
  int teams;         // workgroups of the launch / S
  // drafter rows at one constant distance (uni != 0): row bases from these scalars instead of
  // the row table, so the kernel does not wait for the table at its start
  int uni;
  FastDiv divS, divK;  // by S and K
  int64_t V;
  int64_t dd;          // bytes from drafter i's row (b, k) to drafter i + 1's
  const void* base0;   // the target's rows (rows.ptr[0] and its strides)
  const void* base1;   // drafter 0's rows (rows.ptr[1] and its strides)
  int64_t sb0, sk0, sb1, sk1;
  uint32_t* epoch;     // advanced by the last workgroup to finish
  // ---- 128 bytes ----
  int64_t nvec;
  float c;
  float o;             // integer-valued common offset of the pipelined kernel's sums (launch_round)
  FastDiv divNsub;     // by nsub
  uint64_t* fail;      // set, with the call's tag, by the first wait that gives up
  uint32_t polls;      // polls before a wait gives up (0: every wait gives up at once)
  uint32_t* next_set;  // row sets claimed beyond each team's fixed ones
  uint64_t* finished;  // teams of this launch that have finished (a tagged count)
  uint64_t* mbox;      // [teams][4]: the row set of each team's coming items
  uint64_t* stat;  // [sets][D + 1][3][S]
  uint64_t* norm;  // [sets][D + 1][3] (the single-item kernel's other copies: norm_copy)
  uint64_t* part;  // [G][N][S]
  float* alpha;
  int32_t* argmax_t;
  int32_t* argmax_d;
  uint8_t* agree;
  // learner step in the same launch (learn != 0; alpha kernels only): gamma words gw [B][N][K]
  // are written by the folders (gamma = alpha when learn == 1, agreement when learn == 2), and
  // workgroup b (mod the grid) runs query b's step once it has finished its own items
  int learn;
  uint64_t* gw;
  TailArgs tail;
  RowTable rows;
};


// Mailbox word of a team's item j: the row set in bits 38..63, j mod 64 in bits 32..37, the
// call's tag below, so neither an earlier item's word in the same ring slot nor an earlier
// call's word is taken for it.
__device__ inline uint64_t mbox_word(uint32_t set, int j, uint32_t tag) {
  return ((uint64_t)((set << 6) | ((uint32_t)j & 63u)) << 32) | tag;
}
// The row set posted for item j (bounded as await_word: `none` after a time-out, raising the
// fail flag).
__device__ inline uint32_t await_mbox(const uint64_t* w, int j, uint32_t tag, const TeamArgs& A,
                                      uint32_t none) {
  auto ok = [&](uint64_t v) {
    return (uint32_t)v == tag && ((uint32_t)(v >> 32) & 63u) == ((uint32_t)j & 63u);
  };
  if (A.polls == 0) {
    put_word(A.fail, word_of(1, tag));
    return none;
  }
  uint64_t v = get_word(w);
  for (uint32_t n = 1; !ok(v); ++n) {
    if (n >= A.polls || ((n & 255) == 0 && (uint32_t)get_word(A.fail) == tag)) {
      put_word(A.fail, word_of(1, tag));
      return none;
    }
    __builtin_amdgcn_s_sleep(kPollSleep);
    v = get_word(w);
  }
  return (uint32_t)(v >> 38);
}

// Copy c of the normaliser words: the first at A.norm, the others after the gamma words (the
// single-item kernel only, whose row sets are its teams).
__device__ inline uint64_t* norm_copy(const TeamArgs& A, int c, int rows) {
  if (c == 0) return A.norm;
  const uintptr_t end = reinterpret_cast<uintptr_t>(A.gw + (int64_t)A.B * A.N * A.K);
  return reinterpret_cast<uint64_t*>((end + 255) & ~(uintptr_t)255) +
         (c - 1) * norm_copy_words(A.teams, rows);
}

// A thread's offset for the exp2 sum of its logits of a row, m the largest of them: integer-valued
// and at or above m c (exp_offset_of), so that sums against different offsets rescale exactly and
// no exponent is positive. Held to [-2^29, 2^29], where differences of offsets fit an int32: beyond
// it (logits far outside the range of |z c| <= 2^28) terms are 0 at the lower end and a sum
// infinite at the upper, and without a logit whose scaled value is finite (m c = -inf: the fma
// then gives NaN, as for a NaN m, and fmaxf the lower end) every term is 0, or NaN for a NaN logit.
constexpr int kNoOffset = -(1 << 29);
__device__ inline float thread_offset(float m, float c) {
  const float mc = m * c;
  return fminf(fmaxf(ceilf(fmaf(fabsf(mc), 0x1p-22f, mc)), (float)kNoOffset), 0x1p29f);
}

// A thread's sum against its own offset has its exponents near 0 where they matter, so they are
// rounded least, and nothing waits for a maximum. But maxima, offsets and rescaling are a seventh of
// the pipelined kernel's instructions, which bound it. Against one common offset A.o they fall away
// as long as every sum stays within fp32's range, with room (OWN = false below, without an argmax):
// 16 queries x 64 drafters x 8 positions x 151936 bf16 logits 657 us, with own offsets 694; 64 x 8 x
// 6 x 128256 216 and 222.
// A wave in which a row's sums leave [2^-56, 2^96] (logits far from 0, masked or NaN) decides for
// each row of the item by its threads' largest logits: A.o if all are in_common_range, else every
// thread's own offset, the sums then marked by their sign bits; and it goes on so, without trying
// A.o first, until an item needs it no more. A wave whose sums passed the test would decide for A.o
// as well, so a result does not depend on what the wave did before. Where every wave decides so the
// large calls take 11% longer than with own offsets throughout (the same two at logits 60 lower:
// 775 and 695 us, 249 and 222); launch_t says which kernel a call takes.
constexpr float kCommonLo = 0x1p-56f, kCommonHi = 0x1p96f;
constexpr uint32_t kOwn = 0x80000000u;  // mark of a sum against its own offset
// Largest logit m of up to 8 with a sum against `common` surely within [2^-60, 2^100]: m c - common
// within [-60, 97].
__device__ inline bool in_common_range(float m, float c, float common) {
  return fabsf(fmaf(m, c, -(common + 18.5f))) <= 78.5f;
}

// Words of a row of a row set: S slice offsets (with an argmax: S slice maxima, from which the
// offsets follow; with a common offset: those of marked sums only), S exp2 sums, S argmaxes. Each kind is contiguous, so that a fold's lanes read
// whole lines.
__device__ inline uint64_t* stat_row(const TeamArgs& A, int set, int r, int RM) {
  return A.stat + ((int64_t)set * RM + r) * A.S * 3;
}

// Log2 normaliser o + log2(sum) of row rr, o integer-valued, as an unevaluated sum hi + lo; lane c
// writes copy c. The sum's exponent is taken apart (exactly, also
// from a large o): the logarithm then lies in [-1, 0), where its error is smallest.
template <int D, int NC>
__device__ __forceinline__ void publish_norm(const TeamArgs& A, int set, int rr, float o,
                                             float sum, uint32_t tt, int lane) {
  auto two_sum = [](float a, float b, float& err) {
    const float s = a + b, bb = s - a;
    err = (a - (s - bb)) + (b - bb);
    return s;
  };
  float e0, e1;
  const float n = two_sum(o, (float)__builtin_amdgcn_frexp_expf(sum), e0);
  const float hi = two_sum(n, log2f(__builtin_amdgcn_frexp_mantf(sum)), e1);
  const float lo = e0 + e1;
  if (lane < NC) {
    uint64_t* cw = norm_copy(A, lane, D + 1) + ((int64_t)set * (D + 1) + rr) * 3;
    put_word(cw, word_of(hi, tt));
    put_word(cw + 1, word_of(lo, tt));
  }
}

// Publishes the argmax idx of row rr of row set `set` (tt: tag and taint) and writes the argmax and
// agreement outputs (one lane).
template <int D>
__device__ __forceinline__ void put_argmax(const TeamArgs& A, int set, int rr, int b, int k, int sub,
                                           int idx, uint32_t tag, uint32_t tt) {
  uint64_t* norms = A.norm + (int64_t)set * (D + 1) * 3;
  put_word(norms + 3 * rr + 2, word_of(idx, tt));
  if (rr == 0) {
    if (sub == 0 && A.argmax_t) A.argmax_t[(int64_t)b * A.K + k] = idx;
    return;
  }
  const int64_t oi = ((int64_t)b * A.N + sub * D + rr - 1) * A.K + k;
  if (A.argmax_d) A.argmax_d[oi] = idx;
  if (A.agree) {
    const uint64_t tw = await_word(norms + 2, tag, A);
    const int it = word_i(tw);
    const bool ag = idx == it && it >= 0;
    A.agree[oi] = (uint8_t)ag;
    if (A.learn == 2) put_word(A.gw + oi, word_of(ag ? 1.0f : 0.0f, tt | ((uint32_t)tw & kTaint)));
  }
}

// Fold of row rr of row set `set`: the S slice statistics, two slices per lane per pass
// (lane j takes slices j, j + 64, ... in order), then the wave. Publishes the row's log2
// normaliser as hi + lo (in NC copies) and its argmax; writes the argmax and agreement
// outputs. The published words are tainted when any slice word was lost. OWN: every slice's sum is
// against an offset of its own, else marked ones are.
template <int D, bool NEED_ARG, bool OWN, int NC = 1>
__device__ __forceinline__ void fold_row(const TeamArgs& A, int set, int rr, int b, int k, int sub,
                                uint32_t tag, int lane) {
  constexpr int RM = D + 1;
  const int S = A.S;
  const uint64_t* base = stat_row(A, set, rr, RM);
  float m = -INFINITY, sum = 0.0f;
  int idx = INT_MAX, o = kNoOffset;
  bool lost = false;
  uint32_t marks = 0;
  float plain = 0.0f;  // sum of the sums against A.o
  for (int j0 = 0; j0 < S; j0 += 128) {
    uint64_t w[2][3];
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // issue every load of the pass before waiting on any
      const int j = j0 + lane + 64 * h;
      if (j < S) {
        if (OWN) w[h][0] = get_word(base + j);
        w[h][1] = get_word(base + S + j);
        if (NEED_ARG) w[h][2] = get_word(base + 2 * S + j);
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = j0 + lane + 64 * h;
      if (j < S) {
        if (OWN) {
          if (tag_of(w[h][0]) != tag) w[h][0] = await_word(base + j, tag, A);
          lost |= tainted(w[h][0]);
        }
        if (NEED_ARG) {
          if (tag_of(w[h][2]) != tag) w[h][2] = await_word(base + 2 * S + j, tag, A);
          lost |= tainted(w[h][2]);
          argmax_combine(m, idx, word_f(w[h][0]), word_i(w[h][2]));
        }
        if (tag_of(w[h][1]) != tag) w[h][1] = await_word(base + S + j, tag, A);
        lost |= tainted(w[h][1]);
        if (!OWN && ((uint32_t)(w[h][1] >> 32) & kOwn) == 0) {
          plain += word_f(w[h][1]);
        } else {
          if (!OWN) {
            marks = kOwn;
            w[h][0] = await_word(base + j, tag, A);
            lost |= tainted(w[h][0]);
          }
          const int oj = NEED_ARG ? (int)thread_offset(word_f(w[h][0]), A.c) : word_i(w[h][0]);
          const int on = max(o, oj);
          sum = ldexpf(sum, o - on) + ldexpf(fabsf(word_f(w[h][1])), oj - on);
          o = on;
        }
      }
    }
  }
  if (NEED_ARG) wave_max<true>(m, idx);
  float ro = A.o;
  if (OWN || __ballot(marks != 0) != 0) {
    const int op = plain != 0.0f ? (int)A.o : kNoOffset;
    const int on = wave_max_i(OWN ? o : max(o, op));
    sum = ldexpf(sum, o - on);
    if (!OWN) sum += ldexpf(plain, op - on);
    ro = (float)on;
  } else {
    sum = plain;
  }
  sum = wave_sum_f(sum);
  const uint32_t tt = tag | taint_bits(__ballot(lost) != 0);
  publish_norm<D, NC>(A, set, rr, ro, sum, tt, lane);
  if (NEED_ARG && lane == 0) put_argmax<D>(A, set, rr, b, k, sub, idx, tag, tt);
}

// The argmax-only kernel's fold of row rr of row set `set`: a slice's two words side by side.
template <int D>
__device__ __forceinline__ void fold_row_argmax(const TeamArgs& A, int set, int rr, int b, int k,
                                                int sub, uint32_t tag, int lane) {
  const int S = A.S;
  const uint64_t* base = stat_row(A, set, rr, D + 1);
  float m = -INFINITY;
  int idx = INT_MAX;
  bool lost = false;
  for (int j0 = 0; j0 < S; j0 += 128) {
    uint64_t w[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // issue every load of the pass before waiting on any
      const int j = j0 + lane + 64 * h;
      if (j < S) {
        w[h][0] = get_word(base + 2 * j);
        w[h][1] = get_word(base + 2 * j + 1);
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = j0 + lane + 64 * h;
      if (j < S) {
        if (tag_of(w[h][0]) != tag) w[h][0] = await_word(base + 2 * j, tag, A);
        if (tag_of(w[h][1]) != tag) w[h][1] = await_word(base + 2 * j + 1, tag, A);
        lost |= tainted(w[h][0]) || tainted(w[h][1]);
        argmax_combine(m, idx, word_f(w[h][0]), word_i(w[h][1]));
      }
    }
  }
  wave_max<true>(m, idx);
  const uint32_t tt = tag | taint_bits(__ballot(lost) != 0);
  if (lane == 0) put_argmax<D>(A, set, rr, b, k, sub, idx, tag, tt);
}

// Position of work item (set, slot): row set, slice, group (b, k), drafters n in the set, and
// the calling thread's vector index within the row.
struct ItemPos {
  int set, s, g, sub, b, k, n;
  int vi;  // a row holds fewer than 2^31 logits
};
__device__ inline ItemPos item_pos(const TeamArgs& A, uint32_t set, int slot, int D) {
  ItemPos q;
  q.set = (int)set;
  q.s = slot;
  if (A.nsub == 1) {
    q.g = q.set;
    q.sub = 0;
  } else {
    q.g = (int)fdiv(set, A.divNsub);
    q.sub = q.set - q.g * A.nsub;
  }
  q.b = (int)fdiv((uint32_t)q.g, A.divK);
  q.k = q.g - q.b * A.K;
  q.n = min(D, A.N - q.sub * D);
  q.vi = q.s * kThreads + (int)threadIdx.x;
  return q;
}

// LDS of a team workgroup. Per-thread values of every row are stored transposed, [row][thread],
// so that one 16-lane group reduces one row (group_read) instead of every wave reducing every
// row on its own.
template <int D, bool NEED_ARG, bool SINGLE>
struct TeamLds {
  float xs[D + 1][kThreads];                    // per-thread exp2 sums (SINGLE: later the
                                                // min-sums of the drafters)
  int xo[D + 1][kThreads];                      // the offsets that they are taken against
  float xt[NEED_ARG ? D + 1 : 1][kThreads];     // per-thread maxima
  int xi[NEED_ARG ? D + 1 : 1][kThreads];       // per-thread argmax
  float xp[SINGLE ? 1 : D][kThreads];           // per-thread min-sums of each drafter
  int n[D + 1];     // SINGLE: the rows' rint(hi)
  float G[D];      // SINGLE: 2^(a_t - a_d)
  float no[D + 1];  // minus the offset of the row's exponents (plain form: the target's only)
  float nw[D];     // plain: the exponent addend of drafter d
  float dl[D];     // wide: a_t - a_d
  uint32_t wide;   // the min-sums take the wide form
  float F[D];      // factor of drafter d's group sum, 2^(a_t); SINGLE: 2^(a_d)
  uint32_t next;  // a row set of the team's coming items, posted by thread 0
  uint32_t taint;  // the item's normalisers include a lost word: its partials are tainted
  // the row table, copied from the kernel arguments once (lane-parallel loads instead of a
  // chain of dependent scalar loads per item)
  const char* ptr[kMaxRows];
  int64_t sb[kMaxRows];
  int64_t sk[kMaxRows];
};

// Issue the loads of item q into dst: exactly D + 1 unconditional 16-byte loads, so that the
// number of loads in flight is the same on every path and a later wait for an older item's
// registers can leave these outstanding. Each comes from an address clamped into the row's
// complete vectors (lanes past the row end are masked to -inf before use, mask_tail); rows
// past the set's last drafter, and every row when !valid, read 16 bytes of the workspace's
// control block instead (a cache-resident dummy, never used). The one partial vector at the
// end of a row (V not a multiple of the vector width) is then re-read element by element, in
// a branch taken only by the slice that holds it.
template <int DT, int D, bool UNI = false, typename L>
__device__ __forceinline__ void fetch_item(const TeamArgs& A, const ItemPos& q, bool valid,
                                           const L& sh, typename Vec<DT>::Raw (&dst)[D + 1]) {
  using Vt = Vec<DT>;
  constexpr int E = Vt::kElems;
  const int64_t vfull = A.V / E;  // complete 16-byte vectors per row
  const uint64_t dummy = reinterpret_cast<uint64_t>(A.epoch);
  uint64_t rb[D + 1];
  if (UNI && A.uni) {
    // drafters at a constant distance: uniform scalar arithmetic
    rb[0] = valid ? reinterpret_cast<uint64_t>(A.base0) +
                        (uint64_t)(((int64_t)q.b * A.sb0 + (int64_t)q.k * A.sk0) *
                                   Vt::kBytes)
                  : dummy;
    const uint64_t d0 = reinterpret_cast<uint64_t>(A.base1) +
                        (uint64_t)(((int64_t)q.b * A.sb1 + (int64_t)q.k * A.sk1) *
                                   Vt::kBytes) +
                        (uint64_t)((int64_t)q.sub * D * A.dd);
#pragma unroll
    for (int r = 1; r <= D; ++r)
      rb[r] = valid && r <= q.n ? d0 + (uint64_t)((int64_t)(r - 1) * A.dd) : dummy;
  } else {
    // lane r <= n: the base of row r of the item from the table in LDS, then broadcast
    const int l = threadIdx.x & 63;
    uint64_t base = dummy;
    if (valid && l <= q.n) {
      const int row = l == 0 ? 0 : q.sub * D + l;
      base = reinterpret_cast<uint64_t>(sh.ptr[row]) +
             (uint64_t)(((int64_t)q.b * sh.sb[row] + (int64_t)q.k * sh.sk[row]) * Vt::kBytes);
    }
#pragma unroll
    for (int r = 0; r <= D; ++r) {
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)base, r);
      const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(base >> 32), r);
      rb[r] = ((uint64_t)hi << 32) | lo;
    }
  }
  // uniform row base + 32-bit lane offset (a row holds < 2^31 logits); a global (not flat)
  // 16-byte load. 16-bit rows load nontemporal (every logit is read once; the target slice of
  // a group's later row sets still comes from L2): 1% faster on every bf16 workload measured,
  // but 19% slower on 64 stacked fp32 tiny chains, so fp32 rows load plainly
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  const uint32_t off =
      valid && vfull > 0 ? (uint32_t)((q.vi < vfull ? q.vi : vfull - 1) * 16) : 0u;
#pragma unroll
  for (int r = 0; r <= D; ++r) {
    const uint32_t o = r <= q.n ? off : 0u;
    typedef const __attribute__((address_space(1))) u4* gp4;
    const u4 v = DT != HS_F32 ? __builtin_nontemporal_load((gp4)(rb[r] + o)) : *(gp4)(rb[r] + o);
    __builtin_memcpy(&dst[r], &v, 16);
  }
  if (valid && vfull < A.nvec && (int64_t)(q.s + 1) * kThreads > vfull) {  // the tail slice
#pragma unroll
    for (int r = 0; r <= D; ++r)
      if (r <= q.n && q.vi == vfull)
        dst[r] = Vt::load_raw(reinterpret_cast<const char*>(rb[r]), q.vi, A.V);
  }
}

// -inf for the lanes of the last slice that lie past the row end.
template <int DT, int D>
__device__ __forceinline__ void mask_tail(const TeamArgs& A, const ItemPos& q,
                                          typename Vec<DT>::Raw (&x)[D + 1]) {
  if ((int64_t)(q.s + 1) * kThreads > A.nvec) {
#pragma unroll
    for (int r = 0; r <= D; ++r)
      if (q.vi >= A.nvec) x[r] = Vec<DT>::neg_raw();
  }
}

// min of two values that are >= 0 or +NaN (0 * inf): the unsigned order of the bits is their
// order and a NaN loses, as with fminf, without fminf's canonicalising of the operands.
__device__ inline float min_pos(float a, float b) {
  return __uint_as_float(min(__float_as_uint(a), __float_as_uint(b)));
}

// fminf of two results of arithmetic (never a signalling NaN): the hardware minimum, which
// returns the other operand for a quiet NaN as fminf does. Written out because the compiler
// otherwise re-canonicalises an operand that it cannot prove is a result of arithmetic (the
// target's exponents, once per item).
__device__ inline float min_arith(float a, float b) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Sum of a thread's terms of one row: two interleaved sums, started from the first terms (no
// additions of zero).
template <int E>
__device__ __forceinline__ float sum_elems(const float (&v)[E]) {
  float a0 = v[0], a1 = v[1];
#pragma unroll
  for (int e = 2; e < E; ++e) {
    if (e & 1) a1 += v[e];
    else a0 += v[e];
  }
  return a0 + a1;
}

// 2^(x - lo) of an offset difference x (any magnitude) and a small lo: the integer part of x
// goes to the exponent, so that the fraction keeps its accuracy.
__device__ inline float exp2_split(float x, float lo) {
  if (!(fabsf(x) < 0x1p20f)) return __builtin_amdgcn_exp2f(x - lo);  // 0, infinite or NaN
  const float n = rintf(x);
  return ldexpf(__builtin_amdgcn_exp2f((x - n) - lo), (int)n);
}

// The raw registers of one row made opaque to the compiler: each stage unpacks the logits
// afresh (two integer operations per pair) instead of the compiler keeping the unpacked
// floats of a whole item live from one stage to the next, which would not fit in registers.
template <typename Raw>
__device__ __forceinline__ void launder(Raw& x) {
  static_assert(sizeof(Raw) == 16, "16-byte vectors");
  uint32_t w[4];
  __builtin_memcpy(w, &x, 16);
  asm volatile("" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]));
  __builtin_memcpy(&x, w, 16);
}

// Largest of a thread's logits of one row; NaN when one of them is.
template <int E>
__device__ __forceinline__ float max_or_nan(const float (&z)[E]) {
  float m = maximum3(z[0], z[1], z[2]);
#pragma unroll
  for (int e = 3; e < E; e += 2) m = maximum3(m, z[e], e + 1 < E ? z[e + 1] : z[e]);
  return m;
}

// Max of a thread's logits of one row and its lowest index, to LDS.
template <int E, typename L>
__device__ __forceinline__ float thread_argmax(const TeamArgs& A, const ItemPos& q, int r,
                                               const float (&z)[E], L& sh, int t) {
  float m = -INFINITY;
  int idx = INT_MAX;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    if (z[e] > m) {
      m = z[e];
      idx = q.vi * E + e;
    }
  }
  // a lane whose logits are all -inf still owns its lowest valid index
  if (idx == INT_MAX && q.vi < A.nvec) idx = q.vi * E;
  sh.xt[r][t] = m;
  sh.xi[r][t] = idx;
  return m;
}

// ---- 1. per-thread statistics of every row of item q in one pass, to LDS: the exp2 sum against the
// thread's own offset (KEPT: the e_v stay in x) and, with NEED_ARG, the max and its lowest index.
// An offset per thread needs no pass and no barrier before the sums, and keeps the exponents of
// the terms that matter near 0, where they are rounded least, wherever the logits lie. ----
template <int DT, int D, bool NEED_ARG, bool KEPT, typename L, typename X>
__device__ __forceinline__ void thread_stats(const TeamArgs& A, const ItemPos& q,
                                             typename Vec<DT>::Raw (&raw)[D + 1], X& x, L& sh,
                                             int t) {
  constexpr int E = Vec<DT>::kElems;
#pragma unroll
  for (int r = 0; r <= D; ++r) {
    if (r > q.n) continue;
    launder(raw[r]);
    float z[E];
    Vec<DT>::unpack(raw[r], z);
    float m;
    if (NEED_ARG) m = thread_argmax<E>(A, q, r, z, sh, t);
    else m = max_or_nan(z);
    const float of = thread_offset(m, A.c);
    sh.xo[r][t] = (int)of;
    float v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      v[e] = __builtin_amdgcn_exp2f(fmaf(z[e], A.c, -of));
      if constexpr (KEPT) x[r][e] = v[e];
    }
    sh.xs[r][t] = sum_elems(v);
  }
}

// min and max of three that are NaN when one of them is
__device__ __forceinline__ float minimum3(float a, float b, float c) {
  float r;
  asm("v_minimum3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// The same against the common offset where that fits (own: the wave's last item needed its own
// offsets; updated).
template <int DT, int D, typename L>
__device__ __forceinline__ void thread_stats_common(const TeamArgs& A, const ItemPos& q,
                                             typename Vec<DT>::Raw (&raw)[D + 1], L& sh, int t,
                                             bool& own) {
  constexpr int E = Vec<DT>::kElems;
  const bool past = q.vi >= A.nvec;  // no logit of any row
  if (!own) {
    float lo = 1.0f, hi = 1.0f, prev = 1.0f;
#pragma unroll
    for (int r = 0; r <= D; ++r) {
      if (r > q.n) continue;
      launder(raw[r]);
      float z[E], v[E];
      Vec<DT>::unpack(raw[r], z);
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = __builtin_amdgcn_exp2f(fmaf(z[e], A.c, -A.o));
      const float s = sum_elems(v);
      sh.xs[r][t] = s;
      if (r & 1) {  // two rows at a time
        lo = minimum3(lo, prev, s);
        hi = maximum3(hi, prev, s);
        prev = 1.0f;
      } else {
        prev = s;
      }
    }
    lo = minimum3(lo, prev, prev);
    hi = maximum3(hi, prev, prev);
    own = __ballot(!past && !(lo >= kCommonLo && hi <= kCommonHi)) != 0;
    if (!own) return;
  }
  bool needed = false;
#pragma unroll
  for (int r = 0; r <= D; ++r) {
    if (r > q.n) continue;
    launder(raw[r]);
    float z[E], v[E];
    Vec<DT>::unpack(raw[r], z);
    const float m = max_or_nan(z);
    const bool common = __ballot(!past && !in_common_range(m, A.c, A.o)) == 0;
    needed |= !common;
    const float of = common ? A.o : thread_offset(m, A.c);
    sh.xo[r][t] = (int)of;
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = __builtin_amdgcn_exp2f(fmaf(z[e], A.c, -of));
    sh.xs[r][t] = common ? sum_elems(v) : -fabsf(sum_elems(v));
  }
  own = needed;
}

// ---- 2. row reductions: 16-lane group gi reduces row gi of the LDS rows (groups past the last
// row reduce a copy of it: all 16 lanes of a group must take part in the DPP steps). Waves whose
// groups hold no row skip them. ----
template <typename L>
__device__ __forceinline__ void group_argmax(const L& sh, int n, int gi, int gl, float& m,
                                             int& idx) {
  const int r = min(gi, n);
  float v[16];
  int iv[16];
  group_read(&sh.xt[r][0], gl, v);
  group_read(&sh.xi[r][0], gl, iv);
  m = v[0];
  idx = iv[0];
#pragma unroll
  for (int u = 1; u < 16; ++u) argmax_combine(m, idx, v[u], iv[u]);
  row16_argmax(m, idx);
}
// Slot s's duty index for an item whose duties start at slot rot: duties are numbered from
// rot on, so that the row and alpha folds move round the team from item to item instead of
// falling on the same few members every time (the team goes at its slowest member's pace).
__device__ inline int duty_index(int s, int rot, int S) { return s >= rot ? s - rot : s - rot + S; }

// Reduces and publishes the slice statistics of item q as tagged words: the slice's sum is taken
// against the largest of its threads' offsets and published beside it, the offset before the sum
// (a fold that finds a marked sum then finds its offset on the way).
template <bool NEED_ARG, typename L>
__device__ __forceinline__ void publish_stats(const TeamArgs& A, const ItemPos& q, uint32_t tag,
                                              int RM, L& sh, int gi, int gl) {
  float m = 0.0f;
  int idx = 0;
  if (NEED_ARG) group_argmax(sh, q.n, gi, gl, m, idx);
  const int r = min(gi, q.n);
  int ov[16];
  group_read(&sh.xo[r][0], gl, ov);
  int o = ov[0];
#pragma unroll
  for (int u = 1; u < 16; ++u) o = max(o, ov[u]);
  o = row16_max(o);
  float v[16];
  group_read(&sh.xs[r][0], gl, v);
#pragma unroll
  for (int u = 0; u < 16; ++u) v[u] = ldexpf(v[u], ov[u] - o);  // exact, or to the denormals
  const float s = row16_sum(sum16(v));
  if (gl != 0 || gi > q.n) return;
  uint64_t* wp = stat_row(A, q.set, gi, RM) + q.s;
  put_word(wp, NEED_ARG ? word_of(m, tag) : word_of(o, tag));
  put_word(wp + A.S, word_of(s, tag));
  if (NEED_ARG) put_word(wp + 2 * A.S, word_of(idx, tag));
}

// The same where waves are against the common offset (without an argmax).
template <typename L>
__device__ __forceinline__ void publish_stats_common(const TeamArgs& A, const ItemPos& q,
                                                     uint32_t tag, int RM, L& sh, int gi, int gl) {
  const int r = min(gi, q.n);
  typedef float F4 __attribute__((ext_vector_type(4)));
  typedef int I4 __attribute__((ext_vector_type(4)));
  // this lane's values of wave i: sums and offsets (group_read's order)
  auto sums = [&](int i) { return *reinterpret_cast<const F4*>(&sh.xs[r][64 * i + 4 * gl]); };
  auto offsets = [&](int i) { return *reinterpret_cast<const I4*>(&sh.xo[r][64 * i + 4 * gl]); };
  auto marked = [&](float x) { return (__float_as_uint(x) & kOwn) != 0; };
  int o = kNoOffset;
  uint32_t mark = 0;
  float c[4], first[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const F4 x = sums(i);
    first[i] = x[0];  // the marks of a wave's sums of a row are alike
    c[i] = (x[0] + x[1]) + (x[2] + x[3]);
  }
  if (__ballot(marked(first[0]) || marked(first[1]) || marked(first[2]) || marked(first[3])) != 0) {
    // (some row of this wave's.) Offset of an unmarked sum: A.o (the one in LDS is an earlier
    // item's); it is 0 only past the row's end
    auto offset = [&](const F4& x, const I4& y, int k) {
      if (marked(x[0])) return y[k];
      return (x[0] + x[1]) + (x[2] + x[3]) == 0.0f ? kNoOffset : (int)A.o;
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const F4 x = sums(i);
      const I4 y = offsets(i);
#pragma unroll
      for (int k = 0; k < 4; ++k) o = max(o, offset(x, y, k));
    }
    o = row16_max(o);
    mark = o != (int)A.o ? kOwn : 0u;
    asm volatile("" ::: "memory");  // read again rather than hold 32 registers
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const F4 x = sums(i);
      const I4 y = offsets(i);
      float e[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) e[k] = ldexpf(fabsf(x[k]), offset(x, y, k) - o);  // exact, or far below
      c[i] = (e[0] + e[1]) + (e[2] + e[3]);
    }
  }
  const float s = row16_sum((c[0] + c[1]) + (c[2] + c[3]));
  if (gl != 0 || gi > q.n) return;
  uint64_t* wp = stat_row(A, q.set, gi, RM) + q.s;
  if (mark) put_word(wp, word_of(o, tag));
  put_word(wp + A.S, word_of(__uint_as_float((__float_as_uint(s) & ~kOwn) | mark), tag));
}

// ---- 4. fold duty: rows i, i + S, ... of the row set (i = the slot's duty index for the
// item's rotation rot), spread over the waves, wave `first` taking the first ----
template <int D, bool NEED_ARG, bool OWN, int NC = 1>
__device__ __forceinline__ void fold_item(const TeamArgs& A, const ItemPos& q, uint32_t tag,
                                          int lane, int wv, int first, int rot = 0) {
  const int order = (wv + kWaves - first) % kWaves;
  for (int rr = duty_index(q.s, rot, A.S) + order * A.S; rr <= q.n; rr += kWaves * A.S)
    fold_row<D, NEED_ARG, OWN, NC>(A, q.set, rr, q.b, q.k, q.sub, tag, lane);
}

// ---- 5. normalisers L = hi + lo (the duty wave; a barrier follows): lanes 2r and 2r + 1 wait for
// row r's hi and lo; lane 2r forms a_r = (o_r - hi_r) - lo_r, o_r an integer-valued offset for the
// row's exponents, and for a drafter row the constants of its min-sum to LDS. A row with no finite
// logit folds to hi = -inf, lo = NaN, so its a is NaN: it has no distribution, and F is NaN whenever
// a_t or a_d is, which makes that drafter's alpha NaN in every form. Differences of the a_r are
// taken part by part, so that they lose nothing to a large hi.
// KEPT (6'): o_r = rint(hi_r); G = 2^(a_t - a_d) and F = 2^(a_d).
// Else (6), plain form: one o for all rows, half the target's normaliser. An exponent of a term that
// matters is then about as far from 0 as the addend nw = -o - (a_t - a_d) that holds o and the
// difference in one float, and both are rounded alike, at 2^-24 of half of |hi|. (Rows more than 32
// apart: the whole of it, which leaves |nw| = |hi_d|.) Where either is large (|hi_t| > 128,
// |nw| > 64: 2^-19 of a term) the wide form: o_r = rint(hi_r), and the difference is subtracted
// in an operation of its own. F = 2^(a_t). ----
template <int D, bool KEPT, typename L>
__device__ __forceinline__ void await_norms(const TeamArgs& A, const ItemPos& q, uint32_t tag,
                                            L& sh, int lane) {
  float h = 0.0f;
  bool lost = false;
  if (lane < 2 * (q.n + 1)) {
    constexpr int NC = KEPT ? kNormCopies : 1;  // the single-item kernel's fold writes copies
    const uint64_t w =
        await_word(norm_copy(A, q.s & (NC - 1), D + 1) +
                       ((int64_t)q.set * (D + 1) + (lane >> 1)) * 3 + (lane & 1),
                   tag, A);
    h = word_f(w);
    lost = tainted(w);
  }
  const bool any_lost = __ballot(lost) != 0;
  if (lane == 0) sh.taint = taint_bits(any_lost);
  const float lo = dpp_f<0xB1>(h);  // lane 2r: the lo of row r, from lane 2r + 1
  const bool row = !(lane & 1) && lane < 2 * (q.n + 1), drafter = row && lane >= 2;
  const int d = (lane >> 1) - 1;
  const float ht = lane_f(h, 0), lot = lane_f(lo, 0);
  const bool undefined = ht + lot != ht + lot || h + lo != h + lo;
  const bool apart = !KEPT && __ballot(drafter && fabsf(h - ht) > 32.0f) != 0;
  float o = KEPT ? rintf(h) : rintf(apart ? ht : 0.5f * ht);
  // a_t - a_d for this lane's o
  auto diff = [&]() {
    const float x = o - h;
    return (lane_f(x, 0) - x) - (lot - lo);
  };
  float df = diff();
  if (!KEPT) {
    const float nw = ((ht - o) - h) + (lot - lo);  // -o - df, without df's rounding where rows lie far apart
    const bool wide =
        __ballot((drafter && !undefined && fabsf(nw) > 64.0f) || (lane == 0 && fabsf(ht) > 128.0f)) != 0;
    if (lane == 0) sh.wide = wide;
    if (wide) {
      o = rintf(h);
      df = diff();
    }
    if (drafter) {
      sh.nw[d] = nw;
      sh.dl[d] = df;
    }
    if (row) sh.no[lane >> 1] = fabsf(o) < INFINITY ? -o : 0.0f;
    const float f = exp2_split(lane_f(o, 0) - ht, lot);
    if (drafter) sh.F[d] = undefined ? NAN : f;
  } else {
    if (row) sh.n[lane >> 1] = cvt_i32_sat(o);
    if (drafter) {
      sh.G[d] = __builtin_amdgcn_exp2f(df);
      sh.F[d] = undefined ? NAN : __builtin_amdgcn_exp2f((o - h) - lo);
    }
  }
}

// ---- 6'. per-thread min-sums from kept e_v: with b_r the thread's offset of row r less the
// integer part n_r of the row's normaliser, p_v = e_t,v 2^(b_t + a_t), q_v = e_d,v 2^(b_d + a_d), so
// min(p_v, q_v) = F 2^(b_d) min(e_t,v G 2^(b_t - b_d), e_d,v); one multiply, one min and one add per
// drafter logit. The offset is that of the thread's largest logit, so 2^(b_r) is about the largest
// probability the thread holds: where the factor of e_t overflows, q's share is below 2^-126, and
// where it underflows p's is. A thread without a finite logit of a row has 2^(b_r) = 0. ----
template <int DT, int D, typename L>
__device__ __forceinline__ void thread_minsums_kept(const ItemPos& q,
                                                    const float (&x)[D + 1][Vec<DT>::kElems],
                                                    L& sh, int t) {
  constexpr int E = Vec<DT>::kElems;
  // (n_r saturates for a row without a distribution, whose F is NaN)
  auto less = [](int a, int b) { return (int)((uint32_t)a - (uint32_t)b); };
  const int bt = less(sh.xo[0][t], sh.n[0]);
#pragma unroll
  for (int d = 0; d < D; ++d) {
    if (d >= q.n) continue;
    const int bd = less(sh.xo[d + 1][t], sh.n[d + 1]);
    const float G = ldexpf(sh.G[d], less(bt, bd));
    float y[E];
#pragma unroll
    for (int e = 0; e < E; ++e) y[e] = min_pos(x[0][e] * G, x[d + 1][e]);
    sh.xs[d][t] = sum_elems(y) * ldexpf(sh.F[d], bd);
  }
}

// ---- 6. per-thread min-sums, from the logits again: with u_v = z_t,v c - o_t and
// w_v = z_d,v c - o_d, p_v = 2^(u_v + a_t) and q_v = 2^(w_v + a_d), so
// min(p_v, q_v) = 2^(a_t) 2^min(u_v, w_v - (a_t - a_d)), and in the plain form (one o)
// w_v - (a_t - a_d) is one fma z_d,v c + nw_d; one fma, one min, one exp2 and one add per
// drafter logit. The factor 2^(a_t) is applied to the group sum. Identical rows give nw_d = -o,
// so both operands agree bitwise ----
template <int DT, int D, bool WIDE, typename L>
__device__ __forceinline__ void thread_minsums_form(const TeamArgs& A, const ItemPos& q,
                                                    typename Vec<DT>::Raw (&raw)[D + 1], L& sh,
                                                    int t) {
  constexpr int E = Vec<DT>::kElems;
  float u[E];
  launder(raw[0]);
  Vec<DT>::unpack(raw[0], u);
  const float nt = sh.no[0];
#pragma unroll
  for (int e = 0; e < E; ++e) u[e] = fmaf(u[e], A.c, nt);
#pragma unroll
  for (int d = 0; d < D; ++d) {
    if (d >= q.n) continue;
    float w[E];
    launder(raw[d + 1]);
    Vec<DT>::unpack(raw[d + 1], w);
    float y[E];
    if (!WIDE) {
      const float nw = sh.nw[d];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        // (nw_d is NaN or infinite only for a row without a distribution: F is NaN then)
        y[e] = __builtin_amdgcn_exp2f(min_arith(u[e], fmaf(w[e], A.c, nw)));
      }
    } else {
      // the exact residual z c - o_d first, then the difference
      const float no = sh.no[d + 1], dl = sh.dl[d];
#pragma unroll
      for (int e = 0; e < E; ++e)
        y[e] = __builtin_amdgcn_exp2f(fminf(u[e], fmaf(w[e], A.c, no) - dl));
    }
    sh.xp[d][t] = sum_elems(y);
  }
}
// The form is chosen once per item (uniform), so that each copy of the loop is straight-line
// over all drafters and the compiler can interleave them.
template <int DT, int D, typename L>
__device__ __forceinline__ void thread_minsums(const TeamArgs& A, const ItemPos& q,
                                               typename Vec<DT>::Raw (&raw)[D + 1], L& sh,
                                               int t) {
  if (sh.wide == 0) thread_minsums_form<DT, D, false>(A, q, raw, sh, t);
  else thread_minsums_form<DT, D, true>(A, q, raw, sh, t);
}

// ---- 7. alpha of the set's drafters from the slice partials: output d is summed by slot
// d mod S (wave 1 for the first), lane l taking slices l, l + 64, ... in order, then across the
// wave ----
template <int D>
__device__ __forceinline__ void fold_alpha(const TeamArgs& A, const ItemPos& q, uint32_t tag,
                                           int lane, int wv, int rot = 0) {
  const int S = A.S;
  for (int d = duty_index(q.s, rot, S) + ((wv + 3) & 3) * S; d < q.n; d += kWaves * S) {
    const uint64_t* src = A.part + ((int64_t)q.g * A.N + q.sub * D + d) * S;
    float v = 0.0f;
    bool lost = false;
    for (int j0 = 0; j0 < S; j0 += 128) {
      uint64_t w[2];
#pragma unroll
      for (int h = 0; h < 2; ++h)  // issue every load of the pass before waiting on any
        if (j0 + lane + 64 * h < S) w[h] = get_word(src + j0 + lane + 64 * h);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int j = j0 + lane + 64 * h;
        if (j < S) {
          if (tag_of(w[h]) != tag) w[h] = await_word(src + j, tag, A);
          lost |= tainted(w[h]);
          v += word_f(w[h]);
        }
      }
    }
    v = wave_sum_f(v);
    const uint32_t tt = tag | taint_bits(__ballot(lost) != 0);
    // clamped to [0, 1]; a NaN (a row without a distribution, or a lost word) stays NaN
    if (lane == 0) {
      const int64_t o = ((int64_t)q.b * A.N + q.sub * D + d) * A.K + q.k;
      const float al = v != v ? v : fminf(fmaxf(v, 0.0f), 1.0f);
      A.alpha[o] = al;
      if (A.learn == 1) put_word(A.gw + o, word_of(al, tt));
    }
  }
}

// ---- 9. learner step of query b, once this workgroup has finished its items: the query's
// N * K gamma words are gathered into LDS (the team buffers are free by now), then wave 0 runs
// the step; the learner's state is loaded before the gather, so those loads fly meanwhile.
// When any gamma word is tainted (computed from a lost word) the step is skipped: the
// learner state stays as it was and the query's EAL, prefix and loss outputs are NaN.
// The host only asks for it when the learner's LDS fits in the team's. ----
template <typename L>
__device__ __forceinline__ void learn_query(const TeamArgs& A, uint32_t tag, int b, L& sh,
                                            int t) {
  const int nk = A.N * A.K;
  double* lds = reinterpret_cast<double*>(&sh);
  float* gam = reinterpret_cast<float*>(lds + tail_lds_doubles(A.tail));
  const uint64_t* src = A.gw + (int64_t)b * nk;
  LearnerIn pre{};
  if (t < 64) pre = load_learner_in(A.tail, b);
  __syncthreads();  // the team buffers are no longer read
  bool lost = false;
  for (int o = t; o < nk; o += kThreads) {
    const uint64_t w = await_word(src + o, tag, A);
    lost |= tainted(w);
    gam[o] = word_f(w);
  }
  const bool skip = __syncthreads_or(lost) != 0;
  if (t < 64) {
    if (skip) mark_query_failed(A.tail, b);
    else tail_query(A.tail, b, lds, gam, &pre);
  }
  __syncthreads();
}

// ---- 8. end of a workgroup ----
// A team's leader counts its team once every member has read the call's tag and no claim of
// the team is outstanding: after folding row 0 of the team's last item (at its end), or, with
// one item per workgroup, right after folding row 0. The
// last team counted advances the epoch and resets the row-set counter (one count per team,
// not per workgroup; the count of finished teams is tagged with the call, so it needs no
// reset).
__device__ inline void count_team(const TeamArgs& A, uint32_t tag, int teams) {
  if (tagged_add(A.finished, tag) == (uint32_t)teams - 1u) {
    const uint32_t e = *A.epoch + 1u;
    *A.next_set = 0u;  // every team has finished: nothing claims any more
    put_word(A.finished, (uint64_t)tag_of_epoch(e));  // count 0 for the next call's tag
    *A.epoch = e;      // the next call takes a new tag
  }
}
// When a wait of this call gave up, every workgroup that sees the fail flag at its end marks
// every output (alpha NaN, argmax -2, agreement 0): a wave that took a lost word has seen the
// flag, so each value computed from one is overwritten by the same workgroup, and outputs of
// row sets that no team reached are marked too; values written without a lost word are
// correct either way.
template <typename L>
__device__ __forceinline__ void finish(const TeamArgs& A, uint32_t tag, bool count, int teams,
                                       L& sh, int t) {
  if (t == 0) {
    const uint64_t fw = get_word(A.fail);
    const uint32_t flags = ((uint32_t)fw == tag && (fw >> 32) != 0) ? 2u : 0u;
    if (count) count_team(A, tag, teams);
    sh.next = flags;
  }
  __syncthreads();
  if (sh.next == 0u) return;
  const int64_t outs = (int64_t)A.B * A.N * A.K;
  for (int64_t o = t; o < outs; o += kThreads) {
    if (A.alpha) A.alpha[o] = __int_as_float(0x7FC00000);
    if (A.agree) A.agree[o] = 0;
    if (A.argmax_d) A.argmax_d[o] = -2;
  }
  if (A.argmax_t)
    for (int64_t o = t; o < (int64_t)A.B * A.K; o += kThreads) A.argmax_t[o] = -2;
}

// A team of S workgroups (slot s takes slice s of every item) works through row sets: its
// first three are sets T, T + teams and T + 2 teams (T = team), later ones are claimed three
// items ahead by the team's leader from a device-wide counter and posted in the team's
// mailbox ring, so teams that run faster (the wave arbiter favours older waves) take more sets
// and all finish within an item of each other.
// With alpha two items are in flight per workgroup: iteration j folds item j (published in the
// previous iteration), takes the statistics of item j + 1 and publishes them, and only then
// waits for item j's normalisers and takes its min-sums from the logits again, after which
// item j's registers receive the loads of item j + 2. The exchange of one item thus overlaps
// the statistics of the next. Two raw buffers (not three, with the next loads issued before
// the statistics) keep the kernel within 128 VGPRs, so four workgroups share a CU: 3-4% faster
// on every large workload than three workgroups with three buffers.
// COMMON (pipelined, without an argmax): sums against one common offset where they fit it.
// SINGLE: every team has exactly one item, so nothing is pipelined, the
// e_v stay in registers and drafters at a constant distance are addressed without the table.
// With an argmax as well the pipelined kernel's LDS (47 KB with 8 drafters) leaves room for 3 workgroups
// per CU, and it takes the registers (140) that this leaves; its bound says so (43.9 us and, with a
// bound of 4, 44.3 for 13 queries x 5 drafters x 7 positions x 50257 fp16 logits).
template <int DT, int D, bool NEED_ARG, bool SINGLE, bool COMMON>
__global__ __launch_bounds__(kThreads, NEED_ARG && !SINGLE ? 3 : 4) void hs_team_kernel(TeamArgs A) {
  using Raw = typename Vec<DT>::Raw;
  constexpr int RM = D + 1;
  __shared__ TeamLds<D, NEED_ARG, SINGLE> sh;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  int t, lane, gi, gl;  // 16-lane group gi reduces row gi; gl: lane in it
  // The thread's indices afresh: taken from an opaque copy, so that the pipelined kernel's many LDS
  // and word addresses are formed where they are used instead of being kept across its loop, where
  // they would not fit in registers (a spilled one comes back by a load that waits for the next
  // item's logits).
  auto reindex = [&]() __attribute__((always_inline)) {
    t = threadIdx.x;
    if (!SINGLE) asm volatile("" : "+v"(t));
    lane = t & 63;
    gi = t >> 4;
    gl = t & 15;
  };
  reindex();
  const int S = A.S;
  // every scalar the first loads depend on, requested in one round at entry (otherwise each
  // is loaded just before its first use, one scalar-cache round trip apiece); the pipelined
  // alpha kernel, whose first loads are a small part of its run, loads them at first use
  // instead (0.6% faster there: fewer scalar registers held across its loop)
  if constexpr (SINGLE) {
    asm volatile("" ::"s"(A.N), "s"(A.K), "s"(A.nsub), "s"(A.S), "s"(A.items), "s"(A.teams),
                 "s"(A.uni), "s"(A.divS.m), "s"(A.divS.s1), "s"(A.divS.s2), "s"(A.divK.m),
                 "s"(A.divK.s1), "s"(A.divK.s2), "s"(A.V), "s"(A.dd), "s"(A.base0),
                 "s"(A.base1), "s"(A.sb0), "s"(A.sk0), "s"(A.sb1), "s"(A.sk1), "s"(A.epoch));
  }
  const int teams = A.teams;
  // consecutive workgroups form a team; the workgroups that share a CU (w, w + CUs, ...)
  // then belong to different teams, so that one team's waits leave the CU to the others
  const int T = (int)fdiv(blockIdx.x, A.divS);
  // slot: the member's slice. The pipelined kernel rotates it by the team index, so that the
  // workgroups a CU holds at once (w, w + CUs, ...) take different slices also when S divides
  // the number of CUs (8% on 64 stacked fp32 tiny chains, S = 32; no change where it does not)
  int slot = (int)blockIdx.x - T * S;
  if constexpr (!SINGLE) {
    slot += T - (int)fdiv((uint32_t)T, A.divS) * S;  // + T mod S
    if (slot >= S) slot -= S;
  }
  const uint32_t nsets = fdiv((uint32_t)A.items, A.divS);
  // slot 0 is its team's leader: it waits for the normalisers of each item, which need the whole
  // team, so it can never be more than one item ahead of any member, which keeps a ring of 4
  // mailbox words safe
  const bool leader = slot == 0;
  uint32_t tag = 0;  // the call's tag: read once the first loads are in flight
  uint64_t* mbox = A.mbox + (size_t)T * 4;
  if (!(SINGLE && A.uni) && t < kMaxRows) {
    sh.ptr[t] = reinterpret_cast<const char*>(A.rows.ptr[t]);
    sh.sb[t] = A.rows.sb[t];
    sh.sk[t] = A.rows.sk[t];
  }
  __syncthreads();

  // first slot of the row or alpha fold duties of row set `set` (several items per workgroup):
  // (set (D + 1) + extra) mod S, so consecutive items use different members, and the alpha
  // folds of an item start where its row folds end.
  auto rotation = [&](uint32_t s, int extra) __attribute__((always_inline)) -> int {
    const uint32_t x = s * (uint32_t)RM + (uint32_t)extra;
    return (int)(x - fdiv(x, A.divS) * (uint32_t)S);
  };

  bool own = false;  // COMMON: this wave's last item needed offsets of its own
  // statistics of item q from raw, published
  auto stats = [&](const ItemPos& q, Raw (&raw)[RM]) __attribute__((always_inline)) {
    __builtin_amdgcn_s_setprio(kCritPrio);
    reindex();
    mask_tail<DT, D>(A, q, raw);
    if constexpr (COMMON) thread_stats_common<DT, D>(A, q, raw, sh, t, own);
    else thread_stats<DT, D, NEED_ARG, false>(A, q, raw, sh, sh, t);
    __syncthreads();
    reindex();
    if (wv * 4 <= q.n) {  // this wave holds the group of a row
      if constexpr (COMMON) publish_stats_common(A, q, tag, RM, sh, gi, gl);
      else publish_stats<NEED_ARG>(A, q, tag, RM, sh, gi, gl);
    }
    __builtin_amdgcn_s_setprio(0);
  };
  // the item's slice partials to the workspace (after a barrier), as tagged words
  auto store_partials = [&](const ItemPos& q) __attribute__((always_inline)) {
    if (wv * 4 < q.n) {
      float v[16];
      const int d = min(gi, q.n - 1);
      group_read(SINGLE ? &sh.xs[d][0] : &sh.xp[d][0], gl, v);
      float y = row16_sum(sum16(v));
      if (!SINGLE) y *= sh.F[d];
      if (gl == 0 && gi < q.n)
        put_word(A.part + ((int64_t)q.g * A.N + q.sub * D + gi) * S + q.s,
                 word_of(y, tag | sh.taint));
    }
  };

  // Several items per workgroup: the row sets of one (query, position) group follow each
  // other in a team when there are groups enough to keep every team busy, so the target's
  // slice, the same for all of them, is re-read from this XCD's L2 rather than from HBM. A
  // team's items come in blocks (a group's nsub row sets, else single row sets): its first
  // kB blocks are blocks T, T + teams, ... (at least three items, to fill the pipeline), and
  // later ones are claimed from the device-wide counter three items ahead, by the leader,
  // and posted in the team's mailbox ring.
  const bool blocked = !SINGLE && A.nsub > 1 && nsets >= 4u * (uint32_t)teams * (uint32_t)A.nsub;
  const uint32_t bsz = blocked ? (uint32_t)A.nsub : 1u;
  const uint32_t nblocks = blocked ? fdiv(nsets, A.divNsub) : nsets;
  const int kB = blocked ? (int)((3u + bsz - 1u) / bsz) : 3;
  const bool dyn = kB * teams < (int)nblocks;  // else no team has more than its fixed blocks
  int nblk = 0;  // blocks given to this team so far (the same count in every member)
  auto block_first = [&](uint32_t bl) { return bl < nblocks ? bl * bsz : nsets; };
  // the row set after s (nsets: none), or kClaim when it starts a block that is to be claimed
  constexpr uint32_t kClaim = 0xFFFFFFFFu;
  auto successor = [&](uint32_t s) __attribute__((always_inline)) -> uint32_t {
    if (s >= nsets) return nsets;
    if (blocked && fdiv(s + 1u, A.divNsub) * bsz != s + 1u) return s + 1u;  // same group
    if (nblk < kB) return block_first((uint32_t)(T + (nblk++) * teams));
    return dyn ? kClaim : nsets;
  };

  Raw R0[RM], R1[RM];
  uint32_t set = SINGLE ? (uint32_t)T : block_first((uint32_t)T);
  nblk = 1;
  const ItemPos q0 = item_pos(A, set, slot, D);
  fetch_item<DT, D, SINGLE>(A, q0, true, sh, R0);
  if constexpr (SINGLE) {
    // one item per workgroup: nothing to overlap, so its e_v stay in registers
    tag = call_tag(A.epoch);  // first needed once the first loads are in flight
    const ItemPos& q = q0;
    float x[RM][Vec<DT>::kElems];
    __builtin_amdgcn_s_setprio(kCritPrio);
    mask_tail<DT, D>(A, q, R0);
    thread_stats<DT, D, NEED_ARG, true>(A, q, R0, x, sh, t);
    __syncthreads();
    if (wv * 4 <= q.n) publish_stats<NEED_ARG>(A, q, tag, RM, sh, gi, gl);
    fold_item<D, NEED_ARG, true, kNormCopies>(A, q, tag, lane, wv, 0);
    __builtin_amdgcn_s_setprio(0);
    // with one item per workgroup the leader counts its team once it has folded row 0 (every
    // member has published, so has read the tag), not at its end: the count's round trip
    // then overlaps the normaliser wait instead of following the learner step or the alpha
    // folds. (The fold duties start at wave 0, whose thread 0 counts.)
    if (leader && t == 0) count_team(A, tag, teams);
    if (wv == 0) await_norms<D, true>(A, q, tag, sh, lane);
    __syncthreads();
    thread_minsums_kept<DT, D>(q, x, sh, t);
    __syncthreads();
    store_partials(q);
    fold_alpha<D>(A, q, tag, lane, wv);
    if (A.learn)
      for (int b = blockIdx.x; b < A.B; b += gridDim.x) learn_query(A, tag, b, sh, t);
    finish(A, tag, false, teams, sh, t);
    return;
  }
  uint32_t pset = nsets;  // the team's previous item, whose alpha is still to be folded
  uint32_t set1 = successor(set);
  uint32_t set2 = successor(set1);  // items 0-2 lie in fixed blocks: never kClaim
  fetch_item<DT, D>(A, item_pos(A, min(set1, nsets - 1), slot, D), set1 < nsets, sh,
                    R1);
  tag = call_tag(A.epoch);  // first needed once the first loads are in flight
  stats(q0, R0);
  // the first item's group reductions read every column of the LDS rows that the next
  // item's per-thread statistics overwrite, and nothing else in the first iteration waits
  // for the whole workgroup before those writes (later items are kept apart by the
  // barriers around the min-sums); after it every wave has published its rows
  __syncthreads();

  // iteration j: rc holds item j (statistics published) and then receives item j + 2, rn
  // holds item j + 1 (loaded). Returns false once the team has no item j + 1.
  auto iter = [&](int j, Raw (&rc)[RM], Raw (&rn)[RM])
                  __attribute__((always_inline)) -> bool {
    const ItemPos q = item_pos(A, set, slot, D);
    // the leader's claim of item j + 3 goes out before the fold and is posted after it, so
    // waiting for its result waits for nothing else; the duty wave, which folds, claims
    const uint32_t set3 = successor(set2);  // item j + 3, unless it is to be claimed
    const bool claiming = set3 == kClaim && leader && wv == kDutyWave && lane == 0;
    uint32_t cv = 0;
    if (claiming)
      cv = __hip_atomic_fetch_add(A.next_set, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_setprio(kFoldPrio);
    reindex();
    fold_item<D, NEED_ARG, !COMMON>(A, q, tag, lane, wv, kDutyWave, rotation(set, 0));
    __builtin_amdgcn_s_setprio(0);
    if (claiming)
      put_word(mbox + ((j + 3) & 3),
               mbox_word(block_first((uint32_t)(kB * teams) + cv), j + 3, tag));
    if (set1 < nsets) stats(item_pos(A, set1, slot, D), rn);
    else __syncthreads();  // the previous item's constants in LDS are no longer read
    if (set3 == kClaim && t == 0) sh.next = await_mbox(mbox + ((j + 3) & 3), j + 3, tag, A, nsets);
    reindex();
    if (wv == kDutyWave) await_norms<D, false>(A, q, tag, sh, lane);
    __syncthreads();
    reindex();
    thread_minsums<DT, D>(A, q, rc, sh, t);
    __syncthreads();
    reindex();
    store_partials(q);
    fetch_item<DT, D>(A, item_pos(A, min(set2, nsets - 1), slot, D), set2 < nsets, sh, rc);
    // alpha of the previous item, whose partials were stored an iteration ago; its polls
    // overlap the loads just issued (1.4% faster than folding it before the normaliser wait)
    if (pset < nsets) fold_alpha<D>(A, item_pos(A, pset, slot, D), tag, lane, wv, rotation(pset, RM));
    if (set1 >= nsets) return false;
    pset = set;
    set = set1;
    set1 = set2;
    set2 = set3 == kClaim ? sh.next : set3;
    return true;
  };
  // unrolled by two so that the register buffers alternate without copies
  for (int j = 0;; j += 2) {
    if (!iter(j, R0, R1)) break;
    if (!iter(j + 1, R1, R0)) break;
  }
  fold_alpha<D>(A, item_pos(A, set, slot, D), tag, lane, wv, rotation(set, RM));
  if (A.learn)
    for (int b = blockIdx.x; b < A.B; b += gridDim.x) learn_query(A, tag, b, sh, t);
  finish(A, tag, leader, teams, sh, t);
}

// ---- argmax and agreement alone, few items per workgroup ----
// Teams as above, one exchange per item: maxima and argmaxes are published and folded, while the next
// item's loads fly. With few items per workgroup this is faster than the streaming argmax kernel
// (hs_argmax.hip), where all waves of a group count their arrival at one word (some 80 ns each) and
// one wave folds the group: launch_team_argmax says where the line lies.
template <int D>
struct ArgmaxLds {
  float xt[D + 1][kThreads];  // per-thread maxima
  int xi[D + 1][kThreads];    // per-thread argmax
  uint32_t next;
  const char* ptr[kMaxRows];
  int64_t sb[kMaxRows];
  int64_t sk[kMaxRows];
};
template <int DT, int D>
__global__ __launch_bounds__(kThreads, 4) void hs_team_argmax_kernel(TeamArgs A) {
  using Raw = typename Vec<DT>::Raw;
  constexpr int RM = D + 1, E = Vec<DT>::kElems;
  __shared__ ArgmaxLds<D> sh;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int gi = t >> 4, gl = t & 15;
  // every scalar the first loads depend on, requested in one round at entry
  asm volatile("" ::"s"(A.N), "s"(A.K), "s"(A.nsub), "s"(A.S), "s"(A.items), "s"(A.teams),
               "s"(A.uni), "s"(A.divS.m), "s"(A.divS.s1), "s"(A.divS.s2), "s"(A.divK.m),
               "s"(A.divK.s1), "s"(A.divK.s2), "s"(A.V), "s"(A.epoch));
  const int teams = A.teams;
  const int T = (int)fdiv(blockIdx.x, A.divS), slot = (int)blockIdx.x - T * A.S;
  const uint32_t nsets = fdiv((uint32_t)A.items, A.divS);
  // slot 0 folds row 0 of every item, so it waits for the whole team each item: it can never
  // be more than one item ahead of any member, which keeps a ring of 4 mailbox words safe
  const bool leader = slot == 0;
  const bool dynamic = 2 * teams < (int)nsets;  // else no team has more than its two fixed sets
  uint64_t* mbox = A.mbox + (size_t)T * 4;
  if (t < kMaxRows) {
    sh.ptr[t] = reinterpret_cast<const char*>(A.rows.ptr[t]);
    sh.sb[t] = A.rows.sb[t];
    sh.sk[t] = A.rows.sk[t];
  }
  __syncthreads();
  Raw nxt[RM];
  uint32_t set = (uint32_t)T, next = min((uint32_t)(T + teams), nsets);
  fetch_item<DT, D>(A, item_pos(A, set, slot, D), true, sh, nxt);
  const uint32_t tag = call_tag(A.epoch);  // first needed once the first loads are in flight
  for (int j = 0; set < nsets; ++j) {
    const ItemPos q = item_pos(A, set, slot, D);
    __builtin_amdgcn_s_setprio(kCritPrio);
    mask_tail<DT, D>(A, q, nxt);
#pragma unroll
    for (int r = 0; r <= D; ++r) {
      if (r > q.n) continue;
      launder(nxt[r]);
      float z[E];
      Vec<DT>::unpack(nxt[r], z);
      thread_argmax<E>(A, q, r, z, sh, t);
    }
    // the team's item j + 1 (claimed two items ago), all waves alike after the barrier
    if (j >= 1 && t == 0) sh.next = dynamic ? await_mbox(mbox + ((j + 1) & 3), j + 1, tag, A, nsets) : nsets;
    // leader: claim the row set of item j + 2 and post it (the counter starts past every team's
    // fixed sets, so a set is never claimed twice)
    if (dynamic && leader && t == 0) {
      const uint32_t v = (uint32_t)(2 * teams) +
                         __hip_atomic_fetch_add(A.next_set, 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
      put_word(mbox + ((j + 2) & 3), mbox_word(min(v, nsets), j + 2, tag));
    }
    __syncthreads();
    if (j >= 1) next = sh.next;
    if (next < nsets) fetch_item<DT, D>(A, item_pos(A, next, slot, D), true, sh, nxt);
    if (wv * 4 <= q.n) {
      float m;
      int idx;
      group_argmax(sh, q.n, gi, gl, m, idx);
      if (gl == 0 && gi <= q.n) {
        uint64_t* wp = stat_row(A, q.set, gi, RM) + 2 * q.s;
        put_word(wp, word_of(m, tag));
        put_word(wp + 1, word_of(idx, tag));
      }
    }
    // the folds (fold_item's order), the duty wave first
    for (int rr = q.s + ((wv + kWaves - kDutyWave) % kWaves) * A.S; rr <= q.n; rr += kWaves * A.S)
      fold_row_argmax<D>(A, q.set, rr, q.b, q.k, q.sub, tag, lane);
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();  // the LDS rows are free for the next item
    set = next;
  }
  finish(A, tag, leader, teams, sh, t);
}

// ---- host side -------------------------------------------------------------------------------

namespace {

// Polls before a wait inside the team kernel gives up (about 0.5 s at the default); 0 makes
// every wait give up at once, which tests of the failure path set from the host.
constexpr uint32_t kDefaultPolls = 1u << 18;
std::atomic<uint32_t> g_wait_polls{kDefaultPolls};

uint32_t wait_polls() { return g_wait_polls.load(std::memory_order_relaxed); }

// Workgroups of the team kernel the current device holds at once.
template <typename K>
int capacity_of(K kernel, std::atomic<int> (&cached)[64]) {  // cached per device; 0 = not yet known
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int v = cached[dev].load(std::memory_order_relaxed);
  if (v > 0) return v;
  int per_cu = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kThreads, 0) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  v = per_cu * cus;
  cached[dev].store(v, std::memory_order_relaxed);
  return v;
}
template <int DT, int D, bool NA, bool SG, bool CO>
int capacity_t() {
  static std::atomic<int> cached[64];
  return capacity_of(hs_team_kernel<DT, D, NA, SG, CO>, cached);
}

// Runs the team kernel with as many teams as the device holds at once (no more than there are
// row sets or mailbox rings); the single-item kernel when that covers every row set.
// *learned: whether the launch runs the learner step itself (its LDS fits in the team's).
template <int DT, int D, bool NA>
int launch_t(TeamArgs A, const TeamGeom& g, hipStream_t stream, bool* learned) {
  const int64_t sets = g.items / g.S;
  const bool single = capacity_t<DT, D, NA, true, false>() / g.S >= sets;
  // The common offset's range is 152 binary orders, which at a low temperature the rows' maxima no
  // longer fit: T = 0.4, 0.3, 0.2 and 0.1 with the common offset 217, 221, 233 and 254 us, with own
  // offsets 222, 222, 223 and 228 (64 queries x 8 drafters x 6 positions x 128256 bf16 logits);
  // 51, 51, 60 and 60 us against 51 throughout (64 x 4 x 4 x 32000 fp32).
  constexpr float kCommonScale = 5.0f;  // log2(e) / T: T of about 0.29
  const bool common = !NA && !single && A.c <= kCommonScale;
  const int cap = common ? capacity_t<DT, D, NA, false, !NA>() : capacity_t<DT, D, NA, false, false>();
  const int64_t teams =
      single ? sets : std::min<int64_t>({cap / g.S, sets, (int64_t)kMaxTeams});
  if (teams <= 0) return HS_ERR_LIMIT;
  const int64_t P = teams * g.S;
  if (A.learn) {
    const size_t need = sizeof(double) * (size_t)tail_lds_doubles(A.tail) +
                        sizeof(float) * (size_t)g.N * g.K;
    if (need > (single ? sizeof(TeamLds<D, NA, true>) : sizeof(TeamLds<D, NA, false>))) A.learn = 0;
  }
  *learned = A.learn != 0;
  A.teams = (int)teams;
  if (single) hs_team_kernel<DT, D, NA, true, false><<<(unsigned)P, kThreads, 0, stream>>>(A);
  else if (common) hs_team_kernel<DT, D, NA, false, !NA><<<(unsigned)P, kThreads, 0, stream>>>(A);
  else hs_team_kernel<DT, D, NA, false, false><<<(unsigned)P, kThreads, 0, stream>>>(A);
  return HS_OK;
}

// Argmax and agreement by the team kernel where it is the faster, or the streaming kernel cannot number
// the call's units (*taken), else nothing. The streaming kernel's waves all count their arrival at their
// group's word, which costs little where a group has few waves (wpg) or each wave a long span, as its
// arrivals then spread over the run; teams cost a hop per item, and more where they claim items beyond
// their two fixed ones. us, streaming and by teams:
// - groups of few units or rows of few slices, streaming: 62 queries x 8 drafters x 8 positions x 4050 bf16
//   logits 19.6 and 30.3, 15 x 11 x 1 x 4913 (3 slices) 8.7 and 11.2; 21 x 8 x 6 x 9749 (5) 37.0 and 20.6,
//   9 x 43 x 9 x 8032 (4, and 88 units) 59.6 and 31.5;
// - up to two items per team, teams: 1 x 8 x 8 x 151936 46 and 10.3, 1 x 15 x 8 x 96771 197 and 14.4,
//   23 x 8 x 3 x 33784 fp32 48 and 25.6 at 1.8; with groups of up to 25 waves, up to one and a half:
//   42 x 4 x 2 x 42365 28.1 and 21.4 at 1.2, 21 x 6 x 6 x 40445 25.1 and 29.4 at 2;
// - up to six, with more than 50 waves to a group of at most four units each and up to 128 row sets, which
//   are claimed one by one: 10 x 6 x 3 x 151133 fp32 119 and 41, 8 x 9 x 8 x 62503 (128) 77 and 65; 24 x 17 x 2
//   x 37314 (144) 30.4 and 57.2, 13 x 10 x 5 x 52015 (48 waves) 44.3 and 59.7, 1 x 52 x 24 x 71662
//   (six units) 55.5 and 91, 5 x 42 x 8 x 43670 (five) 52.4 and 99.6; with longer spans where row sets are
//   few: 10 x 7 x 4 x 125874 fp32 (40 sets) 73.6 and 46.7, 1 x 8 x 48 x 128496 fp32 (48) 59.4 and 57.5, 8 x
//   15 x 5 x 101752 fp32 (80) 65.6 and 73.6; and with more than 200 waves to a group: 3 x 63 x 6 x 51371 101
//   and 58, 5 x 47 x 3 x 83876 fp32 71 and 66.
template <int DT, int D>
int launch_team_argmax(TeamArgs A, const TeamGeom& g, hipStream_t stream, bool* taken) {
  static std::atomic<int> cached[64];
  const int cap = capacity_of(hs_team_argmax_kernel<DT, D>, cached);
  const ArgmaxPlan p = argmax_plan(g);
  const int64_t sets = g.items / g.S, teams = std::min<int64_t>({cap / g.S, sets, (int64_t)kMaxTeams});
  const auto wpg_over = [&](int64_t waves) { return p.per_group > waves * p.span; };
  const bool many = wpg_over(200) ||
                    (p.span <= 4 ? wpg_over(50) && sets <= 128 : wpg_over(62) && sets <= 48);
  const bool faster = p.per_group > 20 && (g.S > 4 || p.per_group > 56) &&
                      2 * sets <= (many ? 12 : wpg_over(25) ? 4 : 3) * teams;
  *taken = !argmax_fits(p) || (teams > 0 && faster);
  if (!*taken) return HS_OK;
  if (teams <= 0) return HS_ERR_LIMIT;
  A.learn = 0;
  A.teams = (int)teams;
  hs_team_argmax_kernel<DT, D><<<(unsigned)(A.teams * g.S), kThreads, 0, stream>>>(A);
  return hipGetLastError() == hipSuccess ? HS_OK : HS_ERR_HIP;
}

// Calls F<DT, D, NA>::run(args...) for the geometry and mode.
template <template <int, int, bool> class F, int DT, int D, typename... Args>
int by_mode(bool na, Args&&... args) {
  return na ? F<DT, D, true>::run(args...) : F<DT, D, false>::run(args...);
}
template <template <int, int, bool> class F, int DT, typename... Args>
int by_set(int D, bool na, Args&&... args) {
  switch (D) {
    case 1: return by_mode<F, DT, 1>(na, args...);
    case 2: return by_mode<F, DT, 2>(na, args...);
    case 4: return by_mode<F, DT, 4>(na, args...);
    default: return by_mode<F, DT, kMaxSetDrafters>(na, args...);
  }
}
template <template <int, int, bool> class F, typename... Args>
int dispatch(const TeamGeom& g, bool na, Args&&... args) {
  if (g.dtype == HS_F32) return by_set<F, HS_F32>(g.D, na, args...);
  if (g.dtype == HS_F16) return by_set<F, HS_F16>(g.D, na, args...);
  return by_set<F, HS_BF16>(g.D, na, args...);
}

template <int DT, int D, bool NA>
struct Capacity {  // the smallest of the kernels' (a team must fit in any)
  static int run() {
    return std::min({capacity_t<DT, D, NA, false, !NA>(), capacity_t<DT, D, NA, false, false>(),
                     capacity_t<DT, D, NA, true, false>()});
  }
};
template <int DT, int D, bool NA>
struct Launch {
  static int run(const TeamArgs& A, const TeamGeom& g, hipStream_t s, bool* learned) {
    return launch_t<DT, D, NA>(A, g, s, learned);
  }
};

template <int DT, int D, bool NA>
struct LaunchArgmax {
  static int run(const TeamArgs& A, const TeamGeom& g, hipStream_t s, bool* taken) {
    return launch_team_argmax<DT, D>(A, g, s, taken);
  }
};

}  // namespace

void set_wait_polls(int polls) {
  g_wait_polls.store(polls < 0 ? kDefaultPolls : (uint32_t)polls, std::memory_order_relaxed);
}

int team_capacity(const TeamGeom& g, bool need_arg) {
  return dispatch<Capacity>(g, need_arg);
}

int launch_round(const TeamGeom& g, const RowTable& rows, float c, bool need_sum, bool need_arg,
                 float* alpha, uint8_t* agree, int32_t* argmax_t, int32_t* argmax_d, char* ws,
                 const TailArgs* tail, hipStream_t stream) {
  const TeamWs L = team_ws(g);
  TeamArgs A{};
  A.epoch = reinterpret_cast<uint32_t*>(ws + L.epoch);
  A.fail = reinterpret_cast<uint64_t*>(ws + L.epoch + 8);
  // a learner step of its own, told where to see whether the evaluation failed
  auto tail_after = [&]() -> int {
    TailArgs a = *tail;
    a.round_epoch = A.epoch;
    a.round_fail = A.fail;
    return launch_tail(a, stream);
  };
  A.rows = rows;
  A.base0 = rows.ptr[0];
  A.base1 = rows.ptr[1];
  A.sb0 = rows.sb[0];
  A.sk0 = rows.sk[0];
  A.sb1 = rows.sb[1];
  A.sk1 = rows.sk[1];
  // drafters at one constant distance with equal strides (e.g. one [N][B][K][V] tensor)
  A.uni = 1;
  A.dd = g.N > 1 ? reinterpret_cast<const char*>(rows.ptr[2]) -
                       reinterpret_cast<const char*>(rows.ptr[1])
                 : 0;
  for (int i = 2; i <= g.N && A.uni; ++i)
    A.uni = reinterpret_cast<const char*>(rows.ptr[i]) -
                    reinterpret_cast<const char*>(rows.ptr[i - 1]) ==
                A.dd &&
            rows.sb[i] == rows.sb[1] && rows.sk[i] == rows.sk[1];
  A.B = g.B;
  A.N = g.N;
  A.K = g.K;
  A.nsub = g.nsub;
  A.S = g.S;
  A.divS = make_fastdiv((uint32_t)g.S);
  A.divNsub = make_fastdiv((uint32_t)g.nsub);
  A.divK = make_fastdiv((uint32_t)g.K);
  A.items = (int)g.items;
  A.V = g.V;
  A.nvec = g.nvec;
  A.c = c;
  // About 5.5 logits above 0, as an integer power of two: an exponent is rounded at 2^-24 of its own
  // size, and this puts those of the heavy tokens of a head (logits of 0 to 20) nearest to 0.
  // alpha's error against 64 bits (2-norm, simulated rounding, heads of 50k to 76k tokens): 1.5e-7,
  // 2.2e-7 and 3.3e-7 at T = 1, 0.7 and 0.5; with offset 0 1.8e-7, 2.2e-7 and 5.2e-7, with offset
  // 16 2.0e-7, 2.0e-7 and 3.3e-7, and with each slice's maximum 1.7e-7, 2.3e-7 and 4.7e-7.
  A.o = std::nearbyint(std::min(5.5f * c, 48.0f));
  A.polls = wait_polls();
  A.next_set = reinterpret_cast<uint32_t*>(ws + L.epoch + 16);
  A.finished = reinterpret_cast<uint64_t*>(ws + L.epoch + 24);
  A.mbox = reinterpret_cast<uint64_t*>(ws + L.epoch + 64);
  A.stat = reinterpret_cast<uint64_t*>(ws + L.stat);
  A.norm = reinterpret_cast<uint64_t*>(ws + L.norm);
  A.part = reinterpret_cast<uint64_t*>(ws + L.part);
  A.alpha = alpha;
  A.argmax_t = argmax_t;
  A.argmax_d = argmax_d;
  A.agree = agree;
  // the gamma words (the learner step in the same launch); the single-item kernel's extra
  // normaliser copies follow them
  A.gw = reinterpret_cast<uint64_t*>(ws + L.gw);
  if (!need_sum) {
    bool taken = false;
    int rc = dispatch<LaunchArgmax>(g, true, A, g, stream, &taken);
    if (!rc && !taken) rc = launch_argmax(g, rows, agree, argmax_t, argmax_d, A.polls, ws, stream);
    return rc || !tail ? rc : tail_after();
  }
  if (tail) {  // the learner step in the same launch, when its LDS fits
    A.learn = tail->gamma_src;
    A.tail = *tail;
  }
  bool learned = false;
  int rc = dispatch<Launch>(g, need_arg, A, g, stream, &learned);
  if (rc) return rc;
  if (hipGetLastError() != hipSuccess) return HS_ERR_HIP;
  return tail && !learned ? tail_after() : HS_OK;
}

}  // namespace hs
