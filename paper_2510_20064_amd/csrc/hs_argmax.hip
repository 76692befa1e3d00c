// Greedy agreement without alpha: the argmax of every row and, per drafter, whether it equals the
// target's. Nothing needs a row's normaliser here, so no slice waits for another:
//   1. the rows of all (query, position) groups, cut into units of 8 KB, form one sequence; a wave
//      takes a span of it, one unit in registers and the next one's loads in flight, and
//      publishes the maximum of each row's piece and the vector that holds it, as tagged words;
//   2. the wave that arrives last at a group folds the group's rows, reads the one vector that
//      holds each row's maximum for the element, and writes the argmaxes and agreements; the one
//      that folds the last group marks every output when a wait of any fold has given up.
// Bound by HBM: 64 queries x 8 drafters x 6 positions x 128256 bf16 logits in 142 us (6.2 TB/s; the
// card streams 7.0). The argmax variant of the team kernel, whose members wait for each other's
// words between the loads of one item and the next, takes 189 us; it takes the calls with few items
// (launch_team_argmax).
#include "hs_exchange.h"

namespace hs {
namespace {

constexpr int kStep = kArgmaxStep;
// Polls of an adder for its count to be opened (the opening wave comes first in dispatch order and
// opens while its own first loads fly, so an adder hardly ever meets a count that is not open).
constexpr uint32_t kOpenPolls = 1u << 10;

struct ArgmaxArgs {
  int N, K, G;
  int S;     // units per row
  int span;  // units per wave
  int total;      // units of all groups
  int pieces;     // pieces of a row at most
  FastDiv div_group, divS, divK, div_span;  // by the units of a group, S, K and span
  int64_t V, nvec;
  uint32_t* epoch;
  uint64_t* fail;
  uint32_t polls;
  uint64_t* finished;  // groups folded (a tagged count)
  uint64_t* arrived;   // [G] waves that have published (tagged counts)
  uint64_t* words;     // [G][N + 1][pieces][2]: maximum, vector
  int32_t* argmax_t;
  int32_t* argmax_d;
  uint8_t* agree;
  RowTable rows;
};

template <int DT>
__device__ __forceinline__ const char* row_ptr(const ArgmaxArgs& A, int r, int g) {
  const int b = (int)fdiv((uint32_t)g, A.divK), k = g - b * A.K;
  return static_cast<const char*>(A.rows.ptr[r]) +
         ((int64_t)b * A.rows.sb[r] + (int64_t)k * A.rows.sk[r]) * Vec<DT>::kBytes;
}

// In the count of folded groups: a wait of one of these folds has given up.
constexpr uint32_t kFailed = 1u << 31;

// Output stores go past the caches of this XCD, so that marks written by another one after them
// (mark_all) are what memory holds in the end.
template <typename T>
__device__ __forceinline__ void put_out(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every output of the call invalid (one wave).
__device__ inline void mark_all(const ArgmaxArgs& A, int lane) {
  const int64_t outs = (int64_t)A.G * A.N;
  for (int64_t o = lane; o < outs; o += 64) {
    if (A.agree) put_out(A.agree + o, (uint8_t)0);
    if (A.argmax_d) put_out(A.argmax_d + o, -2);
  }
  if (A.argmax_t)
    for (int64_t o = lane; o < A.G; o += 64) put_out(A.argmax_t + o, -2);
}

// Folds group g (one wave, lane r: row r): its pieces' words, then the element of each maximum. True for
// the call's last fold when this or another one has lost a word.
template <int DT>
__device__ __forceinline__ bool fold_group(const ArgmaxArgs& A, int g, uint32_t tag, int lane) {
  const int R = A.N + 1;
  const int b = (int)fdiv((uint32_t)g, A.divK), k = g - b * A.K;
  int target = -2;
  bool gone = false;  // a word of this group is lost
  for (int r0 = 0; r0 < R; r0 += 64) {
    const int r = r0 + lane;
    int e = -2;
    if (r < R) {
      const uint32_t u0 = (uint32_t)((g * R + r) * A.S);  // the row's first unit
      const int n = (int)(fdiv(u0 + (uint32_t)A.S - 1u, A.div_span) - fdiv(u0, A.div_span)) + 1;
      const uint64_t* w = A.words + ((int64_t)g * R + r) * A.pieces * 2;
      float m = -INFINITY;
      int idx = INT_MAX;
      bool lost = false;
      for (int j0 = 0; j0 < n; j0 += 4) {
        uint64_t a[4], c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {  // issue every load before waiting on any
          const int i = min(j0 + j, n - 1);
          a[j] = get_word(w + 2 * i);
          c[j] = get_word(w + 2 * i + 1);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int i = min(j0 + j, n - 1);
          if (tag_of(a[j]) != tag || A.polls == 0) a[j] = await_word(w + 2 * i, tag, A);
          if (tag_of(c[j]) != tag || A.polls == 0) c[j] = await_word(w + 2 * i + 1, tag, A);
          lost |= tainted(a[j]) || tainted(c[j]);
          argmax_combine(m, idx, word_f(a[j]), word_i(c[j]));
        }
      }
      if (!lost) e = argmax_element<DT>(row_ptr<DT>(A, r, g), A.V, A.nvec, m, idx);
      gone |= lost;
    }
    if (r0 == 0) target = __builtin_amdgcn_readfirstlane(e);
    if (r < R) {
      if (r == 0) {
        if (A.argmax_t) put_out(A.argmax_t + (int64_t)b * A.K + k, e);
      } else {
        const int64_t o = ((int64_t)b * A.N + r - 1) * A.K + k;
        if (A.argmax_d) put_out(A.argmax_d + o, e);
        if (A.agree) put_out(A.agree + o, (uint8_t)(e == target && e >= 0));
      }
    }
  }
  const bool failed = __ballot(gone) != 0;
  uint32_t n = 0;
  if (lane == 0) {
    if (failed) {  // before this group is counted, so that the last one sees it
      open_count(A.finished, tag);
      __hip_atomic_fetch_or(A.finished, (uint64_t)kFailed << 32, __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_AGENT);
    }
    n = tagged_add(A.finished, tag, kOpenPolls);
    if ((n & ~kFailed) == (uint32_t)A.G - 1u) {
      // the last group to be folded advances the epoch and leaves its count open for the next call
      const uint32_t e = *A.epoch + 1u;
      put_word(A.finished, (uint64_t)tag_of_epoch(e));
      *A.epoch = e;
    }
  }
  // (a mark may still be followed by the store of a fold that lost nothing: its value is right)
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)n) == (kFailed | ((uint32_t)A.G - 1u));
}

template <int DT>
__global__ __launch_bounds__(kThreads, 4) void hs_argmax_kernel(ArgmaxArgs A) {
  using Vt = Vec<DT>;
  constexpr int E = Vt::kElems;
  using Raw = typename Vt::Raw;
  const int lane = threadIdx.x & 63;
  const int wave = (int)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int u = wave * A.span;
  const int uend = min(u + A.span, A.total);
  if (u >= uend) return;
  // a cached read: the epoch changes only once every wave has arrived, and one agent-scope load
  // per wave of the same word queues at the memory (some 5 ns each)
  const uint32_t e0 = *A.epoch;
  const int R = A.N + 1;
  const int vfull = (int)(A.V / E);  // complete vectors; a row holds fewer than 2^31 logits
  // the unit whose loads go out next, and the unit in use
  int lg = (int)fdiv((uint32_t)u, A.div_group);
  int lr = (int)fdiv((uint32_t)(u - lg * R * A.S), A.divS);
  int lc = u - (lg * R + lr) * A.S;
  const char* lp = row_ptr<DT>(A, lr, lg);
  int g = lg, r = lr, c = lc;
  const char* p = lp;
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  typedef const __attribute__((address_space(1))) u4* gp4;
  // Exactly kStep loads on every path, so that a wait for an older unit leaves these in flight:
  // every address is clamped into the row's complete vectors (a unit past the span, !valid, reads
  // the row's last one; a row without any, the workspace's control block). What a clamped load
  // brings is not used. 16-bit rows load nontemporal (each logit is read once)
  auto load = [&](Raw (&x)[kStep], bool valid) __attribute__((always_inline)) {
    // uniform row base + 32-bit lane offset
    const uint64_t base = reinterpret_cast<uint64_t>(vfull > 0 ? (const void*)lp : A.epoch);
    const int last = max(vfull - 1, 0), v = valid ? lc * 64 * kStep + lane : last;
#pragma unroll
    for (int i = 0; i < kStep; ++i) {
      const gp4 q = (gp4)(base + (uint32_t)min(v + 64 * i, last) * 16u);
      const u4 y = DT != HS_F32 ? __builtin_nontemporal_load(q) : *q;
      __builtin_memcpy(&x[i], &y, 16);
    }
    if (++lc == A.S) {
      lc = 0;
      if (++lr == R) {
        lr = 0;
        ++lg;
      }
      lp = row_ptr<DT>(A, lr, min(lg, A.G - 1));
    }
  };
  bool mark = false;  // (the call's last fold is its wave's last)
  float best = -INFINITY;
  int bi = c * 64 * kStep + lane < (int)A.nvec ? c * 64 * kStep + lane : INT_MAX;
  // uses unit u from x while the loads of the next go out to y; false after the span's last
  auto step = [&](Raw (&x)[kStep], Raw (&y)[kStep]) __attribute__((always_inline)) -> bool {
    const bool more = u + 1 < uend;
    load(y, more);
    const int v = c * 64 * kStep + lane;
#pragma unroll
    for (int i = 0; i < kStep; ++i) {
      float z[E];
      Vt::unpack(x[i], z);
      const float m = max_elems(z);
      if (m > best && v + 64 * i < vfull) {  // a tie keeps the earlier vector
        best = m;
        bi = v + 64 * i;
      }
    }
    const bool row_end = c + 1 == A.S;
    if (row_end || !more) {
      // the partial vector at the row's end
      if (row_end && vfull < (int)A.nvec && (vfull & 63) == lane) {
        float z[E];
        Vt::load(p, vfull, A.V, z);
        const float m = max_elems(z);
        if (m > best || bi == INT_MAX) {
          best = m;
          bi = vfull;
        }
      }
      wave_max<true>(best, bi);
      const uint32_t tag = (uint32_t)__builtin_amdgcn_readfirstlane((int)tag_of_epoch(e0));
      const uint32_t first = (uint32_t)((g * R + r) * A.S);  // the row's first unit
      if (lane == 0) {
        uint64_t* w = A.words + (((int64_t)g * R + r) * A.pieces +
                                 (wave - (int)fdiv(first, A.div_span))) * 2;
        put_word(w, word_of(best, tag));
        put_word(w + 1, word_of(bi, tag));
      }
      if ((row_end && r + 1 == R) || !more) {
        // arrival: the last of the group's waves folds it. The words carry tags, so the count
        // needs no ordering against them: one still under way is waited for (bounded)
        const uint32_t gu = (uint32_t)(g * R * A.S);
        const uint32_t waves = fdiv(gu + (uint32_t)(R * A.S) - 1u, A.div_span) -
                               fdiv(gu, A.div_span) + 1u;
        uint32_t n = 0;
        if (lane == 0) n = tagged_add(A.arrived + g, tag, kOpenPolls);
        if ((uint32_t)__builtin_amdgcn_readfirstlane((int)n) == waves - 1u)
          mark = fold_group<DT>(A, g, tag, lane);
      }
      best = -INFINITY;
    }
    if (!more) return false;
    ++u;
    if (row_end) {
      c = 0;
      if (++r == R) {
        r = 0;
        ++g;
      }
      p = row_ptr<DT>(A, r, g);
      bi = lane < (int)A.nvec ? lane : INT_MAX;
    } else {
      ++c;
    }
    return true;
  };
  Raw x[kStep], y[kStep];
  load(x, true);
  {  // the counts of the groups that begin in this span (and the first wave: the groups')
    const uint32_t tag = (uint32_t)__builtin_amdgcn_readfirstlane((int)tag_of_epoch(e0));
    const int end = (int)fdiv((uint32_t)(uend - 1), A.div_group);
    const bool begins = u == g * R * A.S;
    if (u == 0 && lane == 63) open_count(A.finished, tag);
    for (int i = (begins ? g : g + 1) + lane; i <= end; i += 64) open_count(A.arrived + i, tag);
  }
  for (;;) {  // unrolled by two so that the register buffers alternate without copies
    if (!step(x, y)) break;
    if (!step(y, x)) break;
  }
  if (mark) mark_all(A, lane);
}

}  // namespace

int launch_argmax(const TeamGeom& g, const RowTable& rows, uint8_t* agree, int32_t* argmax_t,
                  int32_t* argmax_d, uint32_t polls, char* ws, hipStream_t stream) {
  const TeamWs L = team_ws(g);
  ArgmaxArgs A{};
  A.N = g.N;
  A.K = g.K;
  A.G = g.G;
  A.V = g.V;
  A.nvec = g.nvec;
  const ArgmaxPlan p = argmax_plan(g);
  A.S = p.S;
  A.total = (int)p.total;
  A.span = (int)p.span;
  A.pieces = (int)p.pieces;
  A.div_group = make_fastdiv((uint32_t)p.per_group);
  A.divS = make_fastdiv((uint32_t)A.S);
  A.divK = make_fastdiv((uint32_t)g.K);
  A.div_span = make_fastdiv((uint32_t)A.span);
  A.epoch = reinterpret_cast<uint32_t*>(ws + L.epoch);
  A.fail = reinterpret_cast<uint64_t*>(ws + L.epoch + 8);
  A.polls = polls;
  A.finished = reinterpret_cast<uint64_t*>(ws + L.epoch + 24);
  // the region of the team kernel's slice words: a row has at most as many pieces
  // as units, and no more units than slices (a slice is four wave loads), of three words each
  A.words = reinterpret_cast<uint64_t*>(ws + L.stat);
  A.arrived = reinterpret_cast<uint64_t*>(ws + L.arrived());
  A.argmax_t = argmax_t;
  A.argmax_d = argmax_d;
  A.agree = agree;
  A.rows = rows;
  const int64_t waves = (A.total + A.span - 1) / A.span;
  const unsigned grid = (unsigned)((waves + kWaves - 1) / kWaves);
  if (g.dtype == HS_F32) hs_argmax_kernel<HS_F32><<<grid, kThreads, 0, stream>>>(A);
  else if (g.dtype == HS_F16) hs_argmax_kernel<HS_F16><<<grid, kThreads, 0, stream>>>(A);
  else hs_argmax_kernel<HS_BF16><<<grid, kThreads, 0, stream>>>(A);
  return hipGetLastError() == hipSuccess ? HS_OK : HS_ERR_HIP;
}

}  // namespace hs
