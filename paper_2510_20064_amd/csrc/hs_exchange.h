// Shared by the evaluation kernels whose workgroups exchange results: the call's tag, counts and
// bounded waits on tagged words, and the argmax of a vector of logits.
#pragma once

#include "hs_wave.h"

namespace hs {

constexpr int kPollSleep = 2;  // s_sleep units (64 clocks) between polls

// (a vector load: a scalar one would hold up the kernel-argument loads waited on with it)
__device__ inline uint32_t call_tag(const uint32_t* epoch) {
  const uint32_t e =
      __hip_atomic_load(const_cast<uint32_t*>(epoch), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)tag_of_epoch(e));
}

// Adds 1 to the count that the word w keeps for the call with this tag and returns the
// count before (0 for the first add of a call): the word holds (count << 32) | tag, and a
// word with another tag, from an earlier call or never written, counts as 0. So nothing has
// to be reset between calls, and whatever a word held before cannot skew this call's count.
// Once the word carries the call's tag, an add is a single fetch-and-add, which leaves the tag
// half alone and costs every adder one round trip however many add at once. The tag gets there
// beforehand: the control block's count is left at (0 << 32) | the next call's tag by the call
// that completes it; a count anywhere else must not be (another shape keeps other words there,
// which would then look current), and is opened by one wave of the call itself (open_count).
// An add that finds another tag polls for the opening up to `polls` times (its own add went to
// the stale word, which the opening replaces as a whole) and then adds again, or goes on by
// compare-and-swap: the first exchange replaces the whole word, so every adder is counted once,
// by its fetch-and-add on the open word or by its exchange. (Looking at the word before the add
// instead makes every add two operations on it, which queue: 24 groups of 142 adders took
// 114 us for 68.)
__device__ inline uint32_t tagged_add(uint64_t* w, uint32_t tag, uint32_t polls = 0) {
  auto add = [&]() {
    return __hip_atomic_fetch_add(w, 1ull << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  uint64_t cur = add();
  if ((uint32_t)cur == tag) return (uint32_t)(cur >> 32);
  cur = get_word(w);
  for (uint32_t n = 0; n < polls && (uint32_t)cur != tag; ++n) {
    __builtin_amdgcn_s_sleep(kPollSleep);
    cur = get_word(w);
  }
  if ((uint32_t)cur == tag) return (uint32_t)(add() >> 32);  // the tag stays for the call
  for (;;) {  // each failed exchange means another add succeeded: this ends
    const uint32_t n = (uint32_t)cur == tag ? (uint32_t)(cur >> 32) : 0u;
    uint64_t expect = cur;
    if (__hip_atomic_compare_exchange_strong(w, &expect, ((uint64_t)(n + 1u) << 32) | tag,
                                             __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT))
      return n;
    cur = expect;
  }
}

// Opens the count at w for the call with this tag, if no adder has done so yet.
__device__ inline void open_count(uint64_t* w, uint32_t tag) {
  uint64_t cur = get_word(w);
  while ((uint32_t)cur != tag &&  // each failed exchange means an add succeeded: this ends
         !__hip_atomic_compare_exchange_strong(w, &cur, (uint64_t)tag, __ATOMIC_RELAXED,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
  }
}

// The word at w once it carries tag (its taint mark, if any, kept). Bounded: after `polls`
// polls, or as soon as another wait of this call has given up, the value is 0xFFFFFFFE (a NaN
// as float, -2 as int), tainted; the first wait to give up raises the call's fail flag, so one
// lost word costs one time-out, not one per wait. polls = 0 (set from the host, to test the
// failure path) makes every wait give up at once.
template <typename ARGS>
__device__ inline uint64_t await_word(const uint64_t* w, uint32_t tag, const ARGS& A) {
  constexpr uint64_t kLost = (0xFFFFFFFEull << 32) | kTaint;
  if (A.polls == 0) {
    put_word(A.fail, word_of(1, tag));
    return kLost | tag;
  }
  uint64_t v = get_word(w);
  for (uint32_t n = 1; tag_of(v) != tag; ++n) {
    if (n >= A.polls) {
      put_word(A.fail, word_of(1, tag));
      return kLost | tag;
    }
    if ((n & 255) == 0 && (uint32_t)get_word(A.fail) == tag) return kLost | tag;
    __builtin_amdgcn_s_sleep(kPollSleep);
    v = get_word(w);
  }
  return v;
}

// Largest of a thread's logits of one row, NaN ignored (-inf when there is no other), -0 as +0.
// v_maximum3_f32 takes two logits per instruction and returns NaN when it meets one, whatever
// its payload; such a lane then takes the slow way.
__device__ __forceinline__ float maximum3(float a, float b, float c) {
  float r;
  asm("v_maximum3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
template <int E>
__device__ __forceinline__ float max_elems(const float (&z)[E]) {
  float m = maximum3(z[0], z[1], z[2]);
#pragma unroll
  for (int e = 3; e < E; e += 2) m = maximum3(m, z[e], e + 1 < E ? z[e + 1] : z[e]);
  if (m != m) {
    m = -INFINITY;
#pragma unroll
    for (int e = 0; e < E; ++e) m = z[e] > m ? z[e] : m;
  }
  return m + 0.0f;
}

// Lowest index of a logit equal to m in 16-byte vector vi of the row at p (m the vector's maximum; -inf:
// the vector's first logit). The waves of the streaming argmax kernel exchange the vector that holds
// their maximum and the fold reads that one vector, so that no thread tracks an element index along
// its logits (three instructions per logit, where taking the maximum costs half of one).
template <int DT>
__device__ __forceinline__ int argmax_element(const char* p, int64_t V, int64_t nvec, float m,
                                              int vi) {
  using Vt = Vec<DT>;
  constexpr int E = Vt::kElems;
  if (vi < 0 || vi >= nvec) return -2;  // computed from a lost word
  float z[E];
  Vt::load(p, vi, V, z);
  int e = 0;
#pragma unroll
  for (int i = E - 1; i >= 0; --i)
    if (z[i] == m) e = i;
  return vi * E + (m > -INFINITY ? e : 0);
}

}  // namespace hs
