// Device helpers shared by the gfx950 kernels: fixed-order lane reductions,
// the tagged-word and bulk exchanges between workgroups of a persistent
// launch, an LDS-only workgroup barrier and the gate nonlinearities.
#pragma once

#include "kernels.hpp"

namespace alstm {

namespace {

constexpr int kWaves = kThreads / 64;
constexpr unsigned kSpinLimit = 1u << 21;   // about a second at the polling interval below
constexpr int kGatherSlots = 8;             // tagged words per thread per gather pass

// Sum over aligned groups of S lanes (S = 1, 2, 4, 8, 16) with DPP lane
// moves: quad swaps (xor 1, xor 2), then half-row and row mirrors.  Every
// lane of a group ends with the group's sum; the association order is fixed.
template <int S>
__device__ __forceinline__ float group_sum(float v) {
  if constexpr (S >= 2)
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false));
  if constexpr (S >= 4)
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, false));
  if constexpr (S >= 8)
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, false));
  if constexpr (S >= 16)
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xF, 0xF, false));
  return v;
}

// the same for S = 1, 4, 8 or 16 (uniform; lanes_for_level gives no other)
__device__ __forceinline__ float group_sum_rt(float v, int S) {
  if (S == 1) return v;
  v = group_sum<4>(v);
  if (S == 4) return v;
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, false));
  if (S == 8) return v;
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xF, 0xF, false));
  return v;
}

// Full-wave sum (input projection): 16-lane rows, then (r0 + r1) + (r2 + r3)
// over the four row sums, read into scalar registers (v_readlane: no LDS
// round trip, unlike a cross-row lane shuffle).  The result is uniform.
__device__ __forceinline__ float wave_sum(float v) {
  v = group_sum<16>(v);
  const int b = __builtin_bit_cast(int, v);
  const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0));
  const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16));
  const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32));
  const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
  return (r0 + r1) + (r2 + r3);
}

__device__ __forceinline__ void publish(unsigned long long* p, float v, unsigned tag) {
  unsigned long long w = ((unsigned long long)tag << 32) | (unsigned long long)__float_as_uint(v);
  __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long load_tagged(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Gather of tagged exchange words by threads tid < nthr: word i (< n) lands
// at dst[map ? map[i] : i] once it carries `tag`.  Each thread keeps two
// generations of loads of its words in flight (re-issued unconditionally, so
// the in-order completion counter lets one generation be consumed while the
// next travels), which halves the delay between a word's arrival and its
// detection.  Bounded: past the spin limit, or once another wait has failed,
// it records the failure and stores 0.
template <int NS>
__device__ void gather_tagged(float* dst, const uint16_t* map, const unsigned long long* src, int n, unsigned tag,
                              unsigned* err, int tid, int nthr) {
  for (int base = 0; base < n; base += nthr * NS) {
    const unsigned long long* sp[NS];
    unsigned pending = 0;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const int i = base + k * nthr + tid;
      sp[k] = src + (i < n ? i : 0);
      if (i < n) pending |= 1u << k;
    }
    unsigned long long wa[NS], wb[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) wa[k] = load_tagged(sp[k]);
    __builtin_amdgcn_s_sleep(4);
#pragma unroll
    for (int k = 0; k < NS; ++k) wb[k] = load_tagged(sp[k]);
    unsigned spins = 0;
    while (true) {
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (((pending >> k) & 1u) && (unsigned)(wa[k] >> 32) == tag) {
          const int i = base + k * nthr + tid;
          dst[map ? map[i] : i] = __uint_as_float((unsigned)wa[k]);
          pending &= ~(1u << k);
        }
      }
      if (!pending) break;
#pragma unroll
      for (int k = 0; k < NS; ++k) wa[k] = load_tagged(sp[k]);
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (((pending >> k) & 1u) && (unsigned)(wb[k] >> 32) == tag) {
          const int i = base + k * nthr + tid;
          dst[map ? map[i] : i] = __uint_as_float((unsigned)wb[k]);
          pending &= ~(1u << k);
        }
      }
      if (!pending) break;
#pragma unroll
      for (int k = 0; k < NS; ++k) wb[k] = load_tagged(sp[k]);
      spins += 2;
      if ((spins & 254u) == 0u &&
          (spins >= kSpinLimit || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)) {
        __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int k = 0; k < NS; ++k)
          if ((pending >> k) & 1u) {
            const int i = base + k * nthr + tid;
            dst[map ? map[i] : i] = 0.0f;
          }
        break;
      }
    }
  }
}

// Bulk h exchange.  The publisher wave stores its h values with agent-scope
// (sc1, write-through) stores, waits until the wave's stores are acknowledged
// (vmcnt 0), then stores its tag in its flag word.  Readers poll every workgroup's flag, then
// read the whole h_t with agent-scope 16-byte loads; coherent across XCDs
// without any cache writeback or invalidation.
__device__ __forceinline__ void store_coherent(float* p, float v) {
  __hip_atomic_store(reinterpret_cast<unsigned*>(p), __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 1 when flag word w carries `tag` or a later timestep's tag of the same
// launch (tag = launch sequence << 16 | timestep + 1)
__device__ __forceinline__ bool flag_reached(unsigned w, unsigned tag) {
  return (w >> 16) == (tag >> 16) && (w & 0xFFFFu) >= (tag & 0xFFFFu);
}

// threads tid < nthr poll flags [0, P) until each has reached `tag` (bounded)
__device__ __forceinline__ void await_flags(const unsigned* flag, int P, unsigned tag, unsigned* err, int tid,
                                            int nthr) {
  for (int f = tid; f < P; f += nthr) {
    unsigned spins = 0;
    while (!flag_reached(__hip_atomic_load(flag + f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), tag)) {
      __builtin_amdgcn_s_sleep(2);
      if ((++spins & 255u) == 0u &&
          (spins >= kSpinLimit || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)) {
        __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
    }
  }
}

// dst[i] = src[i] for i < n (src 16-byte aligned, readable up to n rounded up
// to 4), agent-scope loads, 4 in flight per thread
__device__ __forceinline__ void read_coherent(float* dst, const float* src, int n, int tid, int nthr) {
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  // the buffer descriptor must be wave-uniform (scalar registers)
  const unsigned long long addr = reinterpret_cast<unsigned long long>(src);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)addr);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(addr >> 32));
  const int n4 = __builtin_amdgcn_readfirstlane((n + 3) >> 2);
  float* base = reinterpret_cast<float*>(((unsigned long long)hi << 32) | lo);
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(base, (short)0, n4 * 16, 0x00020000);
  for (int base = 0; base < n4; base += 4 * nthr) {
    f32x4_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i4 = base + u * nthr + tid;
      v[u] = __builtin_amdgcn_raw_buffer_load_b128(rs, (i4 < n4 ? i4 : 0) * 16, 0, 16 /* sc1 */);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i4 = base + u * nthr + tid;
      if (i4 < n4)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (4 * i4 + c < n) dst[4 * i4 + c] = v[u][c];
    }
  }
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Slot exchange between the workgroups of a group.  A slot holds this pattern
// (a NaN that publish_slot never stores) until its value is there, so that
// every 4-byte value tells by itself whether it has arrived and a poll takes
// four of them with one load.  A slot exists once for each timestep that may
// be under way; its owner empties it when everyone is past reading it, before
// anyone can poll it again.
constexpr unsigned kEmpty = 0xFFFFFFFFu;

// Stores of the exchange: plain (the L2 of the group's XCD) when the whole
// group sits on one XCD, agent scope otherwise.
__device__ __forceinline__ void store_slot(float* p, unsigned bits, bool near) {
  unsigned* q = reinterpret_cast<unsigned*>(p);
  if (near) __hip_atomic_store(q, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(q, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish_slot(float* p, float v, bool near) {
  const unsigned bits = __float_as_uint(v);
  store_slot(p, bits == kEmpty ? 0x7FC00000u : bits, near);
}

// Poll the 16-byte units tid + stride r of src (uniform; `bytes` long) whose bit
// r is set in `pending` until none of their slots is empty; unit r goes to
// dst + map[r] (LDS, 16-byte aligned).  Agent-scope loads pass the L1 by.  The
// first round loads every unit without a branch, so that each is looked at
// as it arrives (kFirst; for many units across XCDs it comes too early and only
// delays the next: see exact_wide_kernel); later rounds load what is missing.  Bounded: past the spin
// limit, or once another wait has failed, the failure is recorded and the
// missing values read 0.
template <int kUnits, bool kFirst = true>
__device__ __forceinline__ void poll_units(float* dst, const float* src, int bytes, const int* map, unsigned pending,
                                           unsigned* err, int stride = kThreads) {
  if (!pending) return;
  const unsigned long long addr = reinterpret_cast<unsigned long long>(src);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)addr);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(addr >> 32));
  void* base = reinterpret_cast<void*>(((unsigned long long)hi << 32) | lo);
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(base, (short)0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
  const int tid = threadIdx.x;
  auto load = [&](int r) {
    return __builtin_amdgcn_raw_buffer_load_b128(rs, (tid + stride * r) * 16, 0, 16 /* sc1 */);
  };
  // empty is the largest unsigned value
  auto full = [](const u32x4& w) { return max(max(w[0], w[1]), max(w[2], w[3])) != kEmpty; };
  if constexpr (kFirst) {
    u32x4 w[kUnits];
#pragma unroll
    for (int r = 0; r < kUnits; ++r) w[r] = load(r);   // past the end: zeros, not looked at
#pragma unroll
    for (int r = 0; r < kUnits; ++r)
      if (((pending >> r) & 1u) && full(w[r])) {
        *reinterpret_cast<u32x4*>(dst + map[r]) = w[r];
        pending &= ~(1u << r);
      }
  }
  unsigned spins = 0;
  while (pending) {
    asm volatile("" ::: "memory");   // the loads of this round are new ones
    u32x4 w[kUnits];
#pragma unroll
    for (int r = 0; r < kUnits; ++r)
      if ((pending >> r) & 1u) w[r] = load(r);
#pragma unroll
    for (int r = 0; r < kUnits; ++r)
      if (((pending >> r) & 1u) && full(w[r])) {
        *reinterpret_cast<u32x4*>(dst + map[r]) = w[r];
        pending &= ~(1u << r);
      }
    if ((++spins & 255u) == 0u && pending &&
        (spins >= kSpinLimit || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)) {
      __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int r = 0; r < kUnits; ++r)
        if ((pending >> r) & 1u) *reinterpret_cast<u32x4*>(dst + map[r]) = u32x4{0u, 0u, 0u, 0u};
      break;
    }
  }
}

// this wave's loads and stores have completed
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// How a group starts: all present (on one XCD, or not), one workgroup alone,
// or nothing left to do here.
enum StartMode { kNear = 0, kFar = 1, kAlone = 2, kLeave = 3 };

// A group's decision: the launch's tag and one of these.
enum StartOutcome : unsigned { kEveryoneGoes = 1, kOneAlone = 2 };

// One lane: the group's outcome if it is already there (of this launch), else
// 0, and then it is `mine` from here on.
__device__ __forceinline__ unsigned decide_start(unsigned long long* decide, unsigned tag, StartOutcome mine) {
  unsigned long long seen = 0ull;   // as cleared
  do {                              // (twice at most, past a decision of another launch)
    if (__hip_atomic_compare_exchange_strong(decide, &seen, ((unsigned long long)tag << 32) | mine, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      return 0u;
  } while ((unsigned)(seen >> 32) != tag);
  return (unsigned)seen;
}

// The start of a group, run by one wave of each of its P workgroups:
// workgroup j's word gets (tag, XCD id), the lanes wait for everyone's words.
// The decision of the group is (tag, StartOutcome).  Words and decisions of
// other launches carry other tags and are as good as empty, so nothing is
// cleared at the end of a run, when some workgroup may still be looking; a
// launch whose tag may have been used before (a replay of a captured one, or
// after the sequence has wrapped) has the words cleared by the kernel before it
// on its stream (clear_start_words).  Bounded: `wait_ticks` (0: one workgroup
// alone in any case), and past a decision that everyone goes the spin limit.
__device__ int group_start(unsigned long long* hand, unsigned long long* decide, int j, int P, unsigned tag,
                           unsigned wait_ticks, unsigned* err) {
  const int lane = threadIdx.x & 63;
  unsigned xcc;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
  xcc &= 15u;
  if (lane == 0)
    __hip_atomic_store(hand + j, ((unsigned long long)tag << 32) | xcc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned long long t0 = wall_clock64();
  bool same = true, late = false;
  unsigned spins = 0;
  while (true) {
    // words lane, lane + 64, ... of the group at once (one after the other took
    // 3 us longer for 250 workgroups)
    unsigned long long w[kSpreadWords / 64];
#pragma unroll
    for (int k = 0; k < kSpreadWords / 64; ++k)
      if (64 * k < P) w[k] = load_tagged(hand + min(lane + 64 * k, P - 1));
    bool all = true;
    same = true;
#pragma unroll
    for (int k = 0; k < kSpreadWords / 64; ++k)
      if (64 * k < P) {
        all = all && (unsigned)(w[k] >> 32) == tag;
        same = same && (unsigned)w[k] == xcc;
      }
    if (__all(all) && wait_ticks != 0) break;
    if (!late && (wall_clock64() - t0 >= (unsigned long long)wait_ticks ||
                  load_tagged(decide) == (((unsigned long long)tag << 32) | kOneAlone))) {
      // one outcome for the whole group: whoever swaps first decides
      late = true;
      unsigned seen = 0u;
      if (lane == 0) seen = decide_start(decide, tag, kOneAlone);
      seen = __builtin_amdgcn_readfirstlane(seen);
      if (seen != kEveryoneGoes) return seen == 0u ? kAlone : kLeave;
      // someone saw everyone: all are resident, their words are coming
    }
    if (late && ++spins >= kSpinLimit) {
      if (lane == 0) __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return kLeave;
    }
  }
  if (!late) {
    // workgroup 0 decides for everyone, the others look (250 swaps of one word
    // take 5 us); it is there, so the decision is coming
    unsigned seen = 0u;
    if (j == 0) {
      if (lane == 0) seen = decide_start(decide, tag, kEveryoneGoes);
    } else if (lane == 0) {
      unsigned long long w = load_tagged(decide);
      for (; (unsigned)(w >> 32) != tag && spins < kSpinLimit; ++spins) w = load_tagged(decide);
      seen = (unsigned)(w >> 32) == tag ? (unsigned)w : kOneAlone;
      if ((unsigned)(w >> 32) != tag) __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (__builtin_amdgcn_readfirstlane(seen) == kOneAlone) return kLeave;
  }
  return __all(same) ? kNear : kFar;
}

// Clears `n` start words (null: none) for the next kernel of the stream, in the
// last workgroup of the grid, which is launched for that alone: true there.
// (Beside a workgroup's own work its loads or its end would wait for the stores.)
__device__ __forceinline__ bool clear_start_words(unsigned long long* ctl, int n) {
  if (!ctl || blockIdx.x != gridDim.x - 1) return false;
  for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x) ctl[i] = 0ull;
  return true;
}

// Workgroup barrier that orders LDS only.  __syncthreads() would also wait
// for every outstanding global store of the wave (gfx9 counts stores in
// vmcnt), i.e. for the agent-scope exchange stores to reach memory.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Gate nonlinearities from the exponential: sigmoid(z) = 1/(1+e^-z) and
// tanh(x) = 2 sigmoid(2x) - 1, with the hardware exp2 and reciprocal
// (relative error ~1e-6 for |z| < 20, exact limits 0 and 1 beyond).
__device__ __forceinline__ float sigmoid_fast(float z) {
  return __builtin_amdgcn_rcpf(1.0f + __expf(-z));
}

__device__ __forceinline__ float tanh_fast(float x) {
  return __builtin_fmaf(2.0f, sigmoid_fast(2.0f * x), -1.0f);
}

// A gate's value from its pre-activation: tanh for the cell candidate,
// sigmoid for the others (one exponential and one reciprocal either way).
__device__ __forceinline__ float gate_value(float y, bool candidate) {
  const float s = sigmoid_fast(candidate ? 2.0f * y : y);
  return candidate ? __builtin_fmaf(2.0f, s, -1.0f) : s;
}

// The cell update of Sec. II from the four gate pre-activations (rows i, f,
// g, o): c' = sigmoid(y_f) c + sigmoid(y_i) tanh(y_g), h = sigmoid(y_o)
// tanh(c').  Every kernel takes it from here, with its one fused
// multiply-add written out, so that the rounding never depends on how a
// kernel's surrounding code lets the compiler contract the expression.
__device__ __forceinline__ void cell_from_gates(float gi, float gf, float gg, float go, float& c, float& h) {
  c = __builtin_fmaf(gf, c, gi * gg);
  h = go * tanh_fast(c);
}

__device__ __forceinline__ void cell_update(float yi, float yf, float yg, float yo, float& c, float& h) {
  cell_from_gates(sigmoid_fast(yi), sigmoid_fast(yf), tanh_fast(yg), sigmoid_fast(yo), c, h);
}

}  // namespace

}  // namespace alstm
