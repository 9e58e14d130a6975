// gfx950 recurrence of the progressive approximate LSTM (arXiv 1905.00689:
// Sec. III Eq. (1) per gate, then the Sec. II cell update) with every factor
// slice in registers: each (level, sequence) pair of a run is its own
// recurrence, computed by a group of P workgroups of 512 threads.
//
// Workgroup j of a group owns up to OM consecutive slots of the z exchange (a
// slot is one term; the slots go lane by lane of a U row, see slot_tau) and up
// to RU consecutive hidden units (share_of, at least one of each): the h-part
// entries of its terms (16 lanes per term, one or two passes) and the U entries
// of its units' four gate rows (S lanes per row, one, two or four rows per thread) stay in registers for the
// whole sequence, P_x of every timestep (input_proj_kernel) in LDS.  Per
// timestep:
//   phase A  each term's lane group sums its h-part entries against h_{t-1}
//            (LDS), reduces over its 16 lanes, forms z = sigma * (P_x + s)
//            and stores it into its exchange slot;
//   z        every thread polls its share of the slots into LDS, four values
//            to a load;
//   phase B  each row's lanes sum u * z over their terms and reduce; the four
//            gate rows of a unit lie in one wave (rows gate-minor), whose
//            lanes apply the gate nonlinearities and the c/h update and store
//            h into its exchange slot and to h_out;
//   h        every thread polls its share of the units' h into LDS.
// With one workgroup (P = 1) nothing is exchanged: z and h go through LDS
// (H = 64, K = 16, T = 100: 1.08 -> 0.76 us per timestep, once the rows applied
// their own gates' nonlinearities and no wait for LDS was one for h_out).
//
// What bounds a timestep is the latency of its two exchanges.  Two things
// make them short:
// * Near groups.  Between workgroups of one XCD a word stored with a plain
//   store is in the L2 they share, and an agent-scope load (which passes the
//   L1 by) finds it there: 0.7-0.85 us for a probe's all-to-all round of 32
//   workgroups (2 to 16 64-bit words each) on MI355X, against 1.3-1.7 us with
//   agent-scope stores between XCDs.  So a group of up to kNearWidth
//   workgroups is placed on one XCD: consecutive blocks go to the XCDs in
//   turn, so group g is the blocks b with b % kXcds == g, and up to kXcds
//   pairs run side by side, one XCD each.  The placement is not assumed:
//   every workgroup tells the others its XCD id once at the start, and a
//   group found on several XCDs uses agent-scope stores.
// * Slots that tell by themselves whether their value has arrived (kEmpty), so
//   that a 16-byte load polls four values: half the bytes of (value, tag)
//   words and a quarter of the loads.
// Driving shape (D = 2048, H = 512, 75% pruning, T = 16, one sequence), whole
// run, us, with tagged words across XCDs / near groups with tagged words /
// near groups with slots: K = 32 75.2 / 60.3 / 36.5, K = 128 76.9 / 63.2 /
// 39.4, K = 512 87.5 / 92.3 / 63.4; phases at K = 64 (A, z, B, h) 0.25, 1.31,
// 0.70, 1.69 -> 0.35, 0.38, 0.38, 0.48 us.  Several pairs, against the general
// kernel's one launch for all of them: eight sequences at K = 128 389 -> 51,
// levels 16, 64, 128, 192 202 -> 46; H = 2048, K = 64, T = 64, eight sequences
// 1505 -> 144; K = 256, T = 32 943 -> 140.
// * Spread groups (SPREAD; a single pair whose slices one XCD cannot hold).
//   Across XCDs a store's acknowledgement takes as long as the exchange, and a
//   wave's loads and stores retire in order, so a wave that polls after storing
//   waits for its own stores first.  There the last wave alone publishes, from
//   LDS, and the others only poll.  H = 1024, K = 512, 75% pruning, T = 32, on
//   128 workgroups: 175 us with tagged words and 185 with slots published by
//   every wave, 146 so; the driving shape without pruning, K = 512: 97, 105, 94.
//   Short sequences of one pair go there too (plan_pair).
//
// Residency.  A group's workgroups wait for each other, so all of them must
// be resident.  When another stream's kernels hold part of an XCD that may
// take time, and two such launches holding parts of one XCD would wait for
// each other.  The start of a group is therefore a bounded decision (group_start):
// once all have arrived they go ahead; a workgroup whose wait runs out first
// decides otherwise, takes the group's pairs alone (every slice read from memory,
// nothing exchanged) and the rest of the group leaves.  Both ways compute every
// sum in one order.
//
// The order of every sum is that of progressive_lstm_kernel (phase A: entry
// sla + 16k of the term's h part at lane sla, k ascending, then the 16-lane
// DPP reduction; phase B: term sl + S*k at lane sl, k ascending, then the
// S-lane reduction, then the bias), so the two kernels' outputs are bitwise
// equal; the launch shape never changes a result.
#include "kernels.hpp"
#include "device_common.hpp"

#include <algorithm>
#include <type_traits>

namespace alstm {

namespace {

// 16-byte units polled per thread and exchange (up to 4096 values).
constexpr int kMaxUnits = 2;

// Threads of a spread group's workgroup that poll (the last wave publishes).
constexpr int kSpreadPollers = kThreads - 64;

// Timestep stamps are kept in LDS (written out at the end) up to this many
// timesteps; beyond, they go straight to memory.
constexpr int kLdsStamps = 255;
constexpr int kStampFloats = 2 * (4 + 4 * kLdsStamps);

// LDS carve-up (floats): h [hpad], with stamps their block (8-byte aligned),
// the group's start mode [4], own z of this timestep [64] (spread groups), P_x [T][OM], the owned terms' places in their groups
// [64], z [G][zst], c [H] (of a
// workgroup that runs its pairs alone; own h of this timestep, spread groups)
// and per wave the gate pre-activations
// of its rows [opt][64 / S] (16-byte aligned).
struct PairLayout {
  int st, mode, px, nown, zs, cs, ys, total;
};
__host__ __device__ inline PairLayout pair_layout(const PairArgs& a) {
  PairLayout l;
  l.st = a.hpad;
  l.mode = l.st + (a.stamps ? kStampFloats : 0);
  l.px = l.mode + 4 + 64;
  l.nown = l.px + ((a.T * a.OMmax + 3) & ~3);
  l.zs = l.nown + 64;
  l.cs = l.zs + a.zfloats;
  l.ys = l.cs + a.hpad;
  l.total = l.ys + kThreads * a.opt;   // [8 waves][opt][64 / S], S >= 1
  return l;
}

// One pair by one workgroup, every slice read from memory: the sums of the
// register path in the same order.  z at its LDS place, c and h in LDS.
__device__ void run_alone(const PairArgs& a, int lev, int b, float* hs, float* zs, float* cs, float* ys) {
  const PairLevel& v = a.lv[lev];
  const int tid = threadIdx.x, H = a.H, G = a.G, T = a.T, TB = a.T * a.B, K = v.K, S = v.S, lgS = v.lgS;
  for (int i = tid; i < H; i += kThreads) {
    hs[i] = a.h0 ? a.h0[(size_t)b * H + i] : 0.0f;
    cs[i] = a.c0 ? a.c0[(size_t)b * H + i] : 0.0f;
  }
  __syncthreads();
  const int sub = tid >> 4, sla = tid & 15;
  const int rs = tid >> lgS, sl = tid & (S - 1), q = rs & 3;
  const int units = kThreads >> (lgS + 2);              // units per pass, their four rows gate-minor
  const int wv = tid >> 6, lane = tid & 63, rpw = 64 >> lgS;
  float* ysw = ys + wv * rpw;
  float* hout = a.h_out + ((size_t)lev * T * a.B + b) * H;
  // the first pair's stamps (nothing is waited for: the z wait ends as it starts)
  const bool stamp = a.stamps && lev == 0 && b == 0 && tid == 0;
  if (stamp) {
    a.stamps[0] = wall_clock64();
    a.stamps[1] = clock64();
  }
  for (int t = 0; t < T; ++t) {
    if (stamp) a.stamps[2 + 4 * t] = clock64();
    const int kt = a.sched ? a.sched[t] : K;
    for (int base = 0; base < G * K; base += kThreads / 16) {
      const int tau = base + sub;
      float acc = 0.0f;
      if (tau < G * kt) {
        const size_t src = (size_t)tau * a.NZ;
        for (int e = a.nx[tau] + sla; e < a.NZ; e += 16) acc += a.vval[src + e] * hs[(int)a.vidx[src + e] - a.D];
      }
      acc = group_sum<16>(acc);
      if (sla == 0 && tau < G * K) {
        const int g = tau % G, n = tau / G;
        zs[g * v.zst + (n & (S - 1)) * v.kst + (n >> lgS)] =
            tau < G * kt ? a.sigma[tau] * (a.px[(size_t)tau * TB + t * a.B + b] + acc) : 0.0f;
      }
    }
    __syncthreads();
    if (stamp) a.stamps[3 + 4 * t] = a.stamps[4 + 4 * t] = clock64();
    for (int u0 = 0; u0 < H; u0 += units) {
      const int u = u0 + (rs >> 2);
      float acc = 0.0f, bias = 0.0f;
      if (u < H) {
        const size_t row = (size_t)q * H + u;
        const float* urow = a.Ut + row * a.N;
        const float* z = zs + (G == 4 ? q : 0) * v.zst + sl * v.kst;
        for (int n = sl; n < K; n += S) acc += urow[n] * z[n >> lgS];
        bias = a.bias[row];
      }
      acc = group_sum_rt(acc, S) + bias;
      if (sl == 0) ysw[lane >> lgS] = acc;
      __syncthreads();
      if (lane < (rpw >> 2)) {
        const int uc = u0 + wv * (rpw >> 2) + lane;
        if (uc < H) {
          float c = cs[uc], h2;
          cell_update(ysw[4 * lane], ysw[4 * lane + 1], ysw[4 * lane + 2], ysw[4 * lane + 3], c, h2);
          cs[uc] = c;
          hs[uc] = h2;
          hout[(size_t)t * a.B * H + uc] = h2;
        }
      }
      __syncthreads();
    }
    if (stamp) a.stamps[5 + 4 * t] = clock64();
  }
  if (stamp) {
    a.stamps[2 + 4 * T] = clock64();
    a.stamps[3 + 4 * T] = wall_clock64();
  }
  if (a.c_out)
    for (int i = tid; i < H; i += kThreads) a.c_out[((size_t)lev * a.B + b) * H + i] = cs[i];
  __syncthreads();
}

// v, in a vector register and looked at again where it is used: a lane mask kept
// over the loop instead takes two scalar registers, and those of the loop are
// spilled already (a spilled mask comes back through v_readlane on the path
// between the cell update and its store: 3 us in 2 x 32 timesteps at H = 1024).
// Not where two workgroups share a compute unit, whose vector registers are the
// scarce ones (driving shape, K = 512: 67.4 us with it, 66.8 without).
__device__ __forceinline__ int in_register(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// OPT output rows per thread with UMAX U entries each in registers, APASS
// phase-A passes with HMAX h-part entries per lane each.  Every loop runs to
// its compile-time bound: entries past a lane's share are zeros (a U entry
// past the budget, an h-part slot past the term's count), whose products add
// nothing, so the sums equal those over the live entries in the same order.
// TWO: the instance keeps to 128 registers, so that two workgroups share a
// compute unit (near groups of more than 32 workgroups).
// SPREAD: the group of a single pair over more than one XCD.
template <int OPT, int UMAX, int APASS, int HMAX, bool TWO, bool SPREAD>
__global__ void __launch_bounds__(kThreads, TWO ? 4 : 2) pair_lstm_kernel(PairArgs a) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  constexpr int kChunk = 16;   // LDS reads in flight per batch
  // group of this workgroup and its place in it
  const int ng = a.groups;
  const int g = ng > 1 ? (int)((blockIdx.x + ng - a.first_xcd) % ng) : 0, j = blockIdx.x / ng;
  if (g >= a.L * a.B) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int D = a.D, H = a.H, G = a.G, N = a.N, NZ = a.NZ, T = a.T, B = a.B;
  const PairLayout lay = pair_layout(a);
  float* ldsf = reinterpret_cast<float*>(lds_raw);
  int* modes = reinterpret_cast<int*>(ldsf + lay.mode);
  float* pxs = ldsf + lay.px;      // P_x [T][OM]
  int* nown = reinterpret_cast<int*>(ldsf + lay.nown);
  float* zpub = ldsf + lay.mode + 4;   // own z of this timestep [64]
  float* hpub = ldsf + lay.cs;         // own h of this timestep [RU]
  float* hs = ldsf;                // h_{t-1} [H]
  float* zs = ldsf + lay.zs;       // z of this timestep [G][zst]
  const int wv = tid >> 6;

  // The group starts once, for the widest of its pairs: the last wave decides
  // while the others load the first pair's slices.
  int pg = 1;
  for (int lb = g; lb < a.L * B; lb += ng) {
    const PairLevel& v = a.lv[lb / B];
    if (v.K > 0) pg = max(pg, v.P);
  }
  const bool started = pg > 1 && j < pg;
  unsigned long long* hand = a.ctl + (size_t)g * kCtlWords;
  unsigned long long* decide = ng > 1 ? hand + kNearWidth : a.ctl + kSpreadWords;
  const size_t exf = 2 * ((size_t)a.zslots + a.hpad);   // floats of a pair's exchange: z [2][zslots], h [2][hpad]
  if (wv == kWaves - 1) {
    int mode = kFar;
    if (started) mode = group_start(hand, decide, j, pg, a.tag_base | 0xFFFFu, a.wait_ticks, a.err);
    if (lane == 0) modes[0] = mode;
  }

  bool near = false, seen_mode = false;
  for (int lb = g; lb < a.L * B; lb += ng) {
    const int lev = lb / B, b = lb - lev * B;
    const PairLevel& v = a.lv[lev];
    const int P = v.P, K = v.K, OM = v.OM, zst = v.zst, kst = v.kst, kpl = v.kpl;
    if (j >= P) continue;
    const bool local = P == 1 || K == 0;   // nothing exchanged
    const Share ho = share_of(H, P, j), zo = share_of(v.slots, P, j);
    // (divisions are vector work: back to scalar registers)
    const int r0 = __builtin_amdgcn_readfirstlane(ho.first), rc = __builtin_amdgcn_readfirstlane(ho.count);
    const int s0 = __builtin_amdgcn_readfirstlane(zo.first), n_owned = __builtin_amdgcn_readfirstlane(zo.count);
    const int S = __builtin_amdgcn_readfirstlane(v.S), lgS = __builtin_amdgcn_readfirstlane(v.lgS);
    // Slot w of the z exchange is entry k = w % kpl of lane sl of a row of group
    // g (w / kpl = g*S + sl), the term n = sl + S*k: a lane's terms are
    // consecutive, and so are a workgroup's slots [s0, s0 + n_owned).  In LDS
    // the entry sits at zs[g*zst + sl*kst + k].  tau < 0: no term (n >= K).
    auto slot_tau = [&](int w) {
      const int blk = w / kpl, n = (blk & (S - 1)) + S * (w - blk * kpl);
      return n < K ? n * G + (blk >> lgS) : -1;
    };
    auto slot_pos = [&](int w) {
      const int blk = w / kpl;
      return (blk >> lgS) * zst + (blk & (S - 1)) * kst + (w - blk * kpl);
    };
    if (lb != g) __syncthreads();   // the previous pair's LDS is done with

    // Prologue loads, ordered so that every independent load is in flight
    // before the first wait: the first share of P_x and h0, sigma and the
    // h/x split of the owned terms, the U entries, bias and c0; then the
    // h-part entries (their addresses need the split).
    const int npx = T * n_owned, TB = T * B;
    float px0 = 0.0f, h00 = 0.0f;
    if (tid < npx) {
      const int io0 = tid / T, tau = slot_tau(s0 + io0);
      if (tau >= 0) px0 = a.px[(size_t)tau * TB + (tid - io0 * T) * B + b];
    }
    if (tid < H && a.h0) h00 = a.h0[(size_t)b * H + tid];

    // ---- phase-A roles: lane group sub (16 lanes) takes owned terms sub + 32p
    const int sub = tid >> 4, sla = tid & 15;
    float hv[APASS][HMAX];
    int hi[APASS][HMAX];
    float sg[APASS];
    int e0v[APASS], tauv[APASS];
#pragma unroll
    for (int p = 0; p < APASS; ++p) {
      const int ia = sub + 32 * p;
      const int tau = ia < n_owned ? slot_tau(s0 + ia) : -1;
      tauv[p] = max(tau, 0);
      if (sla == 0) nown[ia] = tau >= 0 ? tau / G : K;
      sg[p] = tau >= 0 ? a.sigma[tau] : 0.0f;
      e0v[p] = tau >= 0 ? (int)a.nx[tau] : NZ;
    }

    // ---- phase-B roles: row slot rs = tid / S, rows rs + o * (512 / S); row ol
    // is gate q = ol & 3 of owned unit ol >> 2 (gate-minor: a unit's four rows
    // are four adjacent lane groups of one wave)
    const int rs = tid >> lgS, sl = tid & (S - 1);
    const int nslots = kThreads >> lgS;
    float uv[OPT][UMAX];
    float bq[OPT];
    // every row of a thread has gate q = rs & 3 (row slots per pass are a
    // multiple of 4): one z base for all of them
    const int zb = (G == 4 ? (rs & 3) : 0) * zst + sl * kst;
    const bool cand = (rs & 3) == 2;   // the cell candidate's rows: tanh
    int zown[APASS];                   // LDS places of the owned slots (one workgroup)
    int zput[APASS];                   // the slot that this lane publishes per pass, or -1
#pragma unroll
    for (int p = 0; p < APASS; ++p) {
      const bool own = sub + 32 * p < n_owned;
      zown[p] = own ? slot_pos(s0 + sub + 32 * p) : 0;
      zput[p] = own && sla == 0 ? s0 + sub + 32 * p : -1;
    }
    // ---- cell roles: a wave holds the rows of 16 * OPT / S units (row slots
    // [w * 64/S, (w+1) * 64/S) in each of the OPT passes); its lane cl takes
    // unit cl, pass co = cl / (16/S), row slots 4 ck .. 4 ck + 3 (ck = cl %
    // (16/S)), and keeps that unit's c in a register.  The rows' sums reach
    // it through the wave's LDS block ysw[o][64/S] (no cross-wave traffic).
    const int rpw = 64 >> lgS, upw = (16 * OPT) >> lgS;
    const int co = lane >> (4 - lgS), ck = lane & ((16 >> lgS) - 1);
    const int cunit = (wv * rpw + 4 * ck + co * nslots) >> 2;
    const bool cell_ok = lane < upw && cunit < rc;
    const int hput = cell_ok ? r0 + cunit : -1;   // the unit that this lane updates
    float cst = (cell_ok && a.c0) ? a.c0[(size_t)b * H + r0 + cunit] : 0.0f;
    float* ysw = ldsf + lay.ys + (size_t)wv * OPT * rpw;
#pragma unroll
    for (int o = 0; o < OPT; ++o) {
      const int ol = rs + o * nslots, ul = ol >> 2, q = ol & 3;
      const bool rowv = ul < rc;
      const size_t row = (size_t)q * H + r0 + ul;
      bq[o] = rowv ? a.bias[row] : 0.0f;
      const float* urow = a.Ut + (rowv ? row : 0) * N;
#pragma unroll
      for (int k = 0; k < UMAX; ++k) uv[o][k] = urow[max(0, min(sl + S * k, K - 1))];
#pragma unroll
      for (int k = 0; k < UMAX; ++k) uv[o][k] = (rowv && sl + S * k < K) ? uv[o][k] : 0.0f;
    }

#pragma unroll
    for (int p = 0; p < APASS; ++p) {
      const int e0 = e0v[p], cnt = NZ - e0;
      const size_t src = (size_t)tauv[p] * NZ;
      // every load issued (index clamped into the term's entries), then masked
#pragma unroll
      for (int k = 0; k < HMAX; ++k) {
        const int e = min(e0 + sla + 16 * k, NZ - 1);
        hv[p][k] = a.vval[src + e];
        hi[p][k] = (int)a.vidx[src + e];
      }
#pragma unroll
      for (int k = 0; k < HMAX; ++k) {
        const bool live = sla + 16 * k < cnt;
        hv[p][k] = live ? hv[p][k] : 0.0f;
        hi[p][k] = live ? 4 * (hi[p][k] - D) : 0;   // byte offset of h[k - D] in LDS
      }
    }

    // ---- exchange roles: 16-byte units tid + 512 r of z (a lane's slots are a
    // multiple of 4, so a unit's four go to consecutive LDS places) and of h
    int zdi[kMaxUnits], hdi[kMaxUnits];
    unsigned zpend = 0, hpend = 0;
    constexpr int pollers = SPREAD ? kSpreadPollers : kThreads;
#pragma unroll
    for (int r = 0; r < kMaxUnits; ++r) {
      const int u = tid + pollers * r;
      if (tid < pollers && 4 * u < v.slots) zpend |= 1u << r;
      if (tid < pollers && 4 * u < H) hpend |= 1u << r;
      zdi[r] = 4 * u < v.slots ? slot_pos(4 * u) : 0;
      hdi[r] = 4 * u;
    }
    float* zx = a.ex + lb * exf;
    float* hx = zx + 2 * a.zslots;

    // ---- LDS: initial state, P_x of every timestep
    if (tid < H) hs[tid] = h00;
    for (int i = tid + kThreads; i < H; i += kThreads) hs[i] = a.h0 ? a.h0[(size_t)b * H + i] : 0.0f;
    // z slots of terms past the budget (n >= K in a lane's last entry) are
    // never written and must read 0 (their u entries are 0 as well)
    for (int i = tid; i < a.zfloats; i += kThreads) zs[i] = 0.0f;
    if (tid < npx) pxs[(tid % T) * OM + tid / T] = px0;
    for (int i = tid + kThreads; i < npx; i += kThreads) {
      const int io = i / T, t = i - io * T, tau = slot_tau(s0 + io);
      pxs[t * OM + io] = tau >= 0 ? a.px[(size_t)tau * TB + t * B + b] : 0.0f;
    }
    __syncthreads();
    if (lb == g || !seen_mode) {
      const int mode = __builtin_amdgcn_readfirstlane(modes[0]);
      if (mode >= kAlone) break;   // the whole group's outcome: nothing of any pair has begun
      near = mode == kNear;
      seen_mode = true;
    }

    const bool stamp = a.stamps && lb == 0 && j == 0 && tid == 0;
    // stamps of short runs stay in LDS until the end (no stores on the way);
    // two plain stores rather than one through a generic pointer, after which
    // every wait for LDS would wait for outstanding memory stores too
    const bool lds_stamps = T <= kLdsStamps;
    auto put_stamp = [&](int i, unsigned long long v) {
      if (lds_stamps) reinterpret_cast<unsigned long long*>(ldsf + lay.st)[i] = v;
      else a.stamps[i] = v;
    };
    if (stamp) {
      put_stamp(0, wall_clock64());
      put_stamp(1, clock64());
    }
    // one loop for a single workgroup, one for a group on one XCD and one for a
    // spread group.  There a store's acknowledgement takes as long as the
    // exchange, and a wave's loads and stores retire in order: so the last wave
    // alone publishes (and stores h_out) and the others only poll.
    auto steps = [&](auto kind) {
      constexpr bool kLocal = decltype(kind)::value == 0, kSpread = decltype(kind)::value == 2;
      float* hout = a.h_out + ((size_t)lev * TB + b) * H + r0 + (kSpread ? 0 : cunit);
      const size_t hstep = (size_t)B * H;
      int kt = a.sched ? a.sched[0] : K;
      int half = 0;   // t & 1
      for (int t = 0; t < T; ++t, half ^= 1, hout += hstep) {
        float* zxt = zx + (half ? a.zslots : 0);
        float* zxe = zx + (half ? 0 : a.zslots);
        float* hxt = hx + (half ? a.hpad : 0);
        float* hxe = hx + (half ? 0 : a.hpad);
        if (stamp) put_stamp(2 + 4 * t, clock64());

        // ---- phase A: z = sigma * (P_x + prune(v)_h . h_{t-1}) ----
        float z[APASS], pxv[APASS];
#pragma unroll
        for (int p = 0; p < APASS; ++p) pxv[p] = pxs[t * OM + min(sub + 32 * p, OM - 1)];
#pragma unroll
        for (int p = 0; p < APASS; ++p) {
          float acc = 0.0f;
#pragma unroll
          for (int k0 = 0; k0 < HMAX; k0 += kChunk) {
            // the bound k0 + k < HMAX is a constant once unrolled (a last chunk
            // may be partial: HMAX = 24)
            float hg[kChunk];
#pragma unroll
            for (int k = 0; k < kChunk; ++k)
              if (k0 + k < HMAX) hg[k] = *reinterpret_cast<const float*>(lds_raw + hi[p][k0 + k]);
#pragma unroll
            for (int k = 0; k < kChunk; ++k)
              if (k0 + k < HMAX) acc += hv[p][k0 + k] * hg[k];
          }
          z[p] = sg[p] * (pxv[p] + group_sum<16>(acc));
        }
        if (a.sched) {
          // terms past this timestep's budget
#pragma unroll
          for (int p = 0; p < APASS; ++p)
            if (sub + 32 * p < n_owned && nown[sub + 32 * p] >= kt) z[p] = 0.0f;
          if (t + 1 < T) kt = a.sched[t + 1];   // on its way while the exchanges wait
        }
#pragma unroll
        for (int p = 0; p < APASS; ++p) {
          const int w = zput[p];
          if (w >= 0) {
            if constexpr (kLocal) {
              zs[zown[p]] = z[p];
            } else if constexpr (kSpread) {
              zpub[sub + 32 * p] = z[p];
            } else {
              publish_slot(zxt + w, z[p], near);
              // z_{t-1}: everyone's h_{t-1} is here, so everyone has read it
              store_slot(zxe + w, kEmpty, near);
            }
          }
        }
        if (stamp) put_stamp(3 + 4 * t, clock64());
        if constexpr (kSpread) {
          lds_barrier();
          if (wv == kWaves - 1) {
            wait_memory();   // the emptied h slots, before this workgroup's z_t
            if (lane < n_owned) {
              publish_slot(zxt + s0 + lane, zpub[lane], false);
              store_slot(zxe + s0 + lane, kEmpty, false);
            }
          }
          poll_units<kMaxUnits>(zs, zxt, a.zslots * 4, zdi, zpend, a.err, kSpreadPollers);
        } else if constexpr (!kLocal) {
          poll_units<kMaxUnits>(zs, zxt, a.zslots * 4, zdi, zpend, a.err);
          wait_memory();   // the emptied slots too, before this workgroup's h_t
        }
        lds_barrier();
        if (stamp) put_stamp(4 + 4 * t, clock64());

        // ---- phase B: y = b + sum_n u_n z_n, then the cell update ----
        float acc[OPT];
#pragma unroll
        for (int o = 0; o < OPT; ++o) acc[o] = 0.0f;
#pragma unroll
        for (int k0 = 0; k0 < UMAX; k0 += kChunk) {
          float4 z4[kChunk / 4];
#pragma unroll
          for (int k = 0; k < kChunk; k += 4)
            if (k0 + k < UMAX) z4[k / 4] = *reinterpret_cast<const float4*>(zs + zb + k0 + k);
#pragma unroll
          for (int o = 0; o < OPT; ++o)
#pragma unroll
            for (int k = 0; k < kChunk; k += 4)
              if (k0 + k < UMAX) {
                acc[o] += uv[o][k0 + k] * z4[k / 4].x;
                acc[o] += uv[o][k0 + k + 1] * z4[k / 4].y;
                acc[o] += uv[o][k0 + k + 2] * z4[k / 4].z;
                acc[o] += uv[o][k0 + k + 3] * z4[k / 4].w;
              }
        }
        // every row applies its own gate's nonlinearity (the four gates of a
        // unit side by side rather than one after the other in the unit's
        // lane), then the results go to the wave's block and each unit's lane
        // reads its four at once and updates c and h
#pragma unroll
        for (int o = 0; o < OPT; ++o) acc[o] = gate_value(group_sum_rt(acc[o], S) + bq[o], cand);
        if (sl == 0) {
#pragma unroll
          for (int o = 0; o < OPT; ++o) ysw[o * rpw + (lane >> lgS)] = acc[o];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const bool more = t + 1 < T;   // nobody reads the last timestep's h
        const int u = kLocal || TWO ? hput : in_register(hput);
        if (u >= 0) {
          const float4 g4 = *reinterpret_cast<const float4*>(ysw + co * rpw + 4 * ck);
          float h2;
          cell_from_gates(g4.x, g4.y, g4.z, g4.w, cst, h2);
          if constexpr (kLocal) {
            hs[u] = h2;
          } else if constexpr (kSpread) {
            hpub[cunit] = h2;
          } else if (more) {
            publish_slot(hxt + u, h2, near);
            // h_{t-1}: everyone's z_t is here, so everyone has read it
            store_slot(hxe + u, kEmpty, near);
          }
          if constexpr (!kSpread) *hout = h2;
        }
        if (stamp) put_stamp(5 + 4 * t, clock64());
        if constexpr (kSpread) {
          lds_barrier();
          if (wv == kWaves - 1) {
            wait_memory();   // the emptied z slots, before this workgroup's h_t
            for (int i = lane; i < rc; i += 64) {
              const float h2 = hpub[i];
              if (more) {
                publish_slot(hxt + r0 + i, h2, false);
                store_slot(hxe + r0 + i, kEmpty, false);
              }
              hout[i] = h2;
            }
          }
          if (more) poll_units<kMaxUnits>(hs, hxt, a.hpad * 4, hdi, hpend, a.err, kSpreadPollers);
        } else if constexpr (!kLocal) {
          if (more) {
            poll_units<kMaxUnits>(hs, hxt, a.hpad * 4, hdi, hpend, a.err);
            wait_memory();   // the emptied slots too, before this workgroup's z_{t+1}
          }
        }
        lds_barrier();
      }
    };
    if constexpr (SPREAD) steps(std::integral_constant<int, 2>{});
    else if (local) steps(std::integral_constant<int, 0>{});
    else steps(std::integral_constant<int, 1>{});
    if (stamp) {
      put_stamp(2 + 4 * T, clock64());
      put_stamp(3 + 4 * T, wall_clock64());
      if (lds_stamps)
        for (int i = 0; i < 4 + 4 * T; ++i) a.stamps[i] = reinterpret_cast<unsigned long long*>(ldsf + lay.st)[i];
    }
    if (a.c_out && cell_ok) a.c_out[((size_t)lev * B + b) * H + r0 + cunit] = cst;
  }
  if (!started) return;
  __syncthreads();
  const int mode = __builtin_amdgcn_readfirstlane(modes[0]);
  if (mode == kAlone) {
    for (int lb = g; lb < a.L * B; lb += ng) {
      for (int i = tid; i < a.zfloats; i += kThreads) zs[i] = 0.0f;
      __syncthreads();
      run_alone(a, lb / B, lb % B, hs, zs, ldsf + lay.cs, ldsf + lay.ys);
    }
  }
}

template <int OPT, int UMAX, int APASS, int HMAX, bool TWO, bool SPREAD>
hipError_t launch_pair_instance(const PairArgs& a, int P, size_t lds, hipStream_t stream) {
  static bool attr_set = false;
  const void* fn = (const void*)pair_lstm_kernel<OPT, UMAX, APASS, HMAX, TWO, SPREAD>;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsCap);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  pair_lstm_kernel<OPT, UMAX, APASS, HMAX, TWO, SPREAD><<<dim3(P * a.groups), dim3(kThreads), lds, stream>>>(a);
  return hipGetLastError();
}

template <int OPT, int UMAX, int APASS, int HMAX>
hipError_t launch_pair_kernel(const PairArgs& a, int P, size_t lds, hipStream_t stream) {
  // at most 128 registers where the slices are small (two workgroups per
  // compute unit, near groups of up to kNearWidth workgroups)
  constexpr bool kTwo = OPT == 1 && APASS == 1 && HMAX <= kTwoHmax;
  if (a.spread) return launch_pair_instance<OPT, UMAX, APASS, HMAX, false, true>(a, P, lds, stream);
  return launch_pair_instance<OPT, UMAX, APASS, HMAX, kTwo, false>(a, P, lds, stream);
}

// One level's launch shape on P workgroups, output rows per thread at most
// `optcap`; false when its slices do not fit the registers.
struct LevelShape {
  int apass, opt, need_h, upt;
};

// Four rows per thread with 17 to 32 U entries each (128 registers) leave room
// for 64 registers of h parts, and two phase-A passes of long h parts take them
// next to at most 64 of U: 24 entries per lane.  Near groups of 32 workgroups
// that hold this much: H = 2048, K = 256, 90% pruning, T = 32: 167 us on 128
// workgroups before, 113 now; the driving shape at 50% pruning, K = 512: 92 on
// 64 workgroups before, 79 now.  What is left out spilled
// inside the loop: two passes of 32 entries, 107 us on 32 workgroups against
// 97 on a spread group (driving shape, no pruning, K = 512); keeping two
// entries' places in one register cost more (115) than it saved.
bool in_registers(int opt, int upt, int apass, int need_h) {
  if (apass == 2 && need_h > 24) return false;
  return opt < 4 || upt <= 16 || need_h <= (apass == 2 ? 16 : 32);
}

bool level_fits(const PairArgs& a, PairLevel& v, int hcap, int P, int optcap, LevelShape& s) {
  const int OM = (v.slots + P - 1) / P, RU = (a.H + P - 1) / P;
  s.apass = OM <= 32 ? 1 : (OM <= 64 ? 2 : 0);
  s.need_h = (hcap + 15) / 16;             // h-part entries per lane
  s.upt = (v.K + v.S - 1) / v.S;           // U entries per row and lane
  // (two passes of long h parts on one workgroup cost more than an exchange)
  if (!s.apass || s.need_h > (s.apass == 2 && P == 1 ? 16 : 32)) return false;
  const int slots = kThreads / v.S;        // row slots per pass of the threads
  const int opt = (4 * RU + slots - 1) / slots;
  s.opt = opt <= 1 ? 1 : (opt <= 2 ? 2 : (opt <= 4 ? 4 : 0));
  if (!s.opt || s.opt > optcap || s.upt > 32) return false;
  if (!in_registers(s.opt, s.upt, s.apass, s.need_h)) return false;
  // the four gate rows of a unit must be adjacent lane groups of one wave
  if (4 * v.S > 64) return false;
  // Everyone owns slots and units.  A slot is emptied once everyone's values
  // that were computed from it are here (z_{t-1} once h_{t-1} is, h_{t-1} once
  // z_t is), and is polled again only once its owner's next value of the other
  // kind is here, which the owner publishes after the emptied slots are stored.
  // A workgroup without units, or without slots, would take part in neither.
  if (P > 1 && v.K > 0 && P > std::min(v.slots, a.H)) return false;
  if (v.slots > 4 * kMaxUnits * kThreads || a.H > 4 * kMaxUnits * kThreads) return false;
  v.P = P;
  v.OM = OM;
  v.RU = RU;
  return true;
}

// Width of one level (0: none up to `cap` fits); `quick`: of a short sequence
// over the device, where more workgroups load the slices sooner.
int level_width(const PairArgs& a, PairLevel& v, int hcap, int cap, int want, int optcap, bool quick, LevelShape& s) {
  if (want > 0) return want <= cap && level_fits(a, v, hcap, want, optcap, s) ? want : 0;
  if (level_fits(a, v, hcap, 1, optcap, s)) return 1;   // one workgroup: nothing exchanged
  // the exchanges cost about the same at 16 and at 32 workgroups (0.47 and
  // 0.50 us at K = 64), so take the narrowest width at which each thread has
  // one phase-A term group and one output row, else the narrowest that fits
  int P = 0;
  for (int p = 2; p <= cap && !P; ++p)
    if (level_fits(a, v, hcap, p, optcap, s) && s.apass == 1 && s.opt == 1) P = p;
  // beyond one workgroup per compute unit of an XCD, several rows per thread
  // cost less than the wider exchange as long as phase A keeps to one pass
  if ((P == 0 || (P > kXcdCus && !quick)) && kXcdCus <= cap && level_fits(a, v, hcap, kXcdCus, optcap, s) && s.apass == 1)
    P = kXcdCus;
  for (int p = 2; p <= cap && !P; ++p)
    if (level_fits(a, v, hcap, p, optcap, s)) P = p;
  if (!P) return 0;
  // a narrow layer: at least 16 workgroups from 17 terms per group and 32 from
  // 64, each keeping 16 rows or more (driving shape, us per run on 16 / 32 /
  // 64 workgroups: K = 32 40.8 / 41.1 / 48.2, K = 64 43.7 / 42.8 / 48.9,
  // K = 256 62.1 / 54.2 / 59.8)
  const int floor_p = std::min({v.K >= 64 ? 32 : (v.K > 16 ? 16 : 0), (4 * a.H) / 16, cap});
  if (P < floor_p && level_fits(a, v, hcap, floor_p, optcap, s)) return floor_p;
  return level_fits(a, v, hcap, P, optcap, s) ? P : 0;
}

// Shapes of every level with widths up to `cap` and up to `optcap` rows per
// thread, and the instance (register buckets) that holds them all.
int plan_levels(PairArgs& a, const int* hcap, int cap, int want, int optcap, bool quick) {
  int pmax = 0, need_h = 0, upt = 0;
  a.opt = a.apass = 1;
  a.OMmax = a.zslots = 0;
  bool quad = false;   // a level needs both four rows per thread and more than 16 U entries
  for (int l = 0; l < a.L; ++l) {
    PairLevel& v = a.lv[l];
    v.S = lanes_for_level(v.K);
    v.lgS = 31 - __builtin_clz((unsigned)v.S);
    v.kpl = ((v.K + v.S - 1) / v.S + 3) & ~3;
    v.slots = a.G * v.S * v.kpl;
    LevelShape s;
    if (!level_width(a, v, hcap[l], cap, want, optcap, quick, s)) return 0;
    pmax = std::max(pmax, v.P);
    a.opt = std::max(a.opt, s.opt);
    a.apass = std::max(a.apass, s.apass);
    need_h = std::max(need_h, s.need_h);
    upt = std::max(upt, s.upt);
    quad = quad || (s.opt == 4 && s.upt > 16);
    a.OMmax = std::max(a.OMmax, v.OM);
    a.zslots = std::max(a.zslots, v.slots);
  }
  // register buckets: h-part entries per lane, U entries per row and lane
  a.hpl = need_h <= 4 ? 4 : need_h <= 8 ? 8 : need_h <= 12 ? 12 : need_h <= 16 ? 16 : need_h <= 24 ? 24 : 32;
  a.upt = upt;
  if (!in_registers(a.opt, upt, a.apass, a.hpl)) return 0;
  // a level on one workgroup beside a wide one: fewer rows per thread for the
  // narrow one, rather than the largest instance for both (driving shape, K =
  // 16, 64, 128, 192: 48 us, 72 otherwise)
  if (a.opt == 4 && upt > 16 && !quad) return 0;
  a.umax = a.opt == 4 ? (upt <= 8 ? 8 : upt <= 16 ? 16 : 32) : a.opt == 2 ? (upt <= 16 ? 16 : 32) : (upt <= 8 ? 8 : upt <= 16 ? 16 : 32);
  // lane sl's terms at stride kst: it covers the lane's whole register bucket
  // (every read stays in the lane's zero-filled places), and 12, 20 or 36
  // floats put the 16-byte reads of consecutive lanes in distinct banks
  a.zfloats = 0;
  for (int l = 0; l < a.L; ++l) {
    PairLevel& v = a.lv[l];
    v.kst = a.umax + 4;
    v.zst = v.S * v.kst;
    a.zfloats = std::max(a.zfloats, a.G * v.zst);
  }
  a.hpad = (a.H + 3) & ~3;
  return pmax;
}

}  // namespace

int plan_pair(PairArgs& a, const int* hcap, int num_cu, int want, size_t* lds) {
  *lds = 0;
  int kmax = 0;
  for (int l = 0; l < a.L; ++l) kmax = std::max(kmax, a.lv[l].K);
  if (a.G < 1 || a.L > kMaxLevels) return 0;
  const int pairs = a.L * a.B;
  const bool xcds = num_cu >= kXcds * kXcdCus;   // the whole device: one group per XCD
  if (pairs > 1 && (want > 0 || !xcds)) return 0;
  // near groups: up to kNearWidth workgroups where two share a compute unit,
  // up to kXcdCus otherwise; a single pair that needs more runs on every XCD.
  // So does one whose sequence is too short to make up for what its slices cost
  // one XCD to load, in timesteps 1.4 per MB of U rows and 1.8 per MB of h parts;
  // the wider exchange costs wide layers more (us, near / spread; H = 512, 75%
  // pruning: K = 256, T = 1 15.5 / 15.1, T = 2 17.5 / 18.3, K = 512, T = 1 22.5 /
  // 15.7, 6 35.1 / 33.6, 8 40.2 / 40.9; 50%: K = 512, T = 8 46.1 / 44.2, 11 54.9 / 56.6;
  // H = 2048, 90%: K = 128, T = 1 15.4 / 15.9, K = 256, T = 1 21.8 / 15.7, 6 36.1 /
  // 35.3, 8 41.7 / 43.3).
  const double mu = 16e-6 * a.H * a.lv[0].K, mv = 6e-6 * a.G * a.lv[0].K * hcap[0];
  const bool quick = pairs == 1 && a.T < 1.4 * mu + 1.8 * mv - 1.4 - 3.6 * a.H / 1024.0;
  const int caps[2][3] = {{kNearWidth, kXcdCus, num_cu}, {num_cu, kNearWidth, kXcdCus}};
  for (int optcap : {4, 2, 1}) {
    for (int cap : caps[quick]) {
      if (cap == num_cu && (pairs > 1 || num_cu > kSpreadWords)) continue;
      const int P = plan_levels(a, hcap, std::min(cap, std::max(1, num_cu)), want, optcap, quick && cap == num_cu);
      if (!P) continue;
      const bool two = a.opt == 1 && a.apass == 1 && a.hpl <= kTwoHmax;
      const bool near = xcds && P <= (two ? kNearWidth : kXcdCus) && !(quick && cap == num_cu);
      if (!near && cap != num_cu) continue;
      // a spread group's polling threads
      if (!near && P > 1 && std::max(a.zslots, a.hpad) > 4 * kMaxUnits * kSpreadPollers) {
        if (quick) continue;
        return 0;
      }
      a.stamps = reinterpret_cast<unsigned long long*>(1);   // sized with the stamps' block
      const size_t bytes = 4 * (size_t)pair_layout(a).total;
      a.stamps = nullptr;
      if (bytes > (P > kXcdCus && near ? kLdsCap / 2 : kLdsCap)) {
        if ((cap != num_cu || quick) && pairs == 1) continue;
        return 0;
      }
      a.spread = !near && P > 1 && kmax > 0;
      // without terms nothing is exchanged and a group may lie anywhere: as many
      // side by side as there are compute units (T = 16, H = 512, one sequence:
      // 19 us against the general kernel's 28; T = 32, H = 2048, eight: 22 against
      // 131)
      if (kmax == 0) a.groups = std::min(pairs, std::max(1, num_cu / P));
      else a.groups = pairs > 1 || (near && P > 1) ? kXcds : 1;
      *lds = bytes;
      return P;
    }
  }
  return 0;
}

template <int APASS, int HMAX>
hipError_t launch_pair_u(const PairArgs& a, int P, size_t lds, hipStream_t stream) {
  if (a.opt == 4) {
    if (a.umax == 8) return launch_pair_kernel<4, 8, APASS, HMAX>(a, P, lds, stream);
    if (a.umax == 16) return launch_pair_kernel<4, 16, APASS, HMAX>(a, P, lds, stream);
    if constexpr (APASS == 1 || HMAX <= 16) return launch_pair_kernel<4, 32, APASS, HMAX>(a, P, lds, stream);
  } else if (a.opt == 2) {
    if (a.umax == 16) return launch_pair_kernel<2, 16, APASS, HMAX>(a, P, lds, stream);
    return launch_pair_kernel<2, 32, APASS, HMAX>(a, P, lds, stream);
  } else {
    if (a.umax == 8) return launch_pair_kernel<1, 8, APASS, HMAX>(a, P, lds, stream);
    if (a.umax == 16) return launch_pair_kernel<1, 16, APASS, HMAX>(a, P, lds, stream);
    if (a.umax == 32) return launch_pair_kernel<1, 32, APASS, HMAX>(a, P, lds, stream);
  }
  return hipErrorInvalidValue;   // the planner never asks for it
}

hipError_t launch_pair(const RunArgs& proj, const PairArgs& a, int P, hipStream_t stream) {
  hipError_t e = proj.GK > 0 ? launch_input_proj(proj, stream) : hipSuccess;
  if (e != hipSuccess) return e;
  const size_t lds = 4 * (size_t)pair_layout(a).total;
  if (a.apass == 2) {
    switch (a.hpl) {
      case 4: return launch_pair_u<2, 4>(a, P, lds, stream);
      case 8: return launch_pair_u<2, 8>(a, P, lds, stream);
      case 12: return launch_pair_u<2, 12>(a, P, lds, stream);
      case 16: return launch_pair_u<2, 16>(a, P, lds, stream);
      default: return launch_pair_u<2, 24>(a, P, lds, stream);
    }
  }
  switch (a.hpl) {
    case 4: return launch_pair_u<1, 4>(a, P, lds, stream);
    case 8: return launch_pair_u<1, 8>(a, P, lds, stream);
    case 12: return launch_pair_u<1, 12>(a, P, lds, stream);
    case 16: return launch_pair_u<1, 16>(a, P, lds, stream);
    case 24: return launch_pair_u<1, 24>(a, P, lds, stream);
    default: return launch_pair_u<1, 32>(a, P, lds, stream);
  }
}

}  // namespace alstm
