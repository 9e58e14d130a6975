// The exact LSTM on gfx950: the dense baseline the progressive approximation
// is measured against.  Gate pre-activations y = W_x x_t + W_h h_{t-1} + b
// with the full weight matrices (Sec. II, Fig. 1; the augmented matrix of
// Sec. III without any factorisation), then the same cell update.
//
// Two steps per run.  exact_xproj_*_kernel computes the x part of every gate row
// for every timestep at once (it does not depend on h).  Then the recurrence:
// every workgroup owns hidden units and the four W_h rows of each, so one
// timestep needs a single exchange between workgroups (the h all-gather), where
// the progressive scheme needs two (z, then h).  exact_near_kernel (up to 768
// units, a sequence per XCD) and exact_wide_kernel (up to 2048, eight sequences
// at a time over the device) hold W_h in registers; exact_lstm_kernel takes the
// rest: longer sequences than their x parts fit LDS, a few timesteps, more
// units, part of a device, and widths given by the caller.
//
// A row budget (a.rows < H) gives the paper's anytime baseline (Sec. VI-B):
// the dense products stopped after that many rows of every gate, the rows
// not reached holding the bias alone.  Only the computed rows are projected
// and multiplied.
#include <algorithm>
#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"

namespace alstm {

namespace {

constexpr int kExactLanes = 16;   // lanes per W_h row
constexpr int kExactRows = kThreads / kExactLanes;   // rows per pass (32)
constexpr int kExactWpl = 32;     // W_h entries per lane held in registers (H <= 512)
constexpr int kWideH = 2048;      // and up to which it fits those of the device
constexpr int kSkinnyCols = 64;   // x columns per workgroup of the narrow x projection
constexpr int kSkinnyUnits = 16;  // 16-byte units of a W_x row per lane held in registers there
constexpr int kTile = 128;        // gate rows and x columns per workgroup of the tiled x projection
constexpr int kTileK = 32;        // contraction slice staged in LDS there
constexpr int kTileLd = kTileK + 4;   // LDS row (floats): 16-byte reads of 16 rows in distinct banks
constexpr int kExactSeq = 8;      // sequences sharing one read of a W_h row in the recurrence

}  // namespace

// The x part: px[tb][o] = b[o] + W_x[o] . x[tb] for every computed gate row o =
// q*H + r (r < rows) and column tb = t*B + b; the px entries of the other rows
// are not written.  Both kernels run it on v_mfma_f32_16x16x4_f32 (fp32
// operands and sums; A = W_x rows, B = x columns): lane l holds
// A[l%16][l/16], B[l/16][l%16] and result rows 4*(l/16) .. +3 of column l%16.
// The four contraction indices of an instruction may be any four as long as
// both operands agree, so a lane reads 16 bytes (k .. k+3 of its row, k = 4 *
// (l/16)) and feeds four instructions from them.

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma4(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// row index of the ol-th of the 4*rows computed gate rows (clamped)
__device__ __forceinline__ int gate_row(const ExactArgs& a, int ol) {
  const int c = min(ol, 4 * a.rows - 1), q = c / a.rows;
  return q * a.H + (c - q * a.rows);
}

// p[k .. k+3], zeros from index n on (V: p + k is 16-byte aligned and n a
// multiple of 4)
template <bool V>
__device__ __forceinline__ f32x4 load4(const float* p, int k, int n) {
  if constexpr (V) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(p + (k < n ? k : 0));
    return k < n ? v : f32x4{0.f, 0.f, 0.f, 0.f};
  } else {
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = k + i < n ? p[k + i] : 0.f;
    return v;
  }
}

}  // namespace

// Few columns or few rows: what bounds it is reading W_x once (16.8 MB at D =
// 2048, H = 512), so the bytes in flight count.  A workgroup takes 16 gate
// rows and up to 64 columns, its 8 waves an eighth of the contraction each:
// a wave's whole slice of W_x (up to 16 units per lane) is loaded at once,
// x comes straight from L2, and the partial sums of the waves meet in LDS in
// a fixed order.  WV, XV: 16-byte aligned rows of W_x and of x.  MI355X, D =
// 2048, H = 512, 16 columns: 30.5 us (one wave per row, x staged by every
// workgroup) -> 10.5 us.
// U: 16-byte units of W_x per lane held at once, 16, or 4 where a wave's span has
// no more (one column, D = 256: 7.2 us with 16, most of them past the span).
template <bool WV, bool XV, int U>
__global__ void __launch_bounds__(kThreads) exact_xproj_skinny_kernel(ExactArgs a, int nrow) {
  constexpr int kXUnits = U < 8 ? U : 8;   // units of x at a time
  __shared__ float part[kWaves][4][16][17];
  if (clear_start_words(a.ctl, a.ctl_words)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = 4 * (lane >> 4);
  const int TB = a.T * a.B, D = a.D, R = 4 * a.H;
  const int ol0 = (blockIdx.x % nrow) * 16, c0 = (blockIdx.x / nrow) * kSkinnyCols;
  const int nct = min(4, (TB - c0 + 15) / 16);
  const float* w = a.Wx + (size_t)gate_row(a, ol0 + li) * D;
  // contraction span of a wave: a multiple of 16, passes of 16 * U
  const int span = ((D + 16 * kWaves - 1) / (16 * kWaves)) * 16;
  const int k0 = wave * span, k1 = min(D, k0 + span);
  f32x4 acc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kb = k0; kb < k1; kb += 16 * U) {
    f32x4 wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) wv[u] = load4<WV>(w, kb + 16 * u + lk, k1);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c >= nct) break;
      const float* x = a.x + (size_t)min(c0 + 16 * c + li, TB - 1) * D;
#pragma unroll
      for (int u0 = 0; u0 < U; u0 += kXUnits) {
        if (kb + 16 * u0 >= k1) break;
        f32x4 xv[kXUnits];
#pragma unroll
        for (int u = 0; u < kXUnits; ++u) xv[u] = load4<XV>(x, kb + 16 * (u0 + u) + lk, k1);
        // chains of 32 products, added up pairwise
        f32x4 p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < kXUnits; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) p[i] = mfma4(wv[u0 + u][i], xv[u][i], p[i]);
        acc[c] += (p[0] + p[1]) + (p[2] + p[3]);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (c < nct) {
      const f32x4 s = acc[c];
#pragma unroll
      for (int i = 0; i < 4; ++i) part[wave][c][li][(lane >> 4) * 4 + i] = s[i];
    }
  __syncthreads();
  for (int e = tid; e < nct * 256; e += kThreads) {
    const int c = e >> 8, col = (e >> 4) & 15, r = e & 15;
    float s = 0.0f;
#pragma unroll
    for (int wv = 0; wv < kWaves; ++wv) s += part[wv][c][col][r];
    const int ol = ol0 + r, tb = c0 + 16 * c + col;
    if (ol < 4 * a.rows && tb < TB) {
      const int o = gate_row(a, ol);
      a.px[(size_t)tb * R + o] = s + a.bias[o];
    }
  }
}

// Many rows and columns: bound by the matrix cores' fp32 rate.  128 x 128 tile
// per workgroup of 8 waves (64 x 32 each, 2 x 4 waves), contraction in
// slices of 32 through double-buffered LDS; a slice is fetched into registers
// while the one before is multiplied.  A slice is summed apart, eight slices
// apart from the rest, so that no chain of additions is longer than 32
// products, 8 slices or the number of such eights (the error against float64
// is then that of one wave per row, whose lanes summed 32 products each).
// MI355X, D = H = 2048, 512 columns: 3260 us (one wave per row) -> 185 us, 93
// TFLOP/s; a large library product reaches 152.
template <bool WV, bool XV>
__global__ void __launch_bounds__(kThreads) exact_xproj_tile_kernel(ExactArgs a, int nrow) {
  __shared__ __align__(16) float As[2][kTile * kTileLd];
  __shared__ __align__(16) float Bs[2][kTile * kTileLd];
  if (clear_start_words(a.ctl, a.ctl_words)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = 4 * (lane >> 4);
  const int wm = (wave & 1) * 64, wn = (wave >> 1) * 32;
  const int TB = a.T * a.B, D = a.D, R = 4 * a.H;
  // row tiles vary fastest: the workgroups in flight share few column tiles
  const int ol0 = (blockIdx.x % nrow) * kTile, c0 = (blockIdx.x / nrow) * kTile;
  const int sr = tid >> 3, sk = 4 * (tid & 7);
  const float* wp[2];
  const float* xp[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    wp[j] = a.Wx + (size_t)gate_row(a, ol0 + sr + 64 * j) * D;
    xp[j] = a.x + (size_t)min(c0 + sr + 64 * j, TB - 1) * D;
  }
  f32x4 ra[2], rb[2];
  auto fetch = [&](int k) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      ra[j] = load4<WV>(wp[j], k + sk, D);
      rb[j] = load4<XV>(xp[j], k + sk, D);
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      *reinterpret_cast<f32x4*>(&As[buf][(sr + 64 * j) * kTileLd + sk]) = ra[j];
      *reinterpret_cast<f32x4*>(&Bs[buf][(sr + 64 * j) * kTileLd + sk]) = rb[j];
    }
  };
  f32x4 sum[4][2], pair[4][2], acc[4][2];
  int slices = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) sum[i][j] = pair[i][j] = acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  fetch(0);
  stash(0);
  lds_barrier();
  int buf = 0;
  for (int k = 0; k < D; k += kTileK, buf ^= 1) {
    if (k + kTileK < D) fetch(k + kTileK);
#pragma unroll
    for (int kk = 0; kk < kTileK; kk += 16) {
      f32x4 av[4], bv[2];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        av[i] = *reinterpret_cast<const f32x4*>(&As[buf][(wm + 16 * i + li) * kTileLd + kk + lk]);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        bv[j] = *reinterpret_cast<const f32x4*>(&Bs[buf][(wn + 16 * j + li) * kTileLd + kk + lk]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = mfma4(av[i][e], bv[j][e], acc[i][j]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        pair[i][j] += acc[i][j];
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    if ((++slices & 7) == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          sum[i][j] += pair[i][j];
          pair[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    if (k + kTileK < D) {
      stash(buf ^ 1);   // its readers passed the last barrier
      lds_barrier();
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const f32x4 s = sum[i][j] + pair[i][j];
      const int tb = c0 + wn + 16 * j + li;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ol = ol0 + wm + 16 * i + (lane >> 4) * 4 + e;
        if (ol < 4 * a.rows && tb < TB) {
          const int o = gate_row(a, ol);
          a.px[(size_t)tb * R + o] = s[e] + a.bias[o];
        }
      }
    }
}

// The recurrence with W_h in registers.  A sum over h_{t-1} is taken by 16
// lanes (H <= kNearH) or 64 (beyond), lane sl the entries k = sl + L*i with i
// ascending, then the lanes pairwise; then the x part and bias.  The same
// order in every kernel here, so the results do not depend on which one runs.
//
// Slot w of the h exchange is entry i = w % kpl of lane sl = w / kpl (kpl =
// ceil(H / L) rounded up to 4), the unit k = sl + L*i; a workgroup owns RU
// consecutive slots and the four W_h rows of each one's unit.  A slot exists
// three times, for timesteps t mod 3: at timestep t its owner empties the one
// of timesteps t-2 and t+1 (everyone's h_{t-1} is here, so everyone has read
// h_{t-2}) and stores h_t only when that is done.

namespace {

// unit of slot w for L lanes (H or more: none)
__device__ __forceinline__ int slot_unit(int w, int kpl, int L) { return w / kpl + L * (w % kpl); }

// One sequence by one workgroup, W_h read from memory; hs [2][H], cs [H], ys
// [32] in LDS.
template <int L>
__device__ void exact_alone(const ExactArgs& a, int b, float* hs, float* cs, float* ys) {
  const int tid = threadIdx.x, H = a.H, sl = tid % L, rs = tid / L;
  constexpr int units = kThreads / L / 4;   // per pass; rows gate-minor
  for (int i = tid; i < H; i += kThreads) {
    hs[i] = a.h0 ? a.h0[(size_t)b * H + i] : 0.0f;
    cs[i] = a.c0 ? a.c0[(size_t)b * H + i] : 0.0f;
  }
  __syncthreads();
  for (int t = 0; t < a.T; ++t) {
    const float* h = hs + (t & 1) * H;
    float* hn = hs + ((t + 1) & 1) * H;
    const size_t tb = (size_t)t * a.B + b;
    for (int u0 = 0; u0 < H; u0 += units) {
      const int u = u0 + (rs >> 2), o = (rs & 3) * H + u;
      float acc = 0.0f;
      if (u < H && u < a.rows) {
        const float* w = a.Wh + (size_t)o * H;
        for (int k = sl; k < H; k += L) acc += w[k] * h[k];
      }
      if constexpr (L == 16) acc = group_sum<16>(acc);
      else acc = wave_sum(acc);
      if (sl == 0 && u < H) ys[rs] = acc + (u < a.rows ? a.px[tb * 4 * H + o] : a.bias[o]);
      __syncthreads();
      if (tid < units && u0 + tid < H) {
        float c = cs[u0 + tid], hv;
        cell_update(ys[4 * tid], ys[4 * tid + 1], ys[4 * tid + 2], ys[4 * tid + 3], c, hv);
        cs[u0 + tid] = c;
        hn[u0 + tid] = hv;
        a.h_out[tb * H + u0 + tid] = hv;
      }
      __syncthreads();
    }
  }
  if (a.c_out)
    for (int i = tid; i < H; i += kThreads) a.c_out[(size_t)b * H + i] = cs[i];
  __syncthreads();
}

// LDS floats of the near kernel: mode [4], x part [T][4*RU], h [2][16][WPL + 4],
// c [H] (alone) and the rows' sums per wave
__host__ __device__ inline size_t near_lds(const ExactArgs& a, int wpl) {
  return 4 + (((size_t)a.T * 4 * a.RU + 3) & ~(size_t)3) + 2 * 16 * (wpl + 4) + ((a.H + 3) & ~3) + kWaves * 16;
}

__device__ __forceinline__ float dpp_swap1(float v) {   // lane ^ 1
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false));
}
__device__ __forceinline__ float dpp_swap2(float v) {   // lane ^ 2
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, false));
}
__device__ __forceinline__ float dpp_swap4(float v) {   // lane ^ 4: mirrored half rows, quads reversed back
  const int m = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, false);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, m, 0x1B, 0xF, 0xF, false));
}
__device__ __forceinline__ float dpp_swap8(float v) {   // lane ^ 8: rows rotated by 8
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xF, 0xF, false));
}

// v[b] summed over the wave for NB = 1, 2, 4 or 8 values at once; lane l gets
// the sum of v[l % NB].  The pairs are those of wave_sum (lanes 1, 2, 4, 8, 16
// and 32 apart, in that order); while there is more than one value a lane
// hands half of them to its partner and goes on with the other half.
template <int NB>
__device__ __forceinline__ float wave_sums(const float* v, int lane) {
  float r[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) r[i] = v[i];
  if constexpr (NB >= 2) {
#pragma unroll
    for (int i = 0; i < NB / 2; ++i) {
      const float keep = (lane & 1) ? r[2 * i + 1] : r[2 * i], give = (lane & 1) ? r[2 * i] : r[2 * i + 1];
      r[i] = keep + dpp_swap1(give);
    }
  } else {
    r[0] += dpp_swap1(r[0]);
  }
  if constexpr (NB >= 4) {
#pragma unroll
    for (int i = 0; i < NB / 4; ++i) {
      const float keep = (lane & 2) ? r[2 * i + 1] : r[2 * i], give = (lane & 2) ? r[2 * i] : r[2 * i + 1];
      r[i] = keep + dpp_swap2(give);
    }
  } else {
    r[0] += dpp_swap2(r[0]);
  }
  if constexpr (NB >= 8) {
    const float keep = (lane & 4) ? r[1] : r[0], give = (lane & 4) ? r[0] : r[1];
    r[0] = keep + dpp_swap4(give);
  } else {
    r[0] += dpp_swap4(r[0]);
  }
  r[0] += dpp_swap8(r[0]);
  r[0] += __shfl_xor(r[0], 16, 64);
  r[0] += __shfl_xor(r[0], 32, 64);
  return r[0];
}

}  // namespace

// Near groups: one sequence per XCD (more take turns), 32 workgroups (fewer
// for narrow layers) holding its W_h in registers: OPT rows per thread, 16
// lanes per row, WPL entries per lane.  One exchange per timestep, through the
// XCD's L2 (see pair_lstm_kernel on what that saves, and group_start on a
// group that is not all resident).  MI355X, D = 2048, H = 512, T = 16, one
// sequence: the recurrence 43 us on exact_lstm_kernel, 27.4 here.
template <int OPT, int WPL>
__global__ void __launch_bounds__(kThreads) exact_near_kernel(ExactArgs a) {
  extern __shared__ __align__(16) float lds[];
  constexpr int LD = WPL + 4;   // 16-byte reads of the lanes in distinct banks
  const int g = (int)((blockIdx.x + kXcds - a.first_xcd) % kXcds), j = blockIdx.x / kXcds;
  if (g >= a.B) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int H = a.H, B = a.B, T = a.T, R4 = 4 * a.H, RU = a.RU, kpl = a.kpl;
  const bool local = a.P == 1;
  int* modes = reinterpret_cast<int*>(lds);
  float* pxs = lds + 4;
  float* hs = pxs + ((T * 4 * RU + 3) & ~3);
  float* cs = hs + 2 * 16 * LD;
  float* ys = cs + ((H + 3) & ~3);
  const size_t exf = 3 * (size_t)a.slots;
  unsigned long long* hand = a.ctl + (size_t)g * kCtlWords;
  unsigned long long* decide = hand + kNearWidth;
  if (wv == kWaves - 1) {
    int mode = kFar;
    if (!local) {
      for (int b = g; b < B; b += kXcds)
        for (int i = lane; i < 3 * RU; i += 64) {
          const int w = j * RU + i % RU;
          if (w < a.slots) store_slot(a.ex + b * exf + (size_t)(i / RU) * a.slots + w, kEmpty, false);
        }
      wait_memory();
      mode = group_start(hand, decide, j, a.P, a.tag_base | 0xFFFFu, a.wait_ticks, a.err);
    }
    if (lane == 0) modes[0] = mode;
  }
  // rows ol = rs + 32 o: gate ol & 3 of owned slot ol >> 2
  const int sl = tid & 15, rs = tid >> 4;
  float wr[OPT][WPL];
#pragma unroll
  for (int o = 0; o < OPT; ++o) {
    const int ol = rs + 32 * o, ul = ol >> 2, w = j * RU + ul, k = slot_unit(w, kpl, 16);
    const bool live = ul < RU && w < a.slots && k < a.rows;
    const float* wrow = a.Wh + (live ? (size_t)((ol & 3) * H + k) * H : 0);
#pragma unroll
    for (int i = 0; i < WPL; ++i) wr[o][i] = wrow[min(sl + 16 * i, H - 1)];
#pragma unroll
    for (int i = 0; i < WPL; ++i) wr[o][i] = live && sl + 16 * i < H ? wr[o][i] : 0.0f;
  }
  // cell role: lane o < OPT updates owned slot wv + 8 o, whose rows this wave sums
  const int cul = wv + 8 * lane, cw = j * RU + cul, cunit = slot_unit(cw, kpl, 16);
  const bool cell = lane < OPT && cul < RU && cw < a.slots;
  const bool cell_ok = cell && cunit < H;
  // 16-byte unit of the exchange polled by this thread (slots <= 1024)
  const bool upoll = 4 * tid < a.slots;
  int udst[1];

  bool near = false, seen_mode = false;
  for (int b = g; b < B; b += kXcds) {
    if (b != g) __syncthreads();
    float c = (cell_ok && a.c0) ? a.c0[(size_t)b * H + cunit] : 0.0f;
    for (int i = tid; i < 2 * 16 * LD; i += kThreads) {
      const int l = (i / LD) & 15, e = i % LD, k = l + 16 * e;
      hs[i] = (i < 16 * LD && e < WPL && k < H && a.h0) ? a.h0[(size_t)b * H + k] : 0.0f;
    }
    for (int i = tid; i < T * 4 * RU; i += kThreads) {
      const int t = i / (4 * RU), ol = i - t * 4 * RU, w = j * RU + (ol >> 2), k = slot_unit(w, kpl, 16);
      const int o = (ol & 3) * H + k;
      float v = 0.0f;
      if (w < a.slots && k < H) v = k < a.rows ? a.px[((size_t)t * B + b) * R4 + o] : a.bias[o];
      pxs[i] = v;
    }
    __syncthreads();
    if (!seen_mode) {
      const int mode = __builtin_amdgcn_readfirstlane(modes[0]);
      if (mode >= kAlone) break;
      near = mode == kNear;
      seen_mode = true;
    }
    float* ex = a.ex + b * exf;
    for (int t = 0; t < T; ++t) {
      const float* hc = hs + (t & 1) * 16 * LD + sl * LD;
      float* hn = hs + ((t + 1) & 1) * 16 * LD;
      if (cell && !local) store_slot(ex + (size_t)((t + 1) % 3) * a.slots + cw, kEmpty, near);
      float acc[OPT];
#pragma unroll
      for (int o = 0; o < OPT; ++o) acc[o] = 0.0f;
#pragma unroll
      for (int i0 = 0; i0 < WPL; i0 += 8) {
        const float4 h0 = *reinterpret_cast<const float4*>(hc + i0), h1 = *reinterpret_cast<const float4*>(hc + i0 + 4);
#pragma unroll
        for (int o = 0; o < OPT; ++o) {
          acc[o] += wr[o][i0] * h0.x;
          acc[o] += wr[o][i0 + 1] * h0.y;
          acc[o] += wr[o][i0 + 2] * h0.z;
          acc[o] += wr[o][i0 + 3] * h0.w;
          acc[o] += wr[o][i0 + 4] * h1.x;
          acc[o] += wr[o][i0 + 5] * h1.y;
          acc[o] += wr[o][i0 + 6] * h1.z;
          acc[o] += wr[o][i0 + 7] * h1.w;
        }
      }
#pragma unroll
      for (int o = 0; o < OPT; ++o) {
        const float s = group_sum<16>(acc[o]);
        if (sl == 0 && rs + 32 * o < 4 * RU) ys[wv * 16 + o * 4 + (lane >> 4)] = s + pxs[t * 4 * RU + rs + 32 * o];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (cell) {
        const float4 y = *reinterpret_cast<const float4*>(ys + wv * 16 + lane * 4);
        float hv;
        cell_update(y.x, y.y, y.z, y.w, c, hv);
        if (local) {
          hn[(cw / kpl) * LD + cw % kpl] = hv;
        } else {
          wait_memory();   // the emptied slot
          publish_slot(ex + (size_t)(t % 3) * a.slots + cw, cell_ok ? hv : 0.0f, near);
        }
        if (cell_ok) a.h_out[((size_t)t * B + b) * H + cunit] = hv;
      }
      // nobody reads the last timestep's h (one step: the exchange still
      // tells that everyone has started)
      if (!local && (t + 1 < T || T == 1)) {
        udst[0] = upoll ? (4 * tid / kpl) * LD + (4 * tid) % kpl : 0;
        poll_units<1>(hn, ex + (size_t)(t % 3) * a.slots, a.slots * 4, udst, upoll ? 1u : 0u, a.err);
      }
      lds_barrier();
    }
    if (a.c_out && cell_ok) a.c_out[(size_t)b * H + cunit] = c;
  }
  if (local) return;
  __syncthreads();
  const int mode = __builtin_amdgcn_readfirstlane(modes[0]);
  if (mode == kAlone) {
    for (int b = g; b < B; b += kXcds) exact_alone<16>(a, b, hs, cs, ys);
  }
}

// Wide layers: W_h in the registers of the whole device (64 MB at H = 2048),
// every workgroup eight slots, a wave the four rows of one unit: 64 lanes per
// row, WPL entries per lane, each applied to all NB sequences (the run's,
// padded to a power of two).  h of all sequences in LDS, 16-byte reads shared
// by four rows.  What bounds a timestep at eight sequences is the fp32 rate
// (1024 multiply-adds per lane, 3.4 us) and then the exchange of h between
// XCDs (64 KB to every workgroup).  MI355X, D = H = 2048, eight sequences:
// 28.7 us per timestep with W_h read from memory, 7.7 here; 8.7 with a first
// poll round of all units at once (poll_units), which comes too early.
template <int WPL, int NB>
__global__ void __launch_bounds__(kThreads) exact_wide_kernel(ExactArgs a) {
  extern __shared__ __align__(16) float lds[];
  constexpr int LD = WPL + 4, kUnits = (NB * WPL + 31) / 32;   // polled per thread
  const int j = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int H = a.H, B = a.B, nb = a.nb, T = a.T, R4 = 4 * a.H, kpl = a.kpl, slots = a.slots;
  int* modes = reinterpret_cast<int*>(lds);
  float* hown = lds + 4;                 // [NB][8] h of the owned slots
  float* hs = hown + NB * 8;             // [NB][64][LD]
  unsigned long long* hand = a.ctl;
  unsigned long long* decide = a.ctl + kSpreadWords;
  const size_t third = (size_t)NB * slots;
  if (wv == kWaves - 1) {
    for (int i = lane; i < 3 * NB * 8; i += 64)
      store_slot(a.ex + (i / 8) * (size_t)slots + j * 8 + (i & 7), kEmpty, false);
    wait_memory();
    const int mode = group_start(hand, decide, j, a.P, a.tag_base | 0xFFFFu, a.wait_ticks, a.err);
    if (lane == 0) modes[0] = mode;
  }
  const int w = j * 8 + wv, unit = slot_unit(w, kpl, 64);
  const bool live = unit < H, computed = unit < a.rows;
  float wr[4][WPL];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float* wrow = a.Wh + (computed ? (size_t)(q * H + unit) * H : 0);
#pragma unroll
    for (int i = 0; i < WPL; ++i) wr[q][i] = wrow[min(lane + 64 * i, H - 1)];
#pragma unroll
    for (int i = 0; i < WPL; ++i) wr[q][i] = computed && lane + 64 * i < H ? wr[q][i] : 0.0f;
  }
  // cell role: lane b < NB updates this wave's unit for sequence b
  const bool cell_ok = lane < nb && live;
  float c = (cell_ok && a.c0) ? a.c0[(size_t)lane * H + unit] : 0.0f;
  float pxv[4];
  auto fetch_px = [&](int t) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      pxv[q] = cell_ok ? (computed ? a.px[((size_t)t * B + lane) * R4 + q * H + unit] : a.bias[q * H + unit]) : 0.0f;
  };
  fetch_px(0);
  for (int i = tid; i < NB * 64 * LD; i += kThreads) {
    const int b = i / (64 * LD), l = (i / LD) & 63, e = i % LD, k = l + 64 * e;
    hs[i] = (b < nb && e < WPL && k < H && a.h0) ? a.h0[(size_t)b * H + k] : 0.0f;
  }
  int udst[kUnits];
  unsigned upend = 0;
#pragma unroll
  for (int r = 0; r < kUnits; ++r) {
    const int s4 = 4 * (tid + kThreads * r), b = s4 / slots, s = s4 - b * slots;
    if (b < NB) upend |= 1u << r;
    udst[r] = b < NB ? (b * 64 + s / kpl) * LD + s % kpl : 0;
  }
  __syncthreads();
  const int mode = __builtin_amdgcn_readfirstlane(modes[0]);
  if (mode >= kAlone) {
    __syncthreads();
    if (mode == kAlone)
      for (int b = 0; b < nb; ++b) exact_alone<64>(a, b, lds + 4, lds + 4 + 2 * H, lds + 4 + 3 * H);
    return;
  }
  for (int t = 0; t < T; ++t) {
    float* out = a.ex + (t % 3) * third;
    // first wave: the owned slots of timestep t+1 emptied (16 bytes a lane)
    const int eb = lane >> 1, es = j * 8 + 4 * (lane & 1);
    if (wv == 0 && lane < 2 * NB) {
      float* e = a.ex + ((t + 1) % 3) * third + (size_t)eb * slots + es;
#pragma unroll
      for (int i = 0; i < 4; ++i) store_slot(e + i, kEmpty, false);
    }
    float acc[4][NB];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[q][b] = 0.0f;
    const float* hl = hs + lane * LD;
#pragma unroll
    for (int i = 0; i < WPL; i += 4) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const float4 h = *reinterpret_cast<const float4*>(hl + b * 64 * LD + i);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc[q][b] += wr[q][i] * h.x;
          acc[q][b] += wr[q][i + 1] * h.y;
          acc[q][b] += wr[q][i + 2] * h.z;
          acc[q][b] += wr[q][i + 3] * h.w;
        }
      }
    }
    float y[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) y[q] = wave_sums<NB>(acc[q], lane) + pxv[q];
    float hv;
    cell_update(y[0], y[1], y[2], y[3], c, hv);
    if (lane < NB) hown[lane * 8 + wv] = cell_ok ? hv : 0.0f;
    if (wv == 0) wait_memory();   // the emptied slots
    lds_barrier();                // every read of hs is done, hown complete
    if (wv == 0 && lane < 2 * NB) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        publish_slot(out + (size_t)eb * slots + es + i, hown[eb * 8 + 4 * (lane & 1) + i], false);
    }
    if (cell_ok) a.h_out[((size_t)t * B + lane) * H + unit] = hv;
    if (t + 1 < T) fetch_px(t + 1);
    if (t + 1 < T || T == 1) poll_units<kUnits, false>(hs, out, (int)(third * 4), udst, upend, a.err);
    lds_barrier();
  }
  if (a.c_out && cell_ok) a.c_out[(size_t)lane * H + unit] = c;
}

// The recurrence on any width, for the shapes and launches the kernels above do
// not take.  Workgroup j owns hidden units [j*RP, j*RP + rc) and the
// gate rows q*H + r of each (q = i, f, g, o); 16 lanes per row (64 past
// kNearH), rows in passes of 32 (8).  Per timestep and sequence: y = px + W_h . h_{t-1} (lane
// partial sums, fixed-order reduction), the cell update, h published as
// tagged words, then the full h_t gathered by every workgroup.
__global__ void __launch_bounds__(kThreads) exact_lstm_kernel(ExactArgs a) {
  extern __shared__ __align__(16) float lds[];
  const int P = gridDim.x, j = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int H = a.H, B = a.B, T = a.T, RP = a.rows_per, R4 = 4 * H;
  const int r0 = j * RP;
  const int rc = max(0, min(RP, H - r0));
  const int outs = 4 * rc;
  float* hs = lds;                         // [B][H]  h_{t-1}
  float* ys = hs + (size_t)B * H;          // [B][4*RP] y of the owned rows
  float* cs = ys + (size_t)B * 4 * RP;     // [B][RP]   c of the owned units
  float* hown = cs + (size_t)B * RP;       // [B][RP]   new h of the owned units
  float* pxs = hown + (size_t)B * RP;      // [T*B][4*RP] x part of the owned rows (px_lds)

  const int sl = threadIdx.x % kExactLanes, ob = threadIdx.x / kExactLanes;
  const int passes = (outs + kExactRows - 1) / kExactRows;
  const int rlive = max(0, min(rc, a.rows - r0));   // owned units whose rows are computed
  // pass 0's row entries in registers when H fits (the common case); zero for
  // rows not computed, so their sums are 0
  float wr[kExactWpl];
  const bool wreg = a.wreg != 0;
  {
    const int ol = ob;
    const int q = ol < outs ? ol / rc : 0, rr = ol < outs ? ol - q * rc : 0;
    const bool live = ol < outs && rr < rlive;
    const float* wrow = a.Wh + (size_t)(q * H + r0 + rr) * H;
#pragma unroll
    for (int i = 0; i < kExactWpl; ++i) {
      const int k = sl + kExactLanes * i;
      wr[i] = (wreg && live && k < H) ? wrow[k] : 0.0f;
    }
  }
  for (int i = threadIdx.x; i < B * H; i += kThreads) {
    const int b = i / H, r = i - b * H;
    hs[i] = a.h0 ? a.h0[(size_t)b * H + r] : 0.0f;
  }
  for (int i = threadIdx.x; i < B * RP; i += kThreads) {
    const int b = i / RP, rr = i - b * RP;
    cs[i] = (a.c0 && rr < rc) ? a.c0[(size_t)b * H + r0 + rr] : 0.0f;
  }
  if (a.px_lds) {
    for (int i = threadIdx.x; i < T * B * outs; i += kThreads) {
      const int tb = i / outs, ol = i - tb * outs;
      const int q = ol / rc, rr = ol - q * rc;
      const int o = q * H + r0 + rr;
      pxs[tb * 4 * RP + ol] = rr < rlive ? a.px[(size_t)tb * R4 + o] : a.bias[o];
    }
  }
  __syncthreads();

  const bool local = P == 1;
  const bool publisher = wave == kWaves - 1;
  const int gthr = kThreads - 64;
  // y of owned row ol for sequence b: the W_h sum plus the x part and bias
  auto store_y = [&](int t, int b, int ol, float sum) {
    const int q = ol / rc, rr = ol - q * rc;
    const int o = q * H + r0 + rr;
    const float px = a.px_lds ? pxs[(t * B + b) * 4 * RP + ol]
                              : (rr < rlive ? a.px[(size_t)(t * B + b) * R4 + o] : a.bias[o]);
    ys[b * 4 * RP + ol] = sum + px;
  };
  for (int t = 0; t < T; ++t) {
    const unsigned tag = a.tag_base | (unsigned)(t + 1);
    // two halves by parity: the words of t are overwritten at t+2, when everyone's
    // h_{t+1} is here, which each published after it had read all of h_t
    unsigned long long* hx = a.hx + (size_t)(t & 1) * B * H;
    if (wreg) {
      // pass 0's entries are in registers; later passes read their rows
      for (int b = 0; b < B; ++b) {
        const float* h = hs + (size_t)b * H;
        for (int ps = 0; ps < passes; ++ps) {
          const int ol = ob + ps * kExactRows;
          float acc = 0.0f;
          if (ol < outs) {
            if (ps == 0) {
#pragma unroll
              for (int i = 0; i < kExactWpl; ++i) acc += wr[i] * h[min(sl + kExactLanes * i, H - 1)];
            } else {
              const int q = ol / rc, rr = ol - q * rc;
              const float* wrow = a.Wh + (size_t)(q * H + r0 + rr) * H;
              if (rr < rlive) {
#pragma unroll 4
                for (int k = sl; k < H; k += kExactLanes) acc += wrow[k] * h[k];
              }
            }
          }
          acc = group_sum<kExactLanes>(acc);
          if (sl == 0 && ol < outs) store_y(t, b, ol, acc);
        }
      }
    } else {
      // rows are read once per group of up to kExactSeq sequences, each entry
      // applied to every sequence of the group (NB a compile-time group size,
      // so the inner loop carries no predicates); every (row, sequence) sum
      // keeps the per-sequence order
      auto group = [&](auto nbc, auto lanes, int b0) {
        constexpr int NB = decltype(nbc)::value, L = decltype(lanes)::value;
        constexpr int rows = kThreads / L;
        const int sl = threadIdx.x % L, ob = threadIdx.x / L, passes = (outs + rows - 1) / rows;
        for (int ps = 0; ps < passes; ++ps) {
          const int ol = ob + ps * rows;
          float acc[NB];
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[j] = 0.0f;
          if (ol < outs) {
            const int q = ol / rc, rr = ol - q * rc;
            const float* wrow = a.Wh + (size_t)(q * H + r0 + rr) * H;
            if (rr < rlive && NB == 1) {
#pragma unroll 4
              for (int k = sl; k < H; k += L) acc[0] += wrow[k] * hs[(size_t)b0 * H + k];
            } else if (rr < rlive) {
              // 8 entries of the row in flight, then each applied to the group
              for (int k0 = sl; k0 < H; k0 += 8 * L) {
                float wk[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                  const int k = k0 + i * L;
                  wk[i] = wrow[k < H ? k : sl];
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                  const int k = k0 + i * L;
                  if (k < H) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) acc[j] += wk[i] * hs[(size_t)(b0 + j) * H + k];
                  }
                }
              }
            }
          }
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            float sum;
            if constexpr (L == 16) sum = group_sum<16>(acc[j]);
            else sum = wave_sum(acc[j]);
            if (sl == 0 && ol < outs) store_y(t, b0 + j, ol, sum);
          }
        }
      };
      auto run = [&](auto lanes) {
        for (int b0 = 0; b0 < B; b0 += kExactSeq) {
          switch (min(kExactSeq, B - b0)) {
            case 1: group(std::integral_constant<int, 1>{}, lanes, b0); break;
            case 2: group(std::integral_constant<int, 2>{}, lanes, b0); break;
            case 3: group(std::integral_constant<int, 3>{}, lanes, b0); break;
            case 4: group(std::integral_constant<int, 4>{}, lanes, b0); break;
            case 5: group(std::integral_constant<int, 5>{}, lanes, b0); break;
            case 6: group(std::integral_constant<int, 6>{}, lanes, b0); break;
            case 7: group(std::integral_constant<int, 7>{}, lanes, b0); break;
            default: group(std::integral_constant<int, 8>{}, lanes, b0); break;
          }
        }
      };
      if (H <= kNearH) run(std::integral_constant<int, 16>{});
      else run(std::integral_constant<int, 64>{});
    }
    lds_barrier();
    for (int i = threadIdx.x; i < B * rc; i += kThreads) {
      const int b = i / rc, rr = i - b * rc;
      const float* y = ys + b * 4 * RP;
      float c = cs[b * RP + rr], hv;
      cell_update(y[0 * rc + rr], y[1 * rc + rr], y[2 * rc + rr], y[3 * rc + rr], c, hv);
      cs[b * RP + rr] = c;
      hown[b * RP + rr] = hv;
      if (local) hs[(size_t)b * H + r0 + rr] = hv;
    }
    lds_barrier();
    if (publisher) {
      for (int i = lane; i < B * rc; i += 64) {
        const int b = i / rc, rr = i - b * rc;
        const float hv = hown[b * RP + rr];
        a.h_out[((size_t)t * B + b) * H + r0 + rr] = hv;
        if (!local) publish(hx + (size_t)b * H + r0 + rr, hv, tag);
      }
    }
    if (!local && !publisher) gather_tagged<2>(hs, nullptr, hx, B * H, tag, a.err, threadIdx.x, gthr);
    lds_barrier();
  }
  if (a.c_out)
    for (int i = threadIdx.x; i < B * rc; i += kThreads) {
      const int b = i / rc, rr = i - b * rc;
      a.c_out[(size_t)b * H + r0 + rr] = cs[b * RP + rr];
    }
}

size_t plan_exact(ExactArgs& a, int P) {
  a.rows_per = (a.H + P - 1) / P;
  a.wreg = (a.H <= kExactLanes * kExactWpl) ? 1 : 0;
  const size_t base = 4 * ((size_t)a.B * a.H + (size_t)a.B * 4 * a.rows_per + 2 * (size_t)a.B * a.rows_per);
  const size_t pxb = 4 * (size_t)a.T * a.B * 4 * a.rows_per;
  a.px_lds = (base + pxb <= kLdsCap) ? 1 : 0;
  return base + (a.px_lds ? pxb : 0);
}

template <bool WV, bool XV>
static void launch_xproj(const ExactArgs& a, hipStream_t stream) {
  const int TB = a.T * a.B, R = 4 * a.rows;
  // the tiles take the same time until there is more than one per compute
  // unit, the 16-row workgroups time in proportion to the columns: equal at
  // about half a device of tiles (MI355X, 2048 rows, tiles / 16-row groups in
  // us: D = 2048, 512 columns 179 / 103, 1024 185 / 205, 2048 195 / 405; D =
  // 512, 512 columns 55 / 56, 1024 57 / 108)
  const long long nrow = (R + kTile - 1) / kTile, ncol = (TB + kTile - 1) / kTile, clear = a.ctl ? 1 : 0;
  if (2 * nrow * ncol >= a.num_cu)
    exact_xproj_tile_kernel<WV, XV><<<dim3((unsigned)(nrow * ncol + clear)), dim3(kThreads), 0, stream>>>(a, (int)nrow);
  else {
    const auto kernel = a.D <= 4 * 16 * kWaves ? exact_xproj_skinny_kernel<WV, XV, 4>
                                               : exact_xproj_skinny_kernel<WV, XV, kSkinnyUnits>;
    kernel<<<dim3((unsigned)((long long)((R + 15) / 16) * ((TB + kSkinnyCols - 1) / kSkinnyCols) + clear)),
             dim3(kThreads), 0, stream>>>(a, (R + 15) / 16);
  }
}

// Shape of the register kernels: fills P, kpl, slots and RU; returns the floats
// of the exchange (0: neither takes the run).  Both hold W_h in registers, one
// sequence per XCD up to kNearH units, over the whole device up to kWideH.
size_t plan_exact_group(ExactArgs& a) {
  a.P = 0;
  if (a.num_cu < kXcds * kXcdCus || a.num_cu > kSpreadWords) return 0;
  const int H = a.H;
  // A few timesteps do not make up for one XCD's taking all of W_h (H = 768,
  // one sequence, 1 / 2 / 3 timesteps: 20.4 / 21.4 / 23.0 us here, 12.8 / 16.7 /
  // 20.6 by exact_lstm_kernel, every workgroup its rows; H = 512 14.1 / 15.0 / 16.3
  // and 11.5 / 13.8 / 16.1, two sequences 14.4 / 15.4 and 12.5 / 16.2; H = 256
  // 11.5 / 12.0 and 11.0 / 13.5).
  if (H <= kNearH && (H > 512 ? a.T <= 3 && a.T * a.B <= 4 : a.T * a.B <= (H > 256 ? 2 : H > 192 ? 1 : 0))) return 0;
  if (H <= kNearH) {
    const int e = (H + 15) / 16;
    // up to 32 units one workgroup holds every row (four per thread)
    a.kpl = H <= 32 ? e : (e + 3) & ~3;
    a.slots = 16 * a.kpl;
    a.P = H <= 32 ? 1 : std::min(kXcdCus, (a.slots + 7) / 8);
    a.RU = (a.slots + a.P - 1) / a.P;
    if (4 * near_lds(a, H <= 128 ? 8 : H <= 256 ? 16 : H <= 512 ? 32 : 48) > kLdsCap) return a.P = 0;
    return (size_t)a.B * 3 * a.slots;
  }
  if (H <= kWideH) {
    a.kpl = ((H + 63) / 64 + 3) & ~3;
    a.slots = 64 * a.kpl;
    a.P = a.slots / 8;
    a.RU = 8;
    return (size_t)3 * kWideSeq * a.slots;
  }
  return 0;
}

namespace {

template <int OPT, int WPL>
hipError_t launch_near(const ExactArgs& a, hipStream_t stream) {
  static bool attr = false;
  if (!attr) {
    const hipError_t e = hipFuncSetAttribute((const void*)exact_near_kernel<OPT, WPL>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsCap);
    if (e != hipSuccess) return e;
    attr = true;
  }
  exact_near_kernel<OPT, WPL><<<dim3(kXcds * a.P), dim3(kThreads), 4 * near_lds(a, WPL), stream>>>(a);
  return hipGetLastError();
}

template <int WPL, int NB>
hipError_t launch_wide(const ExactArgs& a, hipStream_t stream) {
  static bool attr = false;
  if (!attr) {
    const hipError_t e = hipFuncSetAttribute((const void*)exact_wide_kernel<WPL, NB>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsCap);
    if (e != hipSuccess) return e;
    attr = true;
  }
  // h of every sequence, or (alone) h twice, c and a pass of sums
  const size_t fl = 4 + std::max<size_t>(NB * 8 + (size_t)NB * 64 * (WPL + 4), 3 * (size_t)a.H + 32);
  exact_wide_kernel<WPL, NB><<<dim3(a.P), dim3(kThreads), 4 * fl, stream>>>(a);
  return hipGetLastError();
}

template <int WPL>
hipError_t launch_wide_seq(const ExactArgs& a, hipStream_t stream) {
  if (a.nb <= 1) return launch_wide<WPL, 1>(a, stream);
  if (a.nb <= 2) return launch_wide<WPL, 2>(a, stream);
  if (a.nb <= 4) return launch_wide<WPL, 4>(a, stream);
  return launch_wide<WPL, 8>(a, stream);
}

}  // namespace

hipError_t launch_exact(const ExactArgs& a, int blocks, hipStream_t stream) {
  static bool attr = false;
  if (!attr) {
    const hipError_t e =
        hipFuncSetAttribute((const void*)exact_lstm_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsCap);
    if (e != hipSuccess) return e;
    attr = true;
  }
  if (a.rows > 0) {
    const bool wv = a.D % 4 == 0;
    if (wv && a.xvec) launch_xproj<true, true>(a, stream);
    else if (wv) launch_xproj<true, false>(a, stream);
    else launch_xproj<false, false>(a, stream);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  } else if (a.ctl) {
    const hipError_t e = launch_clear_u64(a.ctl, a.ctl_words, stream);
    if (e != hipSuccess) return e;
  }
  if (a.P > 0) {
    if (a.H > kNearH) {
      // more than kWideSeq sequences take turns (exact_lstm_kernel, which reads W_h
      // from memory at every timestep: H = 1024, 32 sequences, T = 16 1570 us)
      for (int b0 = 0; b0 < a.B; b0 += kWideSeq) {
        ExactArgs c = a;
        c.nb = std::min(kWideSeq, a.B - b0);
        c.tag_base = a.tag_base + ((unsigned)(b0 / kWideSeq) << 16);
        const size_t off = (size_t)b0 * a.H;
        c.px += 4 * off;
        c.h_out += off;
        if (a.h0) c.h0 += off;
        if (a.c0) c.c0 += off;
        if (a.c_out) c.c_out += off;
        const hipError_t e = a.kpl <= 16 ? launch_wide_seq<16>(c, stream) : launch_wide_seq<32>(c, stream);
        if (e != hipSuccess) return e;
      }
      return hipSuccess;
    }
    if (a.P == 1) return launch_near<4, 8>(a, stream);   // 16 or 32 units
    if (a.H <= 128) return launch_near<1, 8>(a, stream);
    if (a.H <= 256) return launch_near<1, 16>(a, stream);
    if (a.H <= 512) return launch_near<2, 32>(a, stream);
    return launch_near<3, 48>(a, stream);
  }
  ExactArgs c = a;
  const size_t lds = plan_exact(c, blocks);
  if (lds > kLdsCap) return hipErrorInvalidValue;
  // only workgroups that own units: nobody waits for one without, whose h would be
  // overwritten under it
  blocks = std::min(blocks, (a.H + c.rows_per - 1) / c.rows_per);
  exact_lstm_kernel<<<dim3(blocks), dim3(kThreads), lds, stream>>>(c);
  return hipGetLastError();
}

}  // namespace alstm
