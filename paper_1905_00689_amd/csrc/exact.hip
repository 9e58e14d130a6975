// The exact LSTM on gfx950: the dense baseline the progressive approximation
// is measured against.  Gate pre-activations y = W_x x_t + W_h h_{t-1} + b
// with the full weight matrices (Sec. II, Fig. 1; the augmented matrix of
// Sec. III without any factorisation), then the same cell update.
//
// Two launches per run.  exact_xproj_kernel computes the x part of every
// gate row for every timestep at once (it does not depend on h).  The
// persistent exact_lstm_kernel then runs the recurrence: workgroup j owns a
// slice of hidden units and the four W_h rows of each, held in registers for
// the whole sequence, so one timestep needs a single exchange between
// workgroups (the h all-gather), where the progressive scheme needs two
// (z, then h).
//
// A row budget (a.rows < H) gives the paper's anytime baseline (Sec. VI-B):
// the dense products stopped after that many rows of every gate, the rows
// not reached holding the bias alone.  Only the computed rows are projected
// and multiplied.
#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"

namespace alstm {

namespace {

constexpr int kExactLanes = 16;   // lanes per W_h row
constexpr int kExactRows = kThreads / kExactLanes;   // rows per pass (32)
constexpr int kExactWpl = 32;     // W_h entries per lane held in registers (H <= 512)
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
template <bool WV, bool XV>
__global__ void __launch_bounds__(kThreads) exact_xproj_skinny_kernel(ExactArgs a, int nrow) {
  __shared__ float part[kWaves][4][16][17];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = 4 * (lane >> 4);
  const int TB = a.T * a.B, D = a.D, R = 4 * a.H;
  const int ol0 = (blockIdx.x % nrow) * 16, c0 = (blockIdx.x / nrow) * kSkinnyCols;
  const int nct = min(4, (TB - c0 + 15) / 16);
  const float* w = a.Wx + (size_t)gate_row(a, ol0 + li) * D;
  // contraction span of a wave: a multiple of 16, passes of 16 * kSkinnyUnits
  const int span = ((D + 16 * kWaves - 1) / (16 * kWaves)) * 16;
  const int k0 = wave * span, k1 = min(D, k0 + span);
  f32x4 acc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kb = k0; kb < k1; kb += 16 * kSkinnyUnits) {
    f32x4 wv[kSkinnyUnits];
#pragma unroll
    for (int u = 0; u < kSkinnyUnits; ++u) wv[u] = load4<WV>(w, kb + 16 * u + lk, k1);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c >= nct) break;
      const float* x = a.x + (size_t)min(c0 + 16 * c + li, TB - 1) * D;
#pragma unroll
      for (int u0 = 0; u0 < kSkinnyUnits; u0 += 8) {
        if (kb + 16 * u0 >= k1) break;
        f32x4 xv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) xv[u] = load4<XV>(x, kb + 16 * (u0 + u) + lk, k1);
        // chains of 32 products, added up pairwise
        f32x4 p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 8; ++u)
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

// The recurrence.  Workgroup j owns hidden units [j*RP, j*RP + rc) and the
// gate rows q*H + r of each (q = i, f, g, o); 16 lanes per row, rows in
// passes of 32.  Per timestep and sequence: y = px + W_h . h_{t-1} (lane
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
      auto group = [&](auto nbc, int b0) {
        constexpr int NB = decltype(nbc)::value;
        for (int ps = 0; ps < passes; ++ps) {
          const int ol = ob + ps * kExactRows;
          float acc[NB];
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[j] = 0.0f;
          if (ol < outs) {
            const int q = ol / rc, rr = ol - q * rc;
            const float* wrow = a.Wh + (size_t)(q * H + r0 + rr) * H;
            if (rr < rlive && NB == 1) {
#pragma unroll 4
              for (int k = sl; k < H; k += kExactLanes) acc[0] += wrow[k] * hs[(size_t)b0 * H + k];
            } else if (rr < rlive) {
              // 8 entries of the row in flight, then each applied to the group
              for (int k0 = sl; k0 < H; k0 += 8 * kExactLanes) {
                float wk[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                  const int k = k0 + i * kExactLanes;
                  wk[i] = wrow[k < H ? k : sl];
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                  const int k = k0 + i * kExactLanes;
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
            const float sum = group_sum<kExactLanes>(acc[j]);
            if (sl == 0 && ol < outs) store_y(t, b0 + j, ol, sum);
          }
        }
      };
      for (int b0 = 0; b0 < B; b0 += kExactSeq) {
        switch (min(kExactSeq, B - b0)) {
          case 1: group(std::integral_constant<int, 1>{}, b0); break;
          case 2: group(std::integral_constant<int, 2>{}, b0); break;
          case 3: group(std::integral_constant<int, 3>{}, b0); break;
          case 4: group(std::integral_constant<int, 4>{}, b0); break;
          case 5: group(std::integral_constant<int, 5>{}, b0); break;
          case 6: group(std::integral_constant<int, 6>{}, b0); break;
          case 7: group(std::integral_constant<int, 7>{}, b0); break;
          default: group(std::integral_constant<int, 8>{}, b0); break;
        }
      }
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
        if (!local) publish(a.hx + (size_t)b * H + r0 + rr, hv, tag);
      }
    }
    if (!local && !publisher) gather_tagged<2>(hs, nullptr, a.hx, B * H, tag, a.err, threadIdx.x, gthr);
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
  const long long nrow = (R + kTile - 1) / kTile, ncol = (TB + kTile - 1) / kTile;
  if (2 * nrow * ncol >= a.num_cu)
    exact_xproj_tile_kernel<WV, XV><<<dim3((unsigned)(nrow * ncol)), dim3(kThreads), 0, stream>>>(a, (int)nrow);
  else
    exact_xproj_skinny_kernel<WV, XV><<<dim3((unsigned)((long long)((R + 15) / 16) * ((TB + kSkinnyCols - 1) / kSkinnyCols))),
                                        dim3(kThreads), 0, stream>>>(a, (R + 15) / 16);
}

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
  }
  ExactArgs c = a;
  const size_t lds = plan_exact(c, blocks);
  if (lds > kLdsCap) return hipErrorInvalidValue;
  exact_lstm_kernel<<<dim3(blocks), dim3(kThreads), lds, stream>>>(c);
  return hipGetLastError();
}

}  // namespace alstm
