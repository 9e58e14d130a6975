// gfx950 bf16 MFMA path for many independent sequences (arXiv 1905.00689,
// Eq. (1) per gate, then the Sec. II cell update).
//
// With a batch of sequences every refinement step becomes a real dense
// contraction, so the factors are kept as zero-filled bf16 panels and the
// three products run on v_mfma_f32_16x16x32_bf16 with fp32 accumulation:
//   x-projection (once per run)  P[tau][t,b] = Vx[tau][:] . x_t[b][:]
//   per timestep, h-projection   z[tau][b]   = sigma_tau (P[tau][t,b] + Vh[tau][:] . h_{t-1}[b][:])
//   per timestep, accumulation   y[o][b]     = bias[o] + U[o][:] . z_g(o)[:][b],  then gates, c, h.
// Pruned entries are stored as zeros, so the MFMA executes the dense work
// (about 1/(1-p) times the method's own count); the results are those of
// Eq. (1) with bf16 operands (x~, the factor values and z) and fp32 sums.
//
// MFMA operand layout (v_mfma_f32_16x16x32_bf16, wave64): lane l holds
// A[l%16][8*(l/16) .. +7], B[8*(l/16) .. +7][l%16], and the result rows
// 4*(l/16) .. +3 of column l%16.  Every operand below is stored with the
// contraction index contiguous, so a lane reads its 8 values as one 16-byte
// load.
#include "device_common.hpp"

#include <algorithm>

namespace alstm {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x4 mfma(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 load8(const uint16_t* p) { return *reinterpret_cast<const bf16x8*>(p); }

__device__ __forceinline__ uint16_t bf16_bits(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }

__device__ __forceinline__ float sigmoid_b(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float tanh_b(float x) { return 2.0f * sigmoid_b(2.0f * x) - 1.0f; }

}  // namespace

// ---------------------------------------------------------------- x-projection
// P[t*Bp + b][r] = sum_k Vx[.][k] * x[t][b][k] for the rows r < a.rows (term
// n of group g at r = g*km + n, km = pld / G).
// One BM (tau) x 128 (t, b) tile per workgroup of BM / 32 waves (BM = 128 or
// 256), each wave a 64 x 64 part (4 x 4 MFMA blocks); the contraction runs in slices of 32
// staged through LDS, double-buffered: slice s+1 is fetched into registers
// (x converted to bf16 on the way) while slice s is multiplied.  Tiles are
// numbered so that each XCD (workgroups are dealt to the 8 XCDs round robin)
// takes whole columns of tiles: the x slice of a column is fetched into that
// XCD's L2 once and shared by every row tile.
// Bound by the LDS passes of a slice between its two barriers (64 KB read and
// 24 KB written per 512 cycles of MFMA with 8 waves): a prefetch of four
// slices instead of two, slices of 64, or another order of the stash changed
// nothing (50-53 us); the 256-row tile reads and converts each x value half
// as often.  2048 x 4096 x 2048: 58.3 us with 128 rows, 50.6 with 256 (0.68
// PFLOP/s).
constexpr int kXBM = kPanelRowAlign, kXWide = 256, kXBN = 128, kXBK = 32;
static_assert(kPanelDAlign == 2 * kXBK, "D is padded to a pair of x-projection slices");
constexpr int kXLD = kXBK + 8;   // LDS row stride (bf16): 80 bytes, conflict-free 16-byte reads

// VEC: x rows are 16-byte aligned and D is a multiple of the D padding (so
// Dp == D): every slice of a live row is whole float4s (no bounds tests in
// the fetch).
// With a.xsplit > 1 workgroup blockIdx.x takes part blockIdx.x / (nM * nN)
// of the contraction (a.Dp / a.xsplit columns) for its tile and writes the
// partial tile to Ppart[part]; batched_xproj_sum_kernel adds the parts.
template <bool VEC, int BM>
__global__ void __launch_bounds__(2 * BM) batched_xproj_kernel(BatchedArgs a, int nM, int nN) {
  constexpr int kAR = BM / 2, kBR = BM / 4;           // rows of A, columns of B that one load of the workgroup covers
  constexpr int kNB = kXBN / kBR;                     // loads of a B slice per thread
  __shared__ __align__(16) uint16_t As[2][BM * kXLD];
  __shared__ __align__(16) uint16_t Bs[2][kXBN * kXLD];
  if (clear_start_words(a.ctl, a.ctl_words)) return;
  const int nt = nM * nN;
  const int part = blockIdx.x / nt, bid = blockIdx.x - part * nt;
  int tile = bid;
  if (nt % 8 == 0) tile = (bid % 8) * (nt / 8) + bid / 8;
  const int row0 = (tile % nM) * BM, col0 = (tile / nM) * kXBN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % (BM / 64), wn = wave / (BM / 64);
  const int li = lane & 15, lk = (lane >> 4) * 8;
  const int NB = a.T * a.Bp;

  // global -> register staging: A 2 x 16 bytes, B kNB x float4 per thread
  const int ar = tid >> 2, ac = tid & 3;       // A chunk: rows ar + kAR*j, bf16 8*ac
  const int bc = tid & 7, bcl = tid >> 3;      // B chunk: columns bcl + kBR*j, floats 4*bc
  // x offsets: row 0 stands in for padding columns, whose values are
  // replaced by zeros at the stash (so that no use of a fetched value precedes
  // it); the host guarantees T*B*D < 2^31 and rows*Dp < 2^31
  // 32-bit lane offsets (elements): the fetches below address a uniform base
  // plus these, so no per-fetch 64-bit address arithmetic is needed
  unsigned aoff[2], xoff[kNB];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    // output row g*km + n is panel row g*Kp + n (km: terms per group of this run)
    const int km = a.pld / a.G, r = min(row0 + ar + kAR * j, a.pld - 1);
    aoff[j] = (unsigned)((r / km) * a.Kp + r % km) * (unsigned)a.Dp + 8u * ac;
  }
  unsigned live = 0;
#pragma unroll
  for (int j = 0; j < kNB; ++j) {
    const int col = col0 + bcl + kBR * j;
    const int t = col / a.Bp, b = col - t * a.Bp;
    const bool l = col < NB && b < a.B;
    live |= (l ? 1u : 0u) << j;
    xoff[j] = (l ? (unsigned)((t * a.B + b) * a.D) : 0u) + 4u * bc;
  }
  u32x4 ra[2][2];
  f32x4 rb[2][kNB];
  const int nsplit = a.xsplit > 1 ? a.xsplit : 1;
  const int nS = a.Dp / kXBK / nsplit;   // slices of this part (even)
  const int kbase = part * nS * kXBK;
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // slice s lives in register set s & 1 from its fetch (issued before the
  // multiplication of slice s-2) until its stash into LDS buffer s & 1 (after
  // the multiplication of slice s-1): two multiplications hide each fetch.
  // A slice is one MFMA contraction step (32).
#define XPROJ_FETCH(R, S)                                                                              \
  do {                                                                                                 \
    const int k0 = kbase + (S) * kXBK;                                                                 \
    const uint16_t* va_ = a.Vx + k0;                                                                   \
    _Pragma("unroll") for (int j = 0; j < 2; ++j) ra[R][j] =                                           \
        *reinterpret_cast<const u32x4*>(va_ + aoff[j]);                                                \
    if constexpr (VEC) {                                                                               \
      const float* xa_ = a.x + k0;                                                                     \
      _Pragma("unroll") for (int j = 0; j < kNB; ++j)                                                    \
          rb[R][j] = *reinterpret_cast<const f32x4*>(xa_ + xoff[j]);                                   \
    } else {                                                                                           \
      const int k = k0 + 4 * bc;                                                                       \
      _Pragma("unroll") for (int j = 0; j < kNB; ++j) {                                                  \
        const float* q = a.x + (xoff[j] - 4u * bc);                                                    \
        const bool l = ((live >> j) & 1u) != 0;                                                        \
        rb[R][j] = f32x4{l && k < a.D ? q[k] : 0.f, l && k + 1 < a.D ? q[k + 1] : 0.f,                 \
                         l && k + 2 < a.D ? q[k + 2] : 0.f, l && k + 3 < a.D ? q[k + 3] : 0.f};        \
      }                                                                                                \
    }                                                                                                  \
  } while (0)
#define XPROJ_STASH(R)                                                                                 \
  do {                                                                                                 \
    _Pragma("unroll") for (int j = 0; j < 2; ++j)                                                      \
        *reinterpret_cast<u32x4*>(&As[R][(ar + kAR * j) * kXLD + 8 * ac]) = ra[R][j];                   \
    _Pragma("unroll") for (int j = 0; j < kNB; ++j) {                                                    \
      const f32x4 v = ((live >> j) & 1u) ? rb[R][j] : f32x4{0.f, 0.f, 0.f, 0.f};                       \
      const uint32_t lo = bf16_bits(v[0]) | ((uint32_t)bf16_bits(v[1]) << 16);                         \
      const uint32_t hi = bf16_bits(v[2]) | ((uint32_t)bf16_bits(v[3]) << 16);                         \
      *reinterpret_cast<u32x2*>(&Bs[R][(bcl + kBR * j) * kXLD + 4 * bc]) = u32x2{lo, hi};               \
    }                                                                                                  \
  } while (0)

#define XPROJ_MUL(BUF)                                                                                 \
  do {                                                                                                 \
    bf16x8 A[4], Bv[4];                                                                                \
    _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                      \
        A[i] = *reinterpret_cast<const bf16x8*>(&As[BUF][(wm * 64 + 16 * i + li) * kXLD + lk]);        \
    _Pragma("unroll") for (int j = 0; j < 4; ++j)                                                      \
        Bv[j] = *reinterpret_cast<const bf16x8*>(&Bs[BUF][(wn * 64 + 16 * j + li) * kXLD + lk]);       \
    _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                      \
        _Pragma("unroll") for (int j = 0; j < 4; ++j) acc[i][j] = mfma(A[i], Bv[j], acc[i][j]);        \
  } while (0)

  // nS is even (Dp is a multiple of 2 slices): the steady-state loop handles
  // a pair of slices with no conditions, the last pair is peeled
  XPROJ_FETCH(0, 0);
  XPROJ_FETCH(1, 1);
  XPROJ_STASH(0);
  lds_barrier();
  // sched_barrier keeps the compiler from hoisting a stash (which must wait
  // for its fetch) above the multiplication it is meant to overlap
  for (int ss = 0; ss + 2 < nS; ss += 2) {
    XPROJ_FETCH(0, ss + 2);   // set 0 was stashed before the last barrier
    __builtin_amdgcn_sched_barrier(0);
    XPROJ_MUL(0);             // slice ss
    __builtin_amdgcn_sched_barrier(0);
    XPROJ_STASH(1);           // slice ss+1; buffer 1's readers passed the last barrier
    lds_barrier();
    XPROJ_FETCH(1, ss + 3);
    __builtin_amdgcn_sched_barrier(0);
    XPROJ_MUL(1);             // slice ss+1
    __builtin_amdgcn_sched_barrier(0);
    XPROJ_STASH(0);           // slice ss+2
    lds_barrier();
  }
  XPROJ_MUL(0);               // slice nS-2
  XPROJ_STASH(1);             // slice nS-1
  lds_barrier();
  XPROJ_MUL(1);
#undef XPROJ_MUL
#undef XPROJ_FETCH
#undef XPROJ_STASH
  // P is column-major in r: the 4 result rows a lane holds are adjacent
  float* dst = nsplit > 1 ? a.Ppart + (size_t)part * NB * a.pld : a.P;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = row0 + wm * 64 + 16 * i + (lane >> 4) * 4;
    if (row >= a.rows) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = col0 + wn * 64 + 16 * j + li;
      if (col < NB)
        *reinterpret_cast<f32x4*>(dst + (size_t)col * a.pld + row) = acc[i][j];
    }
  }
}

// P = Ppart[0] + Ppart[1] + ... in part order, over the [T*Bp][pld] entries
// (pld is a multiple of 32: whole float4s).
__global__ void __launch_bounds__(256) batched_xproj_sum_kernel(BatchedArgs a) {
  const size_t stride = (size_t)a.T * a.Bp * a.pld;
  const size_t n4 = stride / 4;
  const f32x4* src = reinterpret_cast<const f32x4*>(a.Ppart);
  f32x4* out = reinterpret_cast<f32x4*>(a.P);
  for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 256) {
    f32x4 v = src[i];
    for (int k = 1; k < a.xsplit; ++k) v += src[k * (stride / 4) + i];
    out[i] = v;
  }
}

// ---------------------------------------------------------------- h-projection
// z of timestep t for panel rows [32*blockIdx.x, +32) and sequences
// [32*blockIdx.y, +32): z[tau][b] = sigma_tau (P[t*Bp+b] of tau + Vh[tau][:] .
// h[b][:]) for tau < GKl, 0 for the padding rows; stored as bf16 in
// Z[g][b][n] (tau = n*G + g).  The contraction over H is split over the 4
// waves (k-steps w, w+4, ...), each issuing the loads of up to 4 k-steps
// before its MFMAs; the partial tiles are summed in LDS.
__global__ void __launch_bounds__(256) batched_hproj_kernel(BatchedArgs a, int t, int GKl, int first) {
  __shared__ float red[4][32][33];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tau0 = blockIdx.x * 32, b0 = blockIdx.y * 32;
  const int li = lane & 15, lk = (lane >> 4) * 8;
  // epilogue mapping: thread -> one sequence b and 4 terms with consecutive n
  // of one group g; its P and sigma values are fetched first so that their
  // latency overlaps the contraction
  const int b = tid >> 3, jj = tid & 7;
  int g, nl0;
  if (a.G == 4) { g = jj >> 1; nl0 = (jj & 1) * 4; } else { g = 0; nl0 = jj * 4; }
  const float* prow = a.P + (size_t)(t * a.Bp + b0 + b) * a.pld;
  float pv[4], sg[4];
  const int lgG = a.G == 4 ? 2 : 0;
  // terms n0 .. n0+3 of the group (in the panel's padding past the budget)
  const f32x4 p4 = *reinterpret_cast<const f32x4*>(prow + g * (a.pld >> lgG) + (tau0 >> lgG) + nl0);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int tau = tau0 + (nl0 + i) * a.G + g;
    const bool live = tau < GKl;
    pv[i] = live ? p4[i] : 0.0f;
    sg[i] = live ? a.sigma[tau] : 0.0f;
  }
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nks = first ? 0 : (a.Hp >> 5);            // h_{-1} = 0: nothing to contract
  const uint16_t* va = a.Vh + (size_t)(tau0 + li) * a.Hp + lk;
  const uint16_t* hbp = a.hb + (size_t)(b0 + li) * a.Hp + lk;
  for (int base = wave; base < nks; base += 16) {
    bf16x8 A[4][2], Bv[4][2];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int ks = base + 4 * c;
      if (ks < nks) {
#pragma unroll
        for (int i = 0; i < 2; ++i) A[c][i] = load8(va + (size_t)16 * i * a.Hp + 32 * ks);
#pragma unroll
        for (int j = 0; j < 2; ++j) Bv[c][j] = load8(hbp + (size_t)16 * j * a.Hp + 32 * ks);
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (base + 4 * c < nks)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = mfma(A[c][i], Bv[c][j], acc[i][j]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][16 * i + (lane >> 4) * 4 + r][16 * j + li] = acc[i][j][r];
  lds_barrier();
  uint16_t zb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int tl = (nl0 + i) * a.G + g;                 // tau within the tile
    const float s = red[0][tl][b] + red[1][tl][b] + red[2][tl][b] + red[3][tl][b];
    zb[i] = bf16_bits(sg[i] * (pv[i] + s));             // 0 for tau >= GKl
  }
  const int n0 = tau0 / a.G + nl0;
  *reinterpret_cast<u32x2*>(a.Z + ((size_t)g * a.Bp + b0 + b) * a.Kp + n0) =
      u32x2{zb[0] | ((uint32_t)zb[1] << 16), zb[2] | ((uint32_t)zb[3] << 16)};
}

// ---------------------------------------------------------------- accumulation
// y of timestep t and the cell update for hidden units [16*blockIdx.x, +16)
// and sequences [32*blockIdx.y, +32).  8 waves: wave w takes gate q = w & 3
// (rows q*H + r of U, z of group g(q)) and the k-steps of parity w >> 2,
// issuing the loads of up to 8 k-steps before its MFMAs; the halves and the
// four gates meet in LDS for the c/h update.
__global__ void __launch_bounds__(512) batched_accum_kernel(BatchedArgs a, int t, int Kl32, int level, int first) {
  __shared__ float red[8][16][33];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int q = wave & 3, half = wave >> 2;
  const int r0 = blockIdx.x * 16, b0 = blockIdx.y * 32;
  const int li = lane & 15, lk = (lane >> 4) * 8;
  const int g = (a.G == 4) ? q : 0;
  // epilogue operands first (their latency overlaps the contraction)
  const int rr = tid & 15, bb = tid >> 4;
  const int r = r0 + rr, b = b0 + bb;
  const bool unit = r < a.H;
  const int rs = unit ? r : 0;
  const float bi = a.bias[0 * a.H + rs], bf = a.bias[1 * a.H + rs];
  const float bg = a.bias[2 * a.H + rs], bo = a.bias[3 * a.H + rs];
  const float cprev = first ? 0.0f : a.c[(size_t)b * a.H + rs];
  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  const int ru = r0 + li;
  const uint16_t* ua = a.Ut + (size_t)(q * a.H + (ru < a.H ? ru : 0)) * a.Kp + lk;
  const uint16_t* zp = a.Z + ((size_t)g * a.Bp + b0 + li) * a.Kp + lk;
  const int nks = Kl32 >> 5;
  for (int base = half; base < nks; base += 16) {
    bf16x8 A[8], Bv[8][2];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int ks = base + 2 * c;
      if (ks < nks) {
        A[c] = load8(ua + 32 * ks);
#pragma unroll
        for (int j = 0; j < 2; ++j) Bv[c][j] = load8(zp + (size_t)16 * j * a.Kp + 32 * ks);
      }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c)
      if (base + 2 * c < nks)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j] = mfma(A[c], Bv[c][j], acc[j]);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int k = 0; k < 4; ++k) red[wave][(lane >> 4) * 4 + k][16 * j + li] = acc[j][k];
  lds_barrier();
  if (!unit) return;
  const float yi = red[0][rr][bb] + red[4][rr][bb] + bi;
  const float yf = red[1][rr][bb] + red[5][rr][bb] + bf;
  const float yg = red[2][rr][bb] + red[6][rr][bb] + bg;
  const float yo = red[3][rr][bb] + red[7][rr][bb] + bo;
  const float c = sigmoid_b(yf) * cprev + sigmoid_b(yi) * tanh_b(yg);
  const float h = sigmoid_b(yo) * tanh_b(c);
  a.c[(size_t)b * a.H + r] = c;
  a.hb[(size_t)b * a.Hp + r] = bf16_bits(h);
  if (b < a.B) {
    a.h_out[(((size_t)level * a.T + t) * a.B + b) * a.H + r] = h;
    if (a.c_out && t == a.T - 1) a.c_out[((size_t)level * a.B + b) * a.H + r] = c;
  }
}

// initial state given by the caller: hb = bf16(h0), c = c0 (zeros where one
// of them is null; padding sequences zero; padding columns of hb untouched,
// they stay zero from allocation)
__global__ void batched_init_kernel(BatchedArgs a) {
  const int n = a.Bp * a.H;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int b = i / a.H, r = i - b * a.H;
    const bool live = b < a.B;
    a.hb[(size_t)b * a.Hp + r] = bf16_bits((live && a.h0) ? a.h0[(size_t)b * a.H + r] : 0.0f);
    a.c[(size_t)b * a.H + r] = (live && a.c0) ? a.c0[(size_t)b * a.H + r] : 0.0f;
  }
}

// ---------------------------------------------------------------- persistent recurrence
// The whole recurrence of one level in one launch.  Sequences go in cohorts
// of 16 (one MFMA tile wide); a cohort is run by a group of W workgroups of 8
// waves, workgroup w owning hidden units [32w, 32w+32) of all four gates.
// Every wave keeps two operand slices in registers for the whole launch:
//   * one h-projection tile: the 16 terms (g, n0 .. n0+15) of tile w*8 + wave
//     (tiles numbered group-major, so the 4 results a lane holds are
//     consecutive n of one group), their Vh rows over all of H;
//   * one accumulation tile: U rows q*H + 32w + 16*(wave>>2) + (0..15) of gate
//     q = wave & 3 over the K terms of group g(q).
// Per timestep: z tile = sigma (P + Vh . h_{t-1}) -> bf16, published to the
// group; every workgroup gathers all z of the cohort into LDS; y = U . z +
// bias on MFMA; the cell update (one thread per (unit, sequence), c in a
// register); h to h_out and, as bf16, published to the group; every
// workgroup gathers h_t into LDS.  P of the next timestep is fetched before
// the h-projection, so that it has arrived when the exchange polls (loads
// complete in order).
//
// What bounds a timestep is the two exchanges.  They are those of the pair
// kernel: a group sits on one XCD (two cohorts of 16 workgroups fill its 32
// compute units at H = 512), values travel through its L2 as plain stores
// (agent scope where a group finds itself on several XCDs), in slots that are
// empty until written: pairs of bf16 here, polled 16 bytes (eight values) at a
// time.  Everyone publishes h (every workgroup owns units) and polls both z and
// h, but a workgroup may own no z (its eight waves take the first tiles that are
// left, so at K < H the later workgroups have none).  So only h tells what a
// workgroup has read: once everyone's h_{t-1} is here, everyone has read z_{t-1}
// and h_{t-2}.  z_{t-1} is emptied beside z_t, its store waited for before h_t is
// published, and z_{t+1}, in its place, is polled by those who have h_t: two
// halves.  h_{t-2} is emptied beside h_t, its store waited for before h_{t+1} is
// published, and h_{t+2}, in its place, is polled by those who have h_{t+1}: four
// parts (with three, and the store before h_t, 132 us instead of 128 at the
// sizes below).  MI355X, H = 512, 256
// sequences, 16 timesteps, K = 512: flagged and tagged exchanges between XCDs
// 150 us, now 80; per timestep h-projection 0.6, z 1.5 (64 KB to every
// workgroup), accumulation and cell 0.9, h 0.9 us.
//
// The group's workgroups must be resident at once; if they are not within a
// second the group leaves and the error word is set.
constexpr int kMaxKs = 16;     // register-resident contraction steps of 32 (H and K up to 512)
constexpr int kZUnits = 8;     // 16-byte units of z polled per thread (G * K up to 2048 terms of 16 sequences)
constexpr int kHUnits = 2;     // and of h (H up to 512)
constexpr int kHParts = kBatchedHParts;
constexpr unsigned kCohortWait = 100000000u;   // wall ticks (a second)

__device__ __forceinline__ unsigned full_pair(unsigned v) { return v == kEmpty ? 0x7FC07FC0u : v; }

// two slots (four bf16), 8-byte aligned
__device__ __forceinline__ void store_slots(uint16_t* p, unsigned lo, unsigned hi, bool near) {
  const unsigned long long v = ((unsigned long long)hi << 32) | lo;
  unsigned long long* q = reinterpret_cast<unsigned long long*>(p);
  if (near) __hip_atomic_store(q, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(q, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// LDS bytes of a persistent launch with kh and ku contraction steps (h and z
// tiles, y staging, start mode)
__host__ __device__ inline size_t persistent_lds(int G, int kh, int ku) {
  return (size_t)2 * kCohort * ((32 * kh + 8) + (size_t)G * (32 * ku + 8)) + sizeof(float) * 4 * 32 * 17 + 16;
}

// contraction steps a wave holds: the smallest of 4, 8 and 16 that covers n
__host__ inline int step_bucket(int n) { return n <= 4 ? 4 : n <= 8 ? 8 : 16; }

// KH and KU: contraction steps of 32 over H and over the terms, held in
// registers; steps past Hp and Kl32 multiply zeros by zeros.  (With the counts
// at run time every step waited for its own LDS read: h-projection 1.1 us
// instead of 0.6 at H = 512.)
template <int KH, int KU>
__global__ void __launch_bounds__(512) batched_persistent_kernel(BatchedArgs a, int K, int Kl32, int level,
                                                                 int W, int slots, int nx) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  // groups are dealt to nx XCDs (consecutive blocks go to the XCDs in turn)
  const int x = blockIdx.x % nx, i0 = blockIdx.x / nx;
  const int slot = x + nx * (i0 / W), w = i0 % W;
  if (slot >= slots) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lq = lane >> 4, lk = lq * 8;
  const int G = a.G, H = a.H, Hp = a.Hp, Kp = a.Kp;
  constexpr int hld = 32 * KH + 8, zld = 32 * KU + 8;
  uint16_t* hs = reinterpret_cast<uint16_t*>(lds_raw);                      // [16][hld]
  uint16_t* zs = hs + kCohort * hld;                                        // [G][16][zld]
  float* ys = reinterpret_cast<float*>(zs + (size_t)G * kCohort * zld);     // [4][32][17]
  int* modes = reinterpret_cast<int*>(ys + 4 * 32 * 17);
  // the group's exchange: z [2][G*16][Kl32], h [4][16][Hp]
  const int zhalf = G * kCohort * Kl32, hpart = kCohort * Hp;
  uint16_t* zx = a.zx + (size_t)slot * 2 * G * kCohort * Kp;
  uint16_t* hx = a.hx + (size_t)slot * kHParts * hpart;
  unsigned long long* hand = a.ctl + (size_t)slot * kCtlWords;
  unsigned long long* decide = hand + kNearWidth;
  const int nkh = Hp >> 5, nku = Kl32 >> 5;   // live steps
  const int u0 = w * 32;
  const bool exch = K > 0;   // without terms no workgroup reads another's z or h

  if (exch) {
    // this workgroup's share of the slots empty before the others hear of it
    for (int i = w * 512 + tid; i < zhalf; i += W * 512)   // two halves of zhalf / 2 words
      store_slot(reinterpret_cast<float*>(zx) + i, kEmpty, false);
    for (int i = w * 512 + tid; i < kHParts * hpart / 2; i += W * 512)
      store_slot(reinterpret_cast<float*>(hx) + i, kEmpty, false);
    wait_memory();
    lds_barrier();
    if (wave == 7) {
      const int mode = group_start(hand, decide, w, W, a.tag_base | 0xFFFFu, kCohortWait, a.err);
      if (lane == 0) modes[0] = mode;
    }
  } else if (tid == 0) {
    modes[0] = kNear;
  }

  // h-projection tile of this wave and its operands
  const int ntn = Kl32 >> 4;
  const int tile = w * 8 + wave;
  const bool has_tile = tile < G * ntn;
  const int tg = has_tile ? tile / ntn : 0, tn0 = has_tile ? (tile - tg * ntn) * 16 : 0;
  bf16x8 va[KH];
#pragma unroll
  for (int ks = 0; ks < KH; ++ks) {
    va[ks] = bf16x8{};
    if (has_tile && ks < nkh) va[ks] = load8(a.Vh + (size_t)((tn0 + li) * G + tg) * Hp + 32 * ks + lk);
  }
  float sg[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int n = tn0 + 4 * lq + r;
    sg[r] = (has_tile && n < K) ? a.sigma[n * G + tg] : 0.0f;
  }
  // accumulation tile of this wave
  const int q = wave & 3, half16 = wave >> 2;
  const int urow = u0 + 16 * half16 + li;
  bf16x8 ua[KU];
#pragma unroll
  for (int ks = 0; ks < KU; ++ks) {
    ua[ks] = bf16x8{};
    if (urow < H && ks < nku) ua[ks] = load8(a.Ut + (size_t)(q * H + urow) * Kp + 32 * ks + lk);
  }
  const int zg = (G == 4) ? q : 0;
  // cell-update role: unit u0 + (tid >> 4), sequence tid & 15 of the cohort
  const int ul = tid >> 4, gs = tid & 15;
  const int gu = u0 + ul;
  const bool gu_live = gu < H;
  const int gur = gu_live ? gu : 0;
  const float bi = a.bias[gur], bfg = a.bias[H + gur], bgg = a.bias[2 * H + gur], bo = a.bias[3 * H + gur];
  // exchange roles: unit tid + 512 r of z (row of Kl32 / 8 units) and of h
  int zdst[kZUnits], hdst[kHUnits];
  unsigned zpend = 0, hpend = 0;
#pragma unroll
  for (int r = 0; r < kZUnits; ++r) {
    const int u = tid + 512 * r, row = Kl32 ? u / (Kl32 >> 3) : 0;
    if (8 * u < zhalf) zpend |= 1u << r;
    zdst[r] = 8 * u < zhalf ? (row * zld + 8 * (u - row * (Kl32 >> 3))) >> 1 : 0;
  }
#pragma unroll
  for (int r = 0; r < kHUnits; ++r) {
    const int u = tid + 512 * r, row = u / (Hp >> 3);
    if (8 * u < hpart) hpend |= 1u << r;
    hdst[r] = 8 * u < hpart ? (row * hld + 8 * (u - row * (Hp >> 3))) >> 1 : 0;
  }
  // columns of z past Kl32 are never written and must read zero
  for (int i = tid; i < G * kCohort * zld / 2; i += 512) reinterpret_cast<unsigned*>(zs)[i] = 0u;
  const size_t zoff = (size_t)(tg * kCohort + li) * Kl32 + tn0 + 4 * lq;
  const size_t hoff = (size_t)gs * Hp + gu;   // even units carry the pair
  __syncthreads();
  const int mode = __builtin_amdgcn_readfirstlane(modes[0]);
  if (mode >= kAlone) {
    if (tid == 0) __hip_atomic_fetch_or(a.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  const bool near = mode == kNear;

  const int ncoh = (a.B + kCohort - 1) / kCohort;
  int par = 0, hpar = 0;   // timestep mod 2 and mod 4, counted over the group's cohorts
  for (int coh = slot; coh < ncoh; coh += slots) {
    const int b0 = coh * kCohort;
    // h_{-1}; columns past H are zero
    for (int i = tid; i < kCohort * 32 * KH; i += 512) {
      const int sq = i / (32 * KH), k = i - sq * (32 * KH);
      const int b = b0 + sq;
      const float v = (a.h0 && b < a.B && k < H) ? a.h0[(size_t)b * H + k] : 0.0f;
      hs[sq * hld + k] = bf16_bits(v);
    }
    float c = 0.0f;
    if (a.c0 && b0 + gs < a.B && gu_live) c = a.c0[(size_t)(b0 + gs) * H + gu];
    // P of the lane's 4 result terms (sequence li)
    const int km = a.pld / G;
    auto fetch_p = [&](int t) {
      return *reinterpret_cast<const f32x4*>(a.P + (size_t)(t * a.Bp + b0 + li) * a.pld + tg * km + tn0 + 4 * lq);
    };
    f32x4 pv = f32x4{0.f, 0.f, 0.f, 0.f};
    if (has_tile) pv = fetch_p(0);
    lds_barrier();
    for (int t = 0; t < a.T; ++t, par ^= 1, hpar = (hpar + 1) % kHParts) {
      uint16_t* zt = zx + par * zhalf;
      uint16_t* ht = hx + hpar * hpart;
      f32x4 pn = f32x4{0.f, 0.f, 0.f, 0.f};
      if (has_tile) pn = fetch_p(min(t + 1, a.T - 1));
      // ---- h-projection of the wave's tile, published as bf16
      if (has_tile) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KH; ++ks)
          acc = mfma(va[ks], *reinterpret_cast<const bf16x8*>(hs + li * hld + 32 * ks + lk), acc);
        unsigned zb[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) zb[r] = tn0 + 4 * lq + r < K ? bf16_bits(sg[r] * (pv[r] + acc[r])) : 0u;
        store_slots(zt + zoff, full_pair(zb[0] | (zb[1] << 16)), full_pair(zb[2] | (zb[3] << 16)), near);
        store_slots(zx + (par ^ 1) * zhalf + zoff, kEmpty, kEmpty, near);
      }
      pv = pn;
      if (exch) {
        poll_units<kZUnits>(reinterpret_cast<float*>(zs), reinterpret_cast<const float*>(zt), zhalf * 2, zdst, zpend,
                            a.err);
        wait_memory();   // the emptied slots too, before this workgroup's h_t
      }
      lds_barrier();
      // ---- y = U . z for the wave's rows
      {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KU; ++ks)
          acc = mfma(ua[ks], *reinterpret_cast<const bf16x8*>(zs + (zg * kCohort + li) * zld + 32 * ks + lk), acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) ys[(q * 32 + 16 * half16 + 4 * lq + r) * 17 + li] = acc[r];
      }
      lds_barrier();
      // ---- gates and cell update
      const float yi = ys[(0 * 32 + ul) * 17 + gs] + bi;
      const float yf = ys[(1 * 32 + ul) * 17 + gs] + bfg;
      const float yg = ys[(2 * 32 + ul) * 17 + gs] + bgg;
      const float yo = ys[(3 * 32 + ul) * 17 + gs] + bo;
      c = sigmoid_b(yf) * c + sigmoid_b(yi) * tanh_b(yg);
      const float h = sigmoid_b(yo) * tanh_b(c);
      const int b = b0 + gs;
      // the group's very last h is read by nobody
      const bool more = exch && (t + 1 < a.T || coh + slots < ncoh);
      if (more) {
        // units in pairs (lanes l and l+16 hold units 2m and 2m+1 of one
        // sequence); a unit past H travels as zero
        const unsigned hb = gu_live ? (unsigned)bf16_bits(h) : 0u;
        const unsigned hn = (unsigned)__shfl_down((int)hb, 16, 64);
        if ((lq & 1) == 0) {
          store_slot(reinterpret_cast<float*>(ht + hoff), full_pair(hb | (hn << 16)), near);
          store_slot(reinterpret_cast<float*>(hx + (hpar ^ 2) * hpart + hoff), kEmpty, near);   // h_{t-2}
        }
      }
      if (gu_live && b < a.B) {
        a.h_out[(((size_t)level * a.T + t) * a.B + b) * H + gu] = h;
        if (a.c_out && t == a.T - 1) a.c_out[((size_t)level * a.B + b) * H + gu] = c;
      }
      if (more) {
        poll_units<kHUnits>(reinterpret_cast<float*>(hs), reinterpret_cast<const float*>(ht), hpart * 2, hdst, hpend,
                            a.err);
        wait_memory();   // the emptied slots too, before this workgroup's h_{t+1}
      }
      lds_barrier();
    }
  }
}

// Whether the x-projection takes the 256-row tile, from the number of
// 128-row tiles: those run two to a compute unit, so r = ceil(tiles / units)
// of them take 58 us per two and 40 us for an odd one; half as many 256-row
// tiles run one to a unit, 48 us each.  Measured (D = 2048, narrow / wide,
// us): r = 1 40 / 46, r = 2 58.3 / 50.6 (53.2 / 47.9 at 320 tiles), r = 3
// 87.5-90.7 / 89.6-92.3, r = 4 112.5 / 96.7; D = 1000 (no float4 loads of x)
// r = 2 69.0 / 48.8.
static bool batched_xproj_wide(long long tiles, int ncu) {
  const long long r = (tiles + ncu - 1) / ncu;
  return r > 1 && r != 3;
}

int batched_xproj_split(int tiles, int ncu, int nslices) {
  int s = 1;
  while (2 * s <= 8 && (long long)tiles * 2 * s <= ncu && nslices % (4 * s) == 0) s *= 2;
  return s;
}

size_t batched_ppart_floats(int ncu) { return (size_t)std::max(1, ncu) * kXBM * kXBN; }

int plan_batched_persistent(const BatchedArgs& a, int K, int* W, int* slots) {
  const int Kl32 = ((K + 31) / 32) * 32;
  const int w = (a.H + 31) / 32;
  const int ncoh = (a.B + kCohort - 1) / kCohort;
  if (a.Hp > 32 * kMaxKs || Kl32 > 32 * kMaxKs || a.G * (Kl32 / 16) > 8 * w) return 0;
  if (w > a.max_wg || a.Bp % kCohort != 0) return 0;
  if (persistent_lds(a.G, step_bucket(a.Hp / 32), step_bucket(Kl32 / 32)) > kLdsCap) return 0;
  // whole groups per XCD (w <= 16)
  const int fit = a.max_wg >= kXcds * kXcdCus ? kXcds * (kXcdCus / w) : a.max_wg / w;
  const int s = std::max(1, std::min(ncoh, fit));
  *W = w;
  *slots = s;
  return 1;
}

namespace {

template <int KH, int KU>
hipError_t launch_persistent_steps(const BatchedArgs& p, int K, int Kl32, int level, int W, int slots, int nx,
                                   hipStream_t stream) {
  static bool attr = false;
  if (!attr) {
    const hipError_t e = hipFuncSetAttribute((const void*)batched_persistent_kernel<KH, KU>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsCap);
    if (e != hipSuccess) return e;
    attr = true;
  }
  batched_persistent_kernel<KH, KU><<<dim3(nx * W * ((slots + nx - 1) / nx)), dim3(512), persistent_lds(p.G, KH, KU),
                                      stream>>>(p, K, Kl32, level, W, slots, nx);
  return hipGetLastError();
}

template <int KH>
hipError_t launch_persistent_h(const BatchedArgs& p, int K, int Kl32, int level, int W, int slots, int nx,
                               hipStream_t stream) {
  switch (step_bucket(Kl32 / 32)) {
    case 4: return launch_persistent_steps<KH, 4>(p, K, Kl32, level, W, slots, nx, stream);
    case 8: return launch_persistent_steps<KH, 8>(p, K, Kl32, level, W, slots, nx, stream);
    default: return launch_persistent_steps<KH, 16>(p, K, Kl32, level, W, slots, nx, stream);
  }
}

hipError_t launch_persistent(const BatchedArgs& p, int K, int Kl32, int level, int W, int slots, int nx,
                             hipStream_t stream) {
  switch (step_bucket(p.Hp / 32)) {
    case 4: return launch_persistent_h<4>(p, K, Kl32, level, W, slots, nx, stream);
    case 8: return launch_persistent_h<8>(p, K, Kl32, level, W, slots, nx, stream);
    default: return launch_persistent_h<16>(p, K, Kl32, level, W, slots, nx, stream);
  }
}

}  // namespace

hipError_t launch_batched(const BatchedArgs& a, const int* levels, int n_levels, hipStream_t stream) {
  if (a.Bp % kBatchAlign != 0 || a.Bp < a.B || a.Bp > (1 << 20) || a.Dp % kPanelDAlign != 0 || a.Dp < a.D ||
      a.Hp % 32 != 0 || a.Hp < a.H || a.Kp % 32 != 0)
    return hipErrorInvalidValue;
  int kmax = 0;
  for (int l = 0; l < n_levels; ++l) kmax = std::max(kmax, levels[l]);
  if (kmax > a.Kp) return hipErrorInvalidValue;
  BatchedArgs p = a;
  p.pld = a.G * ((kmax + 31) / 32) * 32;                  // every term a level may use, padded
  hipError_t e;
  if (kmax > 0) {
    p.rows = p.pld;
    const int nN = (a.T * a.Bp + kXBN - 1) / kXBN;
    const bool wide = batched_xproj_wide((long long)((p.rows + kXBM - 1) / kXBM) * nN, a.ncu);
    const int bm = wide ? kXWide : kXBM, nM = (p.rows + bm - 1) / bm;
    p.xsplit = a.Ppart && !wide ? batched_xproj_split(nM * nN, a.ncu, a.Dp / kXBK) : 1;
    if (p.xsplit > 1 && (size_t)p.xsplit * a.T * a.Bp * p.pld > a.ppart_cap) p.xsplit = 1;
    const unsigned gx = (unsigned)(nM * nN * p.xsplit);
    const bool vec = a.xvec && a.D % kPanelDAlign == 0;
    const auto xproj = wide ? (vec ? batched_xproj_kernel<true, kXWide> : batched_xproj_kernel<false, kXWide>)
                            : (vec ? batched_xproj_kernel<true, kXBM> : batched_xproj_kernel<false, kXBM>);
    xproj<<<dim3(gx + (a.ctl ? 1 : 0)), dim3(2 * bm), 0, stream>>>(p, nM, nN);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (p.xsplit > 1) {
      const size_t n4 = (size_t)a.T * a.Bp * p.pld / 4;
      const unsigned gs = (unsigned)std::min<size_t>((n4 + 255) / 256, 2048);
      batched_xproj_sum_kernel<<<dim3(gs), dim3(256), 0, stream>>>(p);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  const bool init = a.h0 != nullptr || a.c0 != nullptr;
  for (int l = 0; l < n_levels; ++l) {
    const int K = levels[l];
    const int Kl32 = ((K + 31) / 32) * 32;
    p.rows = a.G * Kl32;
    int W = 0, slots = 0;
    if (a.zx && a.hx && a.ctl && a.err && plan_batched_persistent(p, K, &W, &slots)) {
      // one launch sequence number per level: its tags differ from every earlier launch's
      p.tag_base = a.tag_base + ((unsigned)l << 16);
      const int nx = a.ncu >= kXcds * kXcdCus ? kXcds : 1;
      if ((e = launch_persistent(p, K, Kl32, l, W, slots, nx, stream)) != hipSuccess) return e;
      continue;
    }
    if (init) {
      batched_init_kernel<<<dim3(128), dim3(256), 0, stream>>>(p);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    for (int t = 0; t < a.T; ++t) {
      const int first = (t == 0 && !init) ? 1 : 0;
      if (K > 0) {
        batched_hproj_kernel<<<dim3(p.rows / 32, a.Bp / 32), dim3(256), 0, stream>>>(p, t, a.G * K, first);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
      batched_accum_kernel<<<dim3((a.H + 15) / 16, a.Bp / 32), dim3(512), 0, stream>>>(p, t, Kl32, l, first);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

}  // namespace alstm
