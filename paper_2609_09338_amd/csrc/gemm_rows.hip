// Tiled matrix-core products for passes of more than 128 rows (prompts, large batches):
// Y[r][n] = sum_c X[r][c] W[n][c], bf16 weights, X as bf16 hi / lo pairs (taps: bf16).
//
// The kernel of gemm_mfma.h gives every 64 rows a block of their own, whose weights go
// straight from memory to registers, and splits K into 256-column pieces whatever the
// size: at thousands of rows each weight is read once per 64 rows and 8-16 partial sums
// of every output pass through memory.  Here a block computes 128 or 256 rows x 256 weight
// rows (a wavefront 64 x 128), and K is split only as far as it takes to fill the chip.  Per
// 32 columns a block copies its inputs (hi, lo) and 16 KB of weights straight into LDS
// (buffer loads to LDS, no registers) while it multiplies earlier columns; a wavefront reads
// 16 fragments from LDS for 64 products, about half of what the LDS delivers in that time.
// 128-row blocks run two to a CU with two stages each (64 KB of LDS, 2 wavefronts per SIMD)
// and cover each other's barriers, but a copy has one step to arrive; 256-row blocks have the
// CU to themselves and three stages (144 KB), so that a copy has two steps: each step waits
// for copies requested two steps before (in one step of three the compiler, which cannot tell
// the stages apart there, adds a wait for those of one step before).  16-byte pieces are permuted within a row by the row, so that the 16 rows of a
// fragment read fall into different banks.
//
// The weights are the A operand, so a lane ends with four consecutive output columns of
// one row: float4 stores of partial sums, and for gate/up (a wavefront holds the gate and
// the up tile of the same columns) silu(g) u in registers, written as the down
// projection's hi / lo input without the row kernel and its 2 x 2 F floats per row.
// Blocks go to the XCDs in contiguous ranges of tiles, 1024 rows by rising weight
// tile, so that an XCD's blocks share inputs and weights in its L2.
// Bound by the matrix cores (two products per weight: hi and lo inputs).  Measured, the kernel
// of gemm_mfma.h / this one: gate/up of 8200 rows (2 x 9728 x 2560) 4256 us and 1358 us of
// SwiGLU rows / 1258 us (1.30 PFLOP/s of products; a large library bf16 product reaches 1.19 on
// this card), QKV (6144 x 5120) 2435 / 939 us, taps (2560 x 12288) 2226 / 580 us; 1999 rows of
// the 1024-wide body: QKV 176 / 60, gate/up 114 + 32 / 61, down 66 / 39, taps 226 / 62.
// K is summed whole in fp32 instead of in 256-column partials: keys and values of prompts next
// to a rounding boundary fall to the other bf16 neighbour, and a prompt's distance from 64 bits
// goes from 1.19e-4 to 1.24e-4 (1999 tokens) and from 1.75e-4 to 1.79e-4 (8200, d 2560).
#include "common.h"
#include "internal.h"

#include <algorithm>

namespace osp {

typedef __bf16 gr_bf16x8 __attribute__((ext_vector_type(8)));
typedef float gr_f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned gr_u32x4 __attribute__((ext_vector_type(4)));

constexpr int kGrM = 64;         // input rows per wavefront (two or four wavefronts of a block)
constexpr int kGrN = 256;        // weight rows per block
constexpr int kGrK = 32;         // columns per step
constexpr int kGrP = kGrK / 8;   // 16-byte pieces per row and step
constexpr int kGrGroup = 1024;   // rows walked together
constexpr int kGrXcd = 8;

// Where piece c of row r of a tile lies: four pieces per 64-byte row, permuted so that the
// same piece of eight consecutive rows covers every bank once.
OSP_DEV int gr_slot(int r, int c) { return r * kGrP + (c ^ ((r >> 1) & 3)); }

OSP_DEV void gr_copy(const void* base, gr_u32x4* lds, int voffset, int soffset) {
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7fffffff, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)lds, 16, voffset, soffset,
                                           0, 0);
}

template <int SRC, int EPI, int WM>
__global__ void __launch_bounds__(128 * WM, 2) k_gemm_rows(GemvArgs a, int mt, int nt, int ks, int steps_per_split,
                                                      int fused) {
  constexpr bool EXACT_X = SRC == SRC_TAPS;   // inputs already bf16: no lo part
  constexpr int TM = WM * kGrM;               // input rows per block
  constexpr int XT = TM * kGrP;               // pieces of one input tile
  constexpr int ST = (EXACT_X ? 1 : 2) * XT + kGrN * kGrP;
  constexpr int WR = kGrN / (2 * WM);         // weight rows a wavefront brings
  constexpr int CP = (EXACT_X ? 2 : 4) + WR / 16;   // copies of a wavefront and step
  constexpr bool THREE = WM == 4;             // three stages
  static_assert(CP < 16, "the copies of a step fit the low bits of the wait's vector-memory count");
  __shared__ __attribute__((aligned(16))) gr_u32x4 st0[ST];
  __shared__ __attribute__((aligned(16))) gr_u32x4 st1[ST];
  __shared__ __attribute__((aligned(16))) gr_u32x4 st2[THREE ? ST : 1];

  // ---- this block's tile ------------------------------------------------------------------
  const int tiles = mt * nt, per = (tiles * ks + kGrXcd - 1) / kGrXcd;
  const int id = (int)(blockIdx.x % kGrXcd) * per + (int)(blockIdx.x / kGrXcd);
  if (id >= tiles * ks) return;
  const int split = id / tiles, t = id % tiles;
  constexpr int GT = kGrGroup / TM;           // row tiles walked together
  const int g0 = t / (GT * nt) * GT, gm = min(GT, mt - g0);
  const int tg = t - g0 * nt;
  const int m0 = (g0 + tg % gm) * TM, nb = tg / gm;
  const int rows = a.count ? min(*a.count, a.max_rows) : a.max_rows;
  if (m0 >= rows) return;
  const int n0 = nb * (EPI == EPI_SWIGLU ? kGrN / 2 : kGrN);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row = lane & 15, grp = lane >> 4;
  const int k_beg = split * steps_per_split;
  const int steps = min(steps_per_split, a.Kd / kGrK - k_beg);

  // ---- copies: an instruction fills 16 rows (64 bytes each); a wavefront brings 32 input
  //      rows and WR weight rows of every step.  Rows past the end repeat the last one ---------
  const int cr = lane >> 2;                  // row within an instruction's 16
  int xo[2], wo[WR / 16];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = (wave * 2 + i) * 16 + cr;  // row of the tile
    const int m = min(m0 + r, rows - 1);
    const long ld = SRC == SRC_TAPS ? a.ldt : a.ld_xa;
    const long src = SRC == SRC_TAPS ? a.tap_row[m] : m;
    xo[i] = (int)(src * ld * 2) + (((lane & 3) ^ ((r >> 1) & 3)) * 16);
  }
  // gate/up: the tile's rows are 64 gate rows, the up rows of the same columns, and so on
  const int w64 = wave * WR / 64;
  const void* wbase = (EPI == EPI_SWIGLU && (w64 & 1)) ? a.w1 : a.w0;
#pragma unroll
  for (int i = 0; i < WR / 16; ++i) {
    const int r = i * 16 + cr;
    const int n = min(n0 + (EPI == EPI_SWIGLU ? (w64 >> 1) * 64 + wave * WR % 64 : wave * WR) + r, a.N - 1);
    wo[i] = (int)((long)n * a.Kd * 2) + (((lane & 3) ^ ((r >> 1) & 3)) * 16);
  }
  auto copy_step = [&](gr_u32x4* st, int k) {
    const int col = (k_beg + k) * kGrK;
    if constexpr (SRC == SRC_TAPS) {
#pragma unroll
      for (int i = 0; i < 2; ++i) gr_copy(a.taps, st + (wave * 2 + i) * 64, xo[i], col * 2);
    } else {
      const bool s = col < a.seg;            // (segments are whole steps)
      const void* xh = s ? a.xs_hi : a.xa_hi;
      const void* xl = s ? a.xs_lo : a.xa_lo;
      const int so = (s ? col : col - a.seg) * 2;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        gr_copy(xh, st + (wave * 2 + i) * 64, xo[i], so);
        gr_copy(xl, st + XT + (wave * 2 + i) * 64, xo[i], so);
      }
    }
#pragma unroll
    for (int i = 0; i < WR / 16; ++i)
      gr_copy(wbase, st + (ST - kGrN * kGrP) + (wave * (WR / 16) + i) * 64, wo[i], col * 2);
  };

  // ---- products: wavefront (wm, wn) computes rows 64 wm .., weight rows 128 wn .. -----------
  const int wm = wave % WM, wn = wave / WM;
  const bool work = m0 + wm * 64 < rows;
  gr_f32x4 acc[8][4];
#pragma unroll
  for (int n = 0; n < 8; ++n)
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[n][m] = gr_f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const gr_u32x4* st) {
    if (!work) return;
    gr_bf16x8 xh[4], xl[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int s = gr_slot(wm * 64 + 16 * m + row, grp);
      xh[m] = __builtin_bit_cast(gr_bf16x8, st[s]);
      if constexpr (!EXACT_X) xl[m] = __builtin_bit_cast(gr_bf16x8, st[XT + s]);
    }
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const gr_bf16x8 w =
          __builtin_bit_cast(gr_bf16x8, st[(ST - kGrN * kGrP) + gr_slot(wn * 128 + 16 * n + row, grp)]);
#pragma unroll
      for (int m = 0; m < 4; ++m) acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, xh[m], acc[n][m], 0, 0, 0);
      if constexpr (!EXACT_X)
#pragma unroll
        for (int m = 0; m < 4; ++m) acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, xl[m], acc[n][m], 0, 0, 0);
    }
  };

  // ---- two stages: one fills while the other is multiplied (the barrier waits for the
  //      copies); the stages are arrays of their own, so that reads of one do not wait for
  //      the copies into the other ----------------------------------------------------------
  if constexpr (THREE) {
    // Step k: its copies (requested two steps ahead) have arrived when no more than the next
    // step's are outstanding, and this wavefront's reads of the stage of step k - 1 when no
    // LDS request is; past the barrier both hold for every wavefront, and the copies of step
    // k + 2 go into the stage of step k - 1 (past the end the last step's again, so that the
    // count stays the same).  Without the second wait only the instruction order that the
    // compiler happens to choose would keep a late read apart from the next copy.
    auto step = [&](gr_u32x4* cur, gr_u32x4* next, int k) {
      // vmcnt(CP) lgkmcnt(0), the export counter at its maximum
      __builtin_amdgcn_s_waitcnt(0x0070 | CP);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      copy_step(next, min(k + 2, steps - 1));
      compute(cur);
    };
    copy_step(st0, 0);
    copy_step(st1, min(1, steps - 1));
    for (int k = 0; k < steps; k += 3) {
      step(st0, st2, k);
      if (k + 1 >= steps) break;
      step(st1, st0, k + 1);
      if (k + 2 >= steps) break;
      step(st2, st1, k + 2);
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // no copy into LDS outlives the block
  } else {
  copy_step(st0, 0);
  __syncthreads();
  for (int k = 0; k < steps; k += 2) {
    if (k + 1 < steps) copy_step(st1, k + 1);
    compute(st0);
    __syncthreads();
    if (k + 1 >= steps) break;
    if (k + 2 < steps) copy_step(st0, k + 2);
    compute(st1);
    __syncthreads();
  }
  }

  // ---- lane holds Y[row 16 m + lane % 16][columns 16 n + 4 (lane / 16) .. + 4) ---------------
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int r = m0 + wm * 64 + 16 * m + row;
    if (r >= rows) continue;
    if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int f = n0 + wn * 64 + 16 * i + 4 * grp;
        if (f >= a.N) continue;
        const gr_f32x4 g = acc[i][m], u = acc[4 + i][m];
        if (fused) {
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = g[e] / (1.0f + __expf(-g[e])) * u[e];
          uint32_t h[2], l[2];
          split_bf16x2(y[0], y[1], h[0], l[0]);
          split_bf16x2(y[2], y[3], h[1], l[1]);
          *reinterpret_cast<uint2*>(a.act_hi + (long)r * a.N + f) = make_uint2(h[0], h[1]);
          *reinterpret_cast<uint2*>(a.act_lo + (long)r * a.N + f) = make_uint2(l[0], l[1]);
        } else {
          float* p = a.split_buf + ((long)split * a.max_rows + r) * 2 * a.N + f;
          *reinterpret_cast<gr_f32x4*>(p) = g;
          *reinterpret_cast<gr_f32x4*>(p + a.N) = u;
        }
      }
    } else {
#pragma unroll
      for (int n = 0; n < 8; ++n) {
        const int c = n0 + wn * 128 + 16 * n + 4 * grp;
        if (c < a.N) *reinterpret_cast<gr_f32x4*>(a.split_buf + ((long)split * a.max_rows + r) * a.N + c) = acc[n][m];
      }
    }
  }
}

// K splits: as many as it takes to give every CU two blocks (of 256 rows: one), of at least
// four steps.
static int gemm_rows_splits(int tiles, int blocks, int Kd, int& steps_per_split) {
  const int steps = Kd / kGrK;
  int ks = std::max(1, std::min(std::min(blocks / tiles, steps / 4), kMaxKSplit));
  steps_per_split = (steps + ks - 1) / ks;
  return (steps + steps_per_split - 1) / steps_per_split;
}

// Passes of more than 128 rows (below, one 128-row tile leaves a wavefront pair idle and
// too few blocks: at 96 rows of width 1024 the products took 11.7-13.2 us against
// 11.3-12.1); whole 32-column steps, inputs and weights within the 2 GB a buffer offset reaches, on
// 16-byte boundaries (the copies into LDS move 16 bytes; rows are whole pieces, so the
// caller's taps and weights decide), and rows of equal stride in both input segments; other
// shapes keep the kernel of gemm_mfma.h.
bool gemm_rows_supported(SrcKind src, const GemvArgs& a, long input_rows) {
  const long ld = src == SRC_TAPS ? a.ldt : a.ld_xa;
  const auto at16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  return (src == SRC_TAPS || src == SRC_PREP) && a.max_rows > 2 * kGrM && a.Kd % kGrK == 0 && a.seg % kGrK == 0 && a.N % 4 == 0 && !a.gather &&
         (a.seg == 0 || a.ld_xs == a.ld_xa) && input_rows * ld * 2 < (1L << 31) && (long)a.N * a.Kd * 2 < (1L << 31) &&
         at16(a.w0) && at16(a.w1) && (src != SRC_TAPS || at16(a.taps));
}

// A launch's tiles of 64 WM rows (nper columns each), K splits, and its length: steps per
// CU, in those of a 128-row block.
struct GrPlan {
  int mt, nt, ks, sps;
  double cost;
};
static GrPlan gr_plan(int wm, int rows, int N, int nper, int Kd, int n_cu) {
  GrPlan p;
  p.mt = (rows + wm * kGrM - 1) / (wm * kGrM);
  p.nt = (N + nper - 1) / nper;
  p.ks = gemm_rows_splits(p.mt * p.nt, wm == 4 ? n_cu : 2 * n_cu, Kd, p.sps);
  const int per_cu = (p.mt * p.nt * p.ks + n_cu - 1) / n_cu;
  p.cost = (wm == 4 ? 2 * 0.93 : 1.0) * per_cu * p.sps;
  return p;
}

template <int SRC, int EPI, int WM>
static int launch_tile(const GemvArgs& a, const GrPlan& p, hipStream_t st) {
  const int grid = (p.mt * p.nt * p.ks + kGrXcd - 1) / kGrXcd * kGrXcd;
  const int fused = EPI == EPI_SWIGLU && p.ks == 1 && a.act_hi;
  hipLaunchKernelGGL((k_gemm_rows<SRC, EPI, WM>), dim3(grid), dim3(128 * WM), 0, st, a, p.mt, p.nt, p.ks, p.sps,
                     fused);
  return fused ? 0 : p.ks;
}

// 256-row blocks run a step 7% faster per row (gate/up of 8200 rows, d 2560: 1343 / 1258 us;
// taps of 1999 rows, d 1024: 74.5 / 62) where they fill their rounds of 256 CUs as well:
// 8200 rows make 792 of them for QKV (four rounds, 3.09 full: 20% slower than 1560 of 128
// rows) and 330 for the taps (598 -> 685 us), 300 rows leave 40% of two empty (a whole
// prompt 208 -> 225 us).
template <int SRC, int EPI>
static int launch_t(const GemvArgs& a, int n_cu, hipStream_t st) {
  const int nper = EPI == EPI_SWIGLU ? kGrN / 2 : kGrN;
  const GrPlan wide = gr_plan(4, a.max_rows, a.N, nper, a.Kd, n_cu), half = gr_plan(2, a.max_rows, a.N, nper, a.Kd, n_cu);
  return wide.cost < half.cost ? launch_tile<SRC, EPI, 4>(a, wide, st) : launch_tile<SRC, EPI, 2>(a, half, st);
}

int launch_gemm_rows(SrcKind src, EpiKind epi, const GemvArgs& a, int n_cu, hipStream_t st) {
  if (src == SRC_TAPS) return launch_t<SRC_TAPS, EPI_STORE>(a, n_cu, st);
  if (epi == EPI_SWIGLU) return launch_t<SRC_PREP, EPI_SWIGLU>(a, n_cu, st);
  return launch_t<SRC_PREP, EPI_STORE>(a, n_cu, st);
}

}  // namespace osp
