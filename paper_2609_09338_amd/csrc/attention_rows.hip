// Attention of passes with many query vectors per sequence (prompts, further turns,
// blocks): every query row attends causally over the sequence's pages, the new rows'
// keys and values already appended and their queries prepared (k_rows_qkv).
//
// k_attn_mfma reads a split's pages again for every 16 query vectors, one after another
// in one block: right for decoding, where a page serves few queries, but a 1999-token
// prompt (2 heads per kv head) took 250 such passes in each of 256 blocks, 1422 us per
// layer.  Here a block owns 64 QT query vectors of one kv head (rows x heads of its
// group) and walks the pages once, four pages (64 tokens) per step:
//   * the pages of the next step are loaded into registers while this step computes and
//     written to the other LDS buffer at its end: one barrier per step;
//   * a wavefront keeps its 16 QT queries (bf16 hi + lo) and their outputs in registers
//     and reads the shared pages from LDS: S^T = K Q^T (16x16x32), online softmax (a lane
//     owns one query and 16 tokens of the step), O^T += V^T P^T (16x16x32 over page
//     pairs, P as hi + lo).  The score tile's layout is the second product's B operand
//     when the K index runs over tokens 4 g .. 4 g + 3 of both pages of a pair, so
//     nothing moves between lanes but the row maxima and sums;
//   * key rows are stored with their 16-byte pieces permuted by the token, so that the
//     16 rows a fragment read touches fall into different banks.  Value pages are stored
//     in pairs, the four tokens of a lane's K index from both pages side by side: one read
//     and no register moves per value fragment.
// The matrix cores bound it (four products per score and value, hi and lo): registers
// hold two wavefronts per SIMD, so one's softmax overlaps another's products.
// Blocks are kv head, sequence, row tile (one grid dimension, the head innermost) and
// context split: heads go to the XCDs in turn, so each L2 holds the pages of the heads it
// serves, and the tiles of the longest contexts start first.  With one split the output is
// written directly (hi / lo pairs); a pass of too few tiles to fill the chip splits its
// context, and the merge kernel or the O projection joins the partials.
// Measured per layer, k_attn_mfma / this: one 1999-token prompt (16 / 8 heads x 128) 1422 / 65
// us; four of 8200 tokens in all (32 / 8 heads x 128) 5600 / 608 us; two turns of 770 tokens
// over 6000-8000 cached positions (16 / 8 x 128) 672 / 182 us; a 17-row block (32 / 8 x 64) 24.2
// / 11.9 us.
// (rocprofv3, the two turns: matrix cores busy 23% of the time, 3.4 vector instructions per
// product; on average one wavefront per SIMD of the two that fit.)
#include "common.h"
#include "internal.h"

#include <algorithm>

namespace osp {

typedef __bf16 ar_bf16x8 __attribute__((ext_vector_type(8)));
typedef float ar_f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned ar_u32x4 __attribute__((ext_vector_type(4)));

constexpr int kArTok = 64;   // tokens per step: a page per wavefront
constexpr int kArPage = 16;

template <int HD, int QT>
__global__ void __launch_bounds__(256, 2) k_attn_rows(AttnArgs a, int n_tiles, int tiles_x) {
  constexpr int KC = HD / 32;             // 32-wide head-dim chunks of K Q^T
  constexpr int NT = HD / 16;             // 16-dim output tiles
  constexpr int KROW = HD / 8;            // 16-byte pieces of a key row
  constexpr int PIECES = kArPage * KROW;  // of one page's keys (and of its values)
  constexpr int LD = PIECES / 64;         // per lane
  constexpr int NVB = 64 * QT;            // query vectors per block
  __shared__ __attribute__((aligned(16))) ar_u32x4 sk[2][kArTok * KROW];
  __shared__ __attribute__((aligned(16))) ar_u32x4 sv[2][kArTok * KROW];

  const int g = blockIdx.x % a.nkv, bt_id = blockIdx.x / a.nkv;
  const int b = bt_id % a.B, tile = n_tiles - 1 - (bt_id / a.B + (int)blockIdx.y * tiles_x);
  if (tile < 0) return;
  const int sp = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row = lane & 15, grp = lane >> 4;
  int r_beg = a.cu[b], r_end = a.cu[b + 1];
  const int rows_total = a.rows.count ? min(*a.rows.count, a.rows.max_rows) : a.rows.max_rows;
  r_end = min(r_end, rows_total);
  if (r_beg >= r_end) return;
  const int G = a.nq / a.nkv;
  const int nvec = (r_end - r_beg) * G;
  const int v0 = tile * NVB;              // first query vector of the block
  if (v0 >= nvec) return;
  const int slot = a.slot0 >= 0 ? a.slot0 : a.bslot[b];
  const int nblocks = a.slot_nblocks[slot];
  const int32_t* bt = a.block_table + (long)slot * a.max_blocks;
  // positions the tile's last row sees (rows of a sequence ascend), within this split and
  // the slot's pages
  const int last = a.rows.pos[r_beg + (min(v0 + NVB, nvec) - 1) / G];
  const int p_lo = sp * a.split_len;
  if (p_lo > last) return;                // no row of the tile reads this split
  const int p_hi = min(min(last + 1, p_lo + a.split_len), nblocks * kArPage);
  const int steps = p_hi > p_lo ? (p_hi - p_lo + kArTok - 1) / kArTok : 0;
  const bf16_t* kvb = reinterpret_cast<const bf16_t*>(a.kv);
  const long blk_elems = kv_block_elems(a.n_layers, a.nkv, kArPage, HD);
  const long k_off = (((long)a.layer * 2 + 0) * a.nkv + g) * kArPage * HD;
  const long v_off = (((long)a.layer * 2 + 1) * a.nkv + g) * kArPage * HD;

  // ---- this wavefront's queries: vector j is row r_beg + j / G, head g G + j % G ---------
  ar_bf16x8 qh[QT][KC], ql[QT][KC];
  int qpos[QT];
  int q_min = 0x7fffffff, q_max = -1;
  const int w0 = v0 + wave * 16 * QT;
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    // (vectors past the end repeat the last one and are not written)
    const int j = min(w0 + 16 * q + row, nvec - 1);
    const int r = r_beg + j / G, h = g * G + j % G;
    qpos[q] = a.rows.pos[r];
    q_min = min(q_min, qpos[q]);
    q_max = max(q_max, qpos[q]);
    const float* qp = a.q_prep + ((long)r * a.nq + h) * HD + 8 * grp;
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const float4 x = *reinterpret_cast<const float4*>(qp + 32 * c);
      const float4 y = *reinterpret_cast<const float4*>(qp + 32 * c + 4);
      uint32_t hi[4], lo[4];
      split_bf16x2(x.x, x.y, hi[0], lo[0]);
      split_bf16x2(x.z, x.w, hi[1], lo[1]);
      split_bf16x2(y.x, y.y, hi[2], lo[2]);
      split_bf16x2(y.z, y.w, hi[3], lo[3]);
      qh[q][c] = __builtin_bit_cast(ar_bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
      ql[q][c] = __builtin_bit_cast(ar_bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
    }
  }
  q_min = wave_min_i(q_min);
  q_max = wave_max_i(q_max);

  float m[QT], lsum[QT];
  ar_f32x4 acc[QT][NT];
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    m[q] = -INFINITY;
    lsum[q] = 0.f;
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[q][n] = ar_f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // ---- staging: wavefront w brings page w of a step -----------------------------------------
  ar_u32x4 kr[LD], vr[LD];
  // the wavefront's page-table entries of 64 steps, one per lane (a scalar load per step
  // would stand between the step's start and its page requests); pages past the positions
  // read the last one again and are cleared in put
  const int pg_last = max((p_hi - 1) / kArPage, 0);
  int ent = 0;
  auto request = [&](int t) {
    if ((t & 63) == 0) ent = bt[min(p_lo / kArPage + 4 * (t + lane) + wave, pg_last)];
    const long base = (long)__builtin_amdgcn_readlane(ent, t & 63) * blk_elems;
    const ar_u32x4* kp = reinterpret_cast<const ar_u32x4*>(kvb + base + k_off);
    const ar_u32x4* vp = reinterpret_cast<const ar_u32x4*>(kvb + base + v_off);
#pragma unroll
    for (int i = 0; i < LD; ++i) { kr[i] = kp[i * 64 + lane]; vr[i] = vp[i * 64 + lane]; }
  };
  auto put = [&](int t, int buf) {
    const int t0 = p_lo + t * kArTok + wave * kArPage;   // the page's first position
    if (t0 + kArPage > p_hi) {
      // values past the sequence end are cleared, so that unwritten cache memory cannot
      // reach the sums (0 x NaN); their scores are masked
#pragma unroll
      for (int i = 0; i < LD; ++i) {
        const int p0 = t0 + 8 * (lane & 1);               // piece: 8 tokens of one dimension
#pragma unroll
        for (int e = 0; e < 4; ++e)
          vr[i][e] &= p0 + 2 * e >= p_hi ? 0u : (p0 + 2 * e + 1 >= p_hi ? 0xffffu : 0xffffffffu);
      }
    }
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      const int x = i * 64 + lane;
      const int tok = x / KROW, c = x % KROW;
      sk[buf][(wave * kArPage + tok) * KROW + (c ^ (tok & (KROW - 1)))] = kr[i];
      // values: tokens 4 g .. 4 g + 3 of a dimension beside those of the pair's other page,
      // the order in which the second product takes them
      uint2* v2 = reinterpret_cast<uint2*>(sv[buf]) + (((wave >> 1) * HD + (x >> 1)) * 4 + 2 * (x & 1)) * 2 + (wave & 1);
      v2[0] = make_uint2(vr[i][0], vr[i][1]);
      v2[2] = make_uint2(vr[i][2], vr[i][3]);
    }
  };

  auto compute = [&](int t, int buf) {
    const int t0 = p_lo + t * kArTok;
    if (t0 > q_max) return;                               // past every query of the wavefront
    ar_f32x4 sc[QT][4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
      for (int q = 0; q < QT; ++q) sc[q][p] = ar_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        const ar_bf16x8 ka = __builtin_bit_cast(
            ar_bf16x8, sk[buf][(p * kArPage + row) * KROW + ((4 * c + grp) ^ (row & (KROW - 1)))]);
#pragma unroll
        for (int q = 0; q < QT; ++q) {
          sc[q][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qh[q][c], sc[q][p], 0, 0, 0);
          sc[q][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, ql[q][c], sc[q][p], 0, 0, 0);
        }
      }
    }
    // causal and sequence-end mask (lane: tokens 4 grp + e of page p, query `row`)
    if (t0 + kArTok - 1 > q_min || t0 + kArTok > p_hi) {
#pragma unroll
      for (int q = 0; q < QT; ++q)
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int pos = t0 + p * kArPage + 4 * grp + e;
            if (pos > qpos[q] || pos >= p_hi) sc[q][p][e] = -INFINITY;
          }
    }
    ar_bf16x8 ph[QT][2], pl[QT][2];
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      float bm = -INFINITY;
#pragma unroll
      for (int p = 0; p < 4; ++p)
        bm = fmaxf(bm, fmaxf(fmaxf(sc[q][p][0], sc[q][p][1]), fmaxf(sc[q][p][2], sc[q][p][3])));
      bm = fmaxf(bm, xor_lane_c(bm, 16));
      bm = fmaxf(bm, xor_lane_c(bm, 32));
      const float mn = fmaxf(m[q], bm);
      // (finite, so that a masked score or an empty maximum gives exp(-inf) = 0)
      const float ms = fmaxf(mn, -3.0e38f);
      if (__any(mn > m[q])) {
        const float f = __expf(m[q] - ms);
        lsum[q] *= f;
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[q][n] *= f;
      }
      m[q] = mn;
      float s = 0.f;
      uint32_t hi[8], lo[8];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        float pe[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) pe[e] = __expf(sc[q][p][e] - ms);
        s += (pe[0] + pe[1]) + (pe[2] + pe[3]);
        split_bf16x2(pe[0], pe[1], hi[2 * p], lo[2 * p]);
        split_bf16x2(pe[2], pe[3], hi[2 * p + 1], lo[2 * p + 1]);
      }
      lsum[q] += s;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        ph[q][i] = __builtin_bit_cast(ar_bf16x8, make_uint4(hi[4 * i], hi[4 * i + 1], hi[4 * i + 2], hi[4 * i + 3]));
        pl[q][i] = __builtin_bit_cast(ar_bf16x8, make_uint4(lo[4 * i], lo[4 * i + 1], lo[4 * i + 2], lo[4 * i + 3]));
      }
    }
    // O^T[dim][query] += V^T P^T over page pairs
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const ar_bf16x8 va = __builtin_bit_cast(ar_bf16x8, sv[buf][(i * HD + 16 * n + row) * 4 + grp]);
#pragma unroll
        for (int q = 0; q < QT; ++q) {
          acc[q][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, ph[q][i], acc[q][n], 0, 0, 0);
          acc[q][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pl[q][i], acc[q][n], 0, 0, 0);
        }
      }
    }
  };

  if (steps > 0) {
    request(0);
    put(0, 0);
    __syncthreads();
    for (int t = 0; t < steps; ++t) {
      if (t + 1 < steps) request(t + 1);
      compute(t, t & 1);
      if (t + 1 < steps) put(t + 1, (t + 1) & 1);
      __syncthreads();
    }
  }

  // ---- lane holds O^T[16 n + 4 grp + e][query row] -------------------------------------------
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    float l = lsum[q];
    l += xor_lane_c(l, 16);
    l += xor_lane_c(l, 32);
    const int j = w0 + 16 * q + row;
    if (j >= nvec) continue;
    const int r = r_beg + j / G, h = g * G + j % G;
    if (a.direct) {
      const float inv = l > 0.f ? 1.0f / l : 0.f;
      const long o = (long)r * a.nq * HD + h * HD + 4 * grp;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        uint32_t h2[2], l2[2];
        split_bf16x2(acc[q][n][0] * inv, acc[q][n][1] * inv, h2[0], l2[0]);
        split_bf16x2(acc[q][n][2] * inv, acc[q][n][3] * inv, h2[1], l2[1]);
        *reinterpret_cast<uint2*>(a.o_hi + o + 16 * n) = make_uint2(h2[0], h2[1]);
        *reinterpret_cast<uint2*>(a.o_lo + o + 16 * n) = make_uint2(l2[0], l2[1]);
      }
    } else {
      float* pp = a.part + (((long)r * a.nq + h) * a.n_split + sp) * (HD + 2);
      if (grp == 0) *reinterpret_cast<float2*>(pp) = make_float2(m[q], l);
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        float2* o = reinterpret_cast<float2*>(pp + 2 + 16 * n + 4 * grp);
        o[0] = make_float2(acc[q][n][0], acc[q][n][1]);
        o[1] = make_float2(acc[q][n][2], acc[q][n][3]);
      }
    }
  }
}

// Merge of a few splits for many rows: a wavefront per (row, head), lane l holding
// HD / 64 dimensions of every split, the splits' loads four at a time.  (The general
// merge kernel gives each (row, head) a block with slots for 64 splits: 81 us for two
// splits of 1999 x 16 rows.)  Weights and sums are formed as where the O projection merges
// (skinny.hip), in split order: a row's bits do not depend on which of the two merges it, nor
// on how many splits past its own a pass is planned for.
template <int HD>
__global__ void __launch_bounds__(256) k_attn_join(AttnArgs a) {
  constexpr int DPL = HD / 64;
  const int r = blockIdx.x, h = blockIdx.y * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int rows = a.rows.count ? min(*a.rows.count, a.rows.max_rows) : a.rows.max_rows;
  if (r >= rows || h >= a.nq) return;
  const float* pp = a.part + ((long)r * a.nq + h) * a.n_split * (HD + 2);
  // splits that hold a position this row sees (later ones were not written)
  const int ns = min(a.n_split, a.rows.pos[r] / a.split_len + 1);
  const long rec = (long)min(lane, ns - 1) * (HD + 2);
  const float2 ml = *reinterpret_cast<const float2*>(pp + rec);
  const float m = lane < ns ? ml.x : -INFINITY;
  const float M = wave_max(m);
  const float f = m > -INFINITY ? __expf(m - M) : 0.f;
  float L = 0.f;
  for (int sp = 0; sp < ns; ++sp) {
    const float fs = lane_f(f, sp), ls = lane_f(ml.y, sp);
    L = fs > 0.f ? L + ls * fs : L;
  }
  const float w = L > 0.f ? f / L : 0.f;
  float y[DPL];
#pragma unroll
  for (int e = 0; e < DPL; ++e) y[e] = 0.f;
  for (int s0 = 0; s0 < ns; s0 += 4) {
    float v[4][DPL];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < DPL; ++e) v[i][e] = pp[(long)min(s0 + i, ns - 1) * (HD + 2) + 2 + lane * DPL + e];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float ws = s0 + i < ns ? lane_f(w, min(s0 + i, 63)) : 0.f;
      const bool in = ws != 0.f;
#pragma unroll
      for (int e = 0; e < DPL; ++e) y[e] = in ? y[e] + ws * v[i][e] : y[e];
    }
  }
  const long o = (long)r * a.nq * HD + h * HD + lane * DPL;
#pragma unroll
  for (int e = 0; e < DPL; ++e) {
    const bf16_t yh = f32_to_bf16(y[e]);
    a.o_hi[o + e] = yh;
    a.o_lo[o + e] = f32_to_bf16(y[e] - bf16_to_f32(yh));
  }
}

void launch_attn_join(const AttnArgs& a, hipStream_t st) {
  const dim3 grid(a.rows.max_rows, (a.nq + 3) / 4);
  if (a.hd == 128) hipLaunchKernelGGL(k_attn_join<128>, grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL(k_attn_join<64>, grid, dim3(256), 0, st, a);
}

// Two query tiles per wavefront once a sequence fills more than one block of them.
static int attn_rows_qt(int vectors) { return vectors > 64 ? 2 : 1; }

bool attn_rows_supported(int kvdtype, int rows_per_seq, int group) {
  return kvdtype == 1 && rows_per_seq * group > 16;
}

int attn_rows_tiles(int rows, int rows_per_seq, int group) {
  const int nvb = 64 * attn_rows_qt(rows_per_seq * group);
  return (rows * group + nvb - 1) / nvb;
}

void launch_attention_rows(const AttnArgs& a, hipStream_t st) {
  const int G = a.nq / a.nkv;
  const int qt = attn_rows_qt(a.rows_per_seq * G);
  const int n_tiles = attn_rows_tiles(a.rows_per_seq, a.rows_per_seq, G);
  // Grid y and z end at 65536, which (row tile, sequence) pairs can pass (257 tiles of 256
  // sequences), and x at 2^32 threads: x takes up to 2^20 blocks, then y further tiles.
  const int tiles_x = std::min(n_tiles, std::max(1, (1 << 20) / (a.nkv * a.B)));
  const dim3 grid(a.nkv * a.B * tiles_x, (n_tiles + tiles_x - 1) / tiles_x, a.n_split);
  if (a.hd == 128) {
    if (qt == 2) hipLaunchKernelGGL((k_attn_rows<128, 2>), grid, dim3(256), 0, st, a, n_tiles, tiles_x);
    else hipLaunchKernelGGL((k_attn_rows<128, 1>), grid, dim3(256), 0, st, a, n_tiles, tiles_x);
  } else {
    if (qt == 2) hipLaunchKernelGGL((k_attn_rows<64, 2>), grid, dim3(256), 0, st, a, n_tiles, tiles_x);
    else hipLaunchKernelGGL((k_attn_rows<64, 1>), grid, dim3(256), 0, st, a, n_tiles, tiles_x);
  }
}

}  // namespace osp
