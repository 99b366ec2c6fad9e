// Growing a draft tree (top-k > 1; the paper serves chains, top-k 1, Section 4):
// every node of the frontier runs through the drafter, its k most likely rows become
// candidates scored by the cumulative log-probability of their path (temperature 1),
// the k best candidates of a depth form the next frontier, and the n best candidates
// of all depths form the tree.
//
//   k_tree_step  (B)  per sequence: the rows' k best (logit, row) pairs (larger logit
//                     first, lower row on ties) and log-normalisers, both from the LM-head
//                     records at temperature 1, the new candidates, the next frontier and
//                     the next pass's rows: token, position, node slot, ancestors' slots
//                     and conditioning row (the parent's hidden state)
//   k_tree_final (B)  the n best candidates in generation order, parents re-indexed
//
// A wavefront selects a row's k best: the k-th largest of the distinct range maxima in the
// records bounds them from below (at least k values reach it), so only the logits of the
// ranges that reach it are read, and those that reach it themselves, usually hardly more
// than k, are ranked against each other in one step.  Where the likely ids are neighbours
// (one range holds many of them), logits tie, or few ranges hold a mapped row, more than a
// list of them reaches the bound: then the k ranges of largest max are read, and rounds of
// the wavefront's best pick the ranges and their logits.  Bound by the latency of dependent
// steps: records, logits, candidates, d2t and scores, rows, the copy of the conditioning rows.
// (One sequence of 4 rows: 15 us, 21 for a separate pass over every logit and a step that
// merged its blocks; 12 sequences of 8 rows: 21 us, 65 for rounds over 32 records and 32 logits
// of every lane for two rows per wavefront.  Whole calls with likely ids spread / neighbours,
// copies or few mapped rows: one sequence 728 / 753-758 us, 12 sequences 1645 / 1736-1754; one
// wavefront scanning a row's 151936 logits in the latter cases took 1913-3642 and 6821-7030 us.)
// A frontier row's attention over its ancestors' and its own keys/values (the tree
// cache) is one more split of the context attention, added by the split combine.
#include "common.h"
#include "internal.h"

namespace osp {

constexpr int kTkThreads = kMaxTopk * OSP_WAVE;   // a wavefront per frontier row
constexpr int kTkRecLane = kTkMaxRecords / OSP_WAVE;   // LM-head records per lane

OSP_DEV bool tk_better(float v1, int r1, float v2, int r2) { return v1 > v2 || (v1 == v2 && r1 < r2); }

// Wavefront-wide best (value, row) pair.
OSP_DEV void wave_best(float& v, int& r) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const float ov = xor_lane_c(v, m);
    const int orow = xor_lane_ci(r, m);
    if (tk_better(ov, orow, v, r)) { v = ov; r = orow; }
  }
}

// Candidate c is better than candidate e: larger score, lower index on ties.
OSP_DEV bool cand_better(double s1, int i1, double s2, int i2) { return s1 > s2 || (s1 == s2 && i1 < i2); }

constexpr int kTkRanges = 16;     // record ranges a selection by the bound reads
constexpr int kTkList = OSP_WAVE; // logits it ranks

// One round of a wavefront's selection of its best (value, index) pairs: the best over the
// lanes' N values that are not yet taken (bit q of `gone`: value q), marked as taken by the
// lane that holds it.  index(q) is this lane's index of value q, 0x7fffffff for none.
template <int N, typename F>
OSP_DEV void wave_take_best(const float (&v)[N], F index, unsigned& gone, float& wv, int& wr) {
  static_assert(N <= 32, "one bit per value");
  float bv = -INFINITY;
  int br = 0x7fffffff, bq = 0;
#pragma unroll
  for (int q = 0; q < N; ++q)
    if (!((gone >> q) & 1u) && tk_better(v[q], index(q), bv, br)) { bv = v[q]; br = index(q); bq = q; }
  wv = bv;
  wr = br;
  wave_best(wv, wr);
  if (br == wr && wr != 0x7fffffff) gone |= 1u << bq;
}

__global__ void __launch_bounds__(kTkThreads) k_tree_step(TreeArgs a) {
  __shared__ float s_cv[kMaxTopk][kMaxTopk];
  __shared__ int s_cr[kMaxTopk][kMaxTopk];
  __shared__ double s_lse[kMaxTopk];
  __shared__ double s_sc[kMaxTopk * kMaxTopk];
  __shared__ int s_sel[kMaxTopk];
  __shared__ int s_src[kMaxTopk];
  __shared__ int s_prev[kMaxTopk];
  __shared__ int s_ntok[kMaxTopk * kMaxTopk], s_ndep[kMaxTopk * kMaxTopk];
  __shared__ int s_rank[kMaxTopk * kMaxTopk];
  __shared__ int s_rng[kMaxTopk][kTkRanges];
  __shared__ float s_lv[kMaxTopk][kTkList];
  __shared__ int s_li[kMaxTopk][kTkList];
  __shared__ int s_n0;
  const int b = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int K = a.k, p = a.pass;
  const int nfr = p == 0 ? 1 : K;                 // rows of this pass that are sequence b's
  const int row0 = p == 0 ? b : b * K;
  const long cb = (long)b * kMaxCand;
  // this pass's rows' ancestor lists (read before the next pass's replace them)
  __shared__ int s_anc[kMaxTopk][kMaxTreeDepth];
  if (p > 0 && tid < K * kMaxTreeDepth)
    s_anc[tid / kMaxTreeDepth][tid % kMaxTreeDepth] = a.r_anc[(long)b * K * kMaxTreeDepth + tid];
  if (tid < K) s_prev[tid] = p == 0 ? -1 : a.front[b * kMaxTopk + tid];
  if (tid == 0) s_n0 = p == 0 ? 0 : a.n_cand[b];   // (read before anyone writes it below)
  if (tid < K) { s_sel[tid] = tid; s_src[tid] = p == 0 ? 0 : tid; }   // (overwritten below)
  // ---- each row's K best (logit, row) pairs and its log-normaliser M + log S --------------
  if (wave < nfr) {
    const int j = wave, r = row0 + j;
    // LM-head records of the row (temperature 1): max and rescaled sums, every record
    // of the lane requested at once (clamped addresses; lane l: records l, l + 64, ...)
    const float* rec = a.rec + (long)r * a.nblk * 4;
    float2 rs[kTkRecLane];
#pragma unroll
    for (int q = 0; q < kTkRecLane; ++q)
      rs[q] = *reinterpret_cast<const float2*>(rec + (long)min(lane + q * OSP_WAVE, a.nblk - 1) * 4);
    float m = -INFINITY;
#pragma unroll
    for (int q = 0; q < kTkRecLane; ++q)
      if (lane + q * OSP_WAVE < a.nblk) m = fmaxf(m, rs[q].x);
    const float M = wave_max(m);
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kTkRecLane; ++q)
      if (lane + q * OSP_WAVE < a.nblk && rs[q].x > -INFINITY) s += (double)rs[q].y * (double)__expf(rs[q].x - M);
    const double S = wave_sum_d(s);
    // Mk: the K-th largest distinct range max (the ranges of largest max hold K values >= Mk,
    // so the K-th best value is >= Mk)
    float Mk = M;
    for (int t = 1; t < K; ++t) {
      float x = -INFINITY;
#pragma unroll
      for (int q = 0; q < kTkRecLane; ++q) {
        const float v = lane + q * OSP_WAVE < a.nblk ? rs[q].x : -INFINITY;
        x = fmaxf(x, v < Mk ? v : -INFINITY);
      }
      Mk = wave_max(x);
    }
    int n = 0;
#pragma unroll
    for (int q = 0; q < kTkRecLane; ++q) {
      const int c = lane + q * OSP_WAVE;
      const bool in = c < a.nblk && rs[q].x >= Mk;
      const unsigned long long bal = __ballot(in);
      const int at = n + __popcll(bal & ((1ull << lane) - 1ull));
      if (in && at < kTkRanges) s_rng[j][at] = c;
      n += __popcll(bal);
    }
    __builtin_amdgcn_wave_barrier();
    const float* lg = a.logits + (long)r * a.ld_logits;
    int nl = kTkList + 1;
    if (n <= kTkRanges && Mk > -INFINITY) {
      // every listed range's logits requested at once: lane l reads entries l and l + 64
      float lv[2 * kTkRanges];
#pragma unroll
      for (int i = 0; i < kTkRanges; ++i) {
        const int e0 = (i < n ? s_rng[j][i] : 0) * a.blk_rows + lane;
        lv[2 * i] = lg[min(e0, a.V - 1)];                  // clamped, masked below
        lv[2 * i + 1] = lg[min(e0 + OSP_WAVE, a.V - 1)];
      }
      // those that reach Mk into a list
      nl = 0;
#pragma unroll
      for (int i = 0; i < 2 * kTkRanges; ++i) {
        const int at = (i & 1) * OSP_WAVE + lane;            // place in the range
        const int e = (i / 2 < n ? s_rng[j][i / 2] : 0) * a.blk_rows + at;
        const bool in = i / 2 < n && at < a.blk_rows && e < a.V && lv[i] >= Mk;
        const unsigned long long bal = __ballot(in);
        const int to = nl + __popcll(bal & ((1ull << lane) - 1ull));
        if (in && to < kTkList) { s_lv[j][to] = lv[i]; s_li[j][to] = e; }
        nl += __popcll(bal);
      }
      __builtin_amdgcn_wave_barrier();
    }
    if (__builtin_expect(nl >= K && nl <= kTkList, 1)) {
      // lane l holds entry l; its rank is the number of better ones
      const float v = s_lv[j][min(lane, nl - 1)];
      const int e = s_li[j][min(lane, nl - 1)];
      int rank = lane < nl ? 0 : K;
      for (int i = 0; i < nl; ++i) rank += tk_better(s_lv[j][i], s_li[j][i], v, e) ? 1 : 0;
      if (rank < K) { s_cv[j][rank] = v; s_cr[j][rank] = e; }
    } else {
      // The K ranges of largest max, the lower one on ties, hold the K best logits: a logit of
      // another range has K better ones, the maxima of these (equal maxima lie in lower rows).
      float mv[kTkRecLane];
#pragma unroll
      for (int q = 0; q < kTkRecLane; ++q) mv[q] = lane + q * OSP_WAVE < a.nblk ? rs[q].x : -INFINITY;
      const auto range_of = [&](int q) { return lane + q * OSP_WAVE < a.nblk ? lane + q * OSP_WAVE : 0x7fffffff; };
      unsigned gone = 0;
      for (int t = 0; t < K; ++t) {
        float wv;
        int wc;
        wave_take_best(mv, range_of, gone, wv, wc);
        if (lane == 0) s_rng[j][t] = wc;
      }
      __builtin_amdgcn_wave_barrier();
      float lv[2 * kMaxTopk];
      int li[2 * kMaxTopk];
#pragma unroll
      for (int i = 0; i < 2 * kMaxTopk; ++i) {
        const int c = i / 2 < K ? s_rng[j][i / 2] : 0x7fffffff;     // (0x7fffffff: fewer ranges than K)
        const int at = (i & 1) * OSP_WAVE + lane;
        const int e = (c < a.nblk ? c : 0) * a.blk_rows + at;
        lv[i] = lg[min(e, a.V - 1)];
        li[i] = c < a.nblk && at < a.blk_rows && e < a.V ? e : 0x7fffffff;
      }
#pragma unroll
      for (int i = 0; i < 2 * kMaxTopk; ++i) lv[i] = li[i] < a.V ? lv[i] : -INFINITY;
      gone = 0;
      for (int t = 0; t < K; ++t) {
        float wv;
        int wr;
        wave_take_best(lv, [&](int q) { return li[q]; }, gone, wv, wr);
        if (lane == 0) { s_cv[j][t] = wv; s_cr[j][t] = wr; }
      }
    }
    if (lane == 0) s_lse[j] = (double)M + log(S);
  }
  __syncthreads();
  // ---- the new candidates (row j, rank t) in generation order -----------------------------
  const int n0 = s_n0;
  const int nnew = nfr * K;
  if (tid < nnew) {
    const int j = tid / K, t = tid % K;
    const int par = s_prev[j];
    const int c = n0 + tid;
    const int rr = s_cr[j][t];
    const bool ok = rr >= 0 && rr < a.V;
    const double sc = (par >= 0 ? a.c_score[cb + par] : 0.0) + ((double)s_cv[j][t] - s_lse[j]);
    const int tok = ok ? a.d2t[rr] : -1;
    const int dep = (par >= 0 ? a.c_depth[cb + par] : 0) + 1;
    a.c_tok[cb + c] = tok;
    a.c_par[cb + c] = par;
    a.c_score[cb + c] = sc;
    a.c_depth[cb + c] = dep;
    s_sc[tid] = sc;
    s_ntok[tid] = tok;                              // (read back below from LDS: another
    s_ndep[tid] = dep;                              // wavefront's global writes may not be)
  }
  if (tid == 0) a.n_cand[b] = n0 + nnew;
  __syncthreads();
  if (p + 1 >= a.depth) {                         // the last pass: no next frontier
    if (tid < nnew) a.c_slot[cb + n0 + tid] = -1;
    return;
  }
  // ---- the next frontier: the K best new candidates, then in generation order -------------
  if (tid < nnew) {
    int rank = 0;
    for (int e = 0; e < nnew; ++e) rank += cand_better(s_sc[e], e, s_sc[tid], tid) ? 1 : 0;
    s_rank[tid] = rank;
  }
  __syncthreads();
  if (tid < nnew) {
    int pos = K;
    if (s_rank[tid] < K) {
      pos = 0;            // place among the selected, by generation order
      for (int e = 0; e < tid; ++e) pos += s_rank[e] < K ? 1 : 0;
    }
    if (pos < K) {        // (scores that are not numbers could put more than K below rank K)
      s_sel[pos] = tid;                             // (new candidate n0 + tid)
      s_src[pos] = tid / K;                         // the frontier row of its parent
      // (each new candidate's slot is written once, by its own thread)
      a.c_slot[cb + n0 + tid] = b * kMaxTreeProc + p * K + pos;
    } else {
      a.c_slot[cb + n0 + tid] = -1;
    }
  }
  __syncthreads();
  // ---- the next pass's rows ---------------------------------------------------------------
  if (tid < K) {
    const int j = tid;
    const int e0 = s_sel[j];                        // index among the new candidates
    const int c = n0 + e0;
    const int slot = b * kMaxTreeProc + p * K + j;  // run through the drafter in pass p + 1
    a.front[b * kMaxTopk + j] = c;
    const int r = b * K + j;
    const int L = a.committed[b];
    a.r_tok[r] = max(s_ntok[e0], 0);
    a.r_pos[r] = L + s_ndep[e0] - 1;
    a.r_attpos[r] = L - 1;
    a.r_node[r] = slot;
    if (j == 0) {                                   // the next pass's rows of sequence b
      a.r_cu[b] = b * K;
      if (b == a.B - 1) a.r_cu[a.B] = a.B * K;
    }
    // ancestors' slots, the root's child first, then the node itself: the parent's list
    // (a row of this pass; root children: none) followed by the node's slot
    const int pr = s_src[j];
    int cnt = 0;
#pragma unroll
    for (int i = 0; i < kMaxTreeDepth; ++i)
      if (p > 0 && cnt == i && s_anc[pr][i] >= 0) cnt = i + 1;
#pragma unroll
    for (int i = 0; i < kMaxTreeDepth; ++i)
      a.r_anc[r * kMaxTreeDepth + i] = i < cnt ? s_anc[pr][i] : (i == cnt ? slot : -1);
  }
  // ---- conditioning rows: the parent's hidden state (root: the last ingest row); the
  //      buffers do not overlap, so the loads of several iterations go out together -------
  const int d4 = a.d / 4, nv = K * d4;
  const float4* __restrict__ x4 = reinterpret_cast<const float4*>(a.x);
  float4* __restrict__ s4 = reinterpret_cast<float4*>(a.r_s) + (long)b * K * d4;
#pragma unroll 4
  for (int i = tid; i < nv; i += kTkThreads) {
    const int j = i / d4;
    const int src = p == 0 ? (a.last_row ? a.last_row[b] : b) : b * K + s_src[j];
    s4[i] = x4[(long)src * d4 + (i - j * d4)];
  }
}

// A thread per candidate; the kept candidates' places come from the wavefronts' ballots.
__global__ void __launch_bounds__(kMaxCand) k_tree_final(TreeArgs a) {
  constexpr int kWaves = kMaxCand / OSP_WAVE;
  __shared__ double s_sc[kMaxCand];
  __shared__ int s_keep[kMaxCand];
  __shared__ int s_pos[kMaxCand];
  __shared__ unsigned long long s_bal[kWaves];
  const int b = blockIdx.x, c = threadIdx.x, lane = c & 63, wave = c >> 6;
  const long cb = (long)b * kMaxCand;
  const int n = min(a.n_cand[b], kMaxCand);
  const int N = min(a.n_nodes, n);
  const double mine = c < n ? a.c_score[cb + c] : 0.0;
  s_sc[c] = mine;
  __syncthreads();
  int rank = 0;
#pragma unroll 8
  for (int e = 0; e < n; ++e) rank += cand_better(s_sc[e], e, mine, c) ? 1 : 0;
  const bool keep = c < n && rank < N;
  const unsigned long long bal = __ballot(keep);
  if (lane == 0) s_bal[wave] = bal;
  s_keep[c] = keep ? 1 : 0;
  __syncthreads();
  int pos = __popcll(bal & ((1ull << lane) - 1ull));
  for (int w = 0; w < wave; ++w) pos += __popcll(s_bal[w]);
  s_pos[c] = pos;
  __syncthreads();
  if (keep && pos < a.n_nodes) {
    const int i = pos;
    const int par = a.c_par[cb + c];
    a.out_tok[(long)b * a.n_nodes + i] = a.c_tok[cb + c];
    // (the parent scores at least as high and comes earlier: it is kept too)
    a.out_par[(long)b * a.n_nodes + i] = par >= 0 ? (s_keep[par] ? s_pos[par] : -2) : -1;
    if (a.out_score) a.out_score[(long)b * a.n_nodes + i] = s_sc[c];
  }
  for (int i = N + c; i < a.n_nodes; i += kMaxCand) {
    a.out_tok[(long)b * a.n_nodes + i] = -1;
    a.out_par[(long)b * a.n_nodes + i] = -2;
    if (a.out_score) a.out_score[(long)b * a.n_nodes + i] = -INFINITY;
  }
}

void launch_tree_step(const TreeArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_tree_step, dim3(a.B), dim3(kTkThreads), 0, st, a);
}

void launch_tree_final(const TreeArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_tree_final, dim3(a.B), dim3(kMaxCand), 0, st, a);
}

}  // namespace osp
