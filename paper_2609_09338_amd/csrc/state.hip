// Device-side sequence state: row layout of an ingest, KV append, lengths.
//
// The committed length of every slot and the tokens committed by the last
// verification live on the device, so a steady-state draft -> verify -> draft
// loop needs no host synchronisation: k_setup turns them into the packed row
// list (sequence, absolute position, token, tap row) of the next ingest.
#include "common.h"
#include "internal.h"

#include <algorithm>

namespace osp {

// Threads b < kMaxBatch own sequence b; all of them then share the rows.  A prompt has
// thousands of rows, so they are dealt to the whole block, kSetupRows per thread with
// their loads together (a sequence's own thread filling its rows one dependent load at a
// time took 359 us for one 1999-token prompt and 587 us for 8200 rows of four; now 7.2 and
// 10.7 us).  Passes of few rows launch only the threads that own sequences.
constexpr int kSetupThreads = 1024;
constexpr int kSetupRows = 4;
static_assert(kSetupThreads >= kMaxBatch, "one thread per sequence");

__global__ void __launch_bounds__(kSetupThreads) k_setup(SetupArgs a) {
  const int n_waves = blockDim.x / 64;
  __shared__ int s_tot[kSetupThreads / 64];
  __shared__ int s_cu[kMaxBatch + 1], s_cun[kMaxBatch], s_n[kMaxBatch], s_len[kMaxBatch], s_slot[kMaxBatch];
  const int b = threadIdx.x;
  const int lane = b & 63, wave = b >> 6;
  const bool act = b < a.B;
  int slot = 0, len = 0, n = 0;
  if (act) {
    slot = a.slots[b];
    len = a.slot_len[slot];
    n = a.explicit_rows ? a.n_new[b] : a.pend_n[slot];
    if (n < 1 || n > a.max_new) {
      atomicOr(a.err, 1u << 0);
      n = min(max(n, 1), a.max_new);
    }
  }
  // block drafting: the block's mask rows follow the sequence's new rows
  const int m = act ? a.extra : 0;
  // exclusive prefixes over the batch (integer scans: wave scan + wave totals) of the
  // rows (n + m) and of the new rows alone (packed tap rows)
  const int inc = wave_incl_scan<int>(n + m), incn = wave_incl_scan<int>(n);
  __shared__ int s_totn[kSetupThreads / 64];
  if (lane == 63) { s_tot[wave] = inc; s_totn[wave] = incn; }
  __syncthreads();
  int before = 0, total = 0, beforen = 0;
  for (int w = 0; w < n_waves; ++w) {
    if (w < wave) { before += s_tot[w]; beforen += s_totn[w]; }
    total += s_tot[w];
  }
  const int cu = before + inc - (n + m);
  const int cun = beforen + incn - n;
  if (act) {
    a.cu[b] = cu;
    a.last_row[b] = cu + n - 1;
    a.committed[b] = len + n;
    a.bslot[b] = slot;
    a.ar_pos[b] = len + n;
    s_cu[b] = cu;
    s_cun[b] = cun;
    s_n[b] = n;
    s_len[b] = len;
    s_slot[b] = slot;
    if (m > 0) {
      for (int k = 0; k <= m; ++k) {
        a.blk_gather[b * (m + 1) + k] = cu + n - 1 + k;
        a.blk_temp[b * (m + 1) + k] = a.temp[b];
      }
    }
    const int cap = a.slot_nblocks[slot] * a.kv_block;
    if (len + n + (a.K > 0 ? a.K - 1 : 0) > cap) atomicOr(a.err, 1u << 2);
    a.slot_len[slot] = len + n;
    a.pend_n[slot] = 0;
  }
  if (b == 0) {
    a.cu[a.B] = total;
    a.n_rows[0] = total;
  }
  // ---- the rows: a sequence's new tokens, then (block drafting) its mask rows with the
  //      anchor's tap row (its conditioning input, broadcast) --------------------------------
  __syncthreads();
  for (int r0 = threadIdx.x; r0 < total; r0 += (int)blockDim.x * kSetupRows) {
    int q[kSetupRows], t[kSetupRows];
#pragma unroll
    for (int i = 0; i < kSetupRows; ++i) {
      // the sequence of row r: the last whose first row is not past it
      const int r = min(r0 + i * (int)blockDim.x, total - 1);
      int lo = 0, hi = a.B;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (s_cu[mid] <= r) lo = mid; else hi = mid;
      }
      q[i] = lo;
      const int j = min(r - s_cu[lo], s_n[lo] - 1);
      t[i] = a.explicit_rows ? a.new_tokens[s_cun[lo] + j] : a.pend_tok[(long)s_slot[lo] * a.pend_ld + j];
    }
#pragma unroll
    for (int i = 0; i < kSetupRows; ++i) {
      const int r = r0 + i * (int)blockDim.x;
      if (r >= total) continue;
      const int j = r - s_cu[q[i]], jn = min(j, s_n[q[i]] - 1);
      int tok = t[i];
      if (j >= s_n[q[i]]) {
        tok = a.mask;
      } else if (tok < 0 || tok >= a.V_T) {
        atomicOr(a.err, 1u << 1);
        tok = min(max(tok, 0), a.V_T - 1);
      }
      a.ing_seq[r] = q[i];
      a.ing_pos[r] = s_len[q[i]] + j;
      a.ing_tok[r] = tok;
      a.ing_tap[r] = a.taps_stride > 0 ? q[i] * a.taps_stride + jn : s_cun[q[i]] + jn;
    }
  }
  // ---- attention work list: every split but the last of each sequence covers
  //      split_len positions; those come first (sequence-major), then the last
  //      splits by decreasing length, so the longest blocks start first.  An item
  //      carries the sequence's slot, so that a block finds its page table without
  //      one more dependent load ---------------------------------------------------------
  if (a.attn_items) {
    __shared__ int s_last[kMaxBatch];
    const int nmax = act ? len + n + (a.K > 0 ? a.K - 1 : 0) : 0;
    const int ns = act ? (nmax + a.split_len - 1) / a.split_len : 0;
    const int nfull = ns > 0 ? ns - 1 : 0;
    const int last = act ? nmax - nfull * a.split_len : -1;
    if (b < kMaxBatch) s_last[b] = last;
    const int finc = wave_incl_scan<int>(nfull);
    __syncthreads();
    if (lane == 63) s_tot[wave] = finc;
    __syncthreads();
    int fbefore = 0, ftotal = 0;
    for (int w = 0; w < n_waves; ++w) {
      if (w < wave) fbefore += s_tot[w];
      ftotal += s_tot[w];
    }
    if (act) {
      const int f0 = fbefore + finc - nfull;
      for (int sp = 0; sp < nfull; ++sp) a.attn_items[f0 + sp] = b | (slot << 8) | (sp << 16);
      int rank = 0;
      for (int o = 0; o < a.B; ++o) rank += (s_last[o] > last || (s_last[o] == last && o < b)) ? 1 : 0;
      a.attn_items[ftotal + rank] = b | (slot << 8) | (nfull << 16);
    }
    if (b == 0) a.attn_n_items[0] = ftotal + a.B;
  }
}

void launch_setup(const SetupArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_setup, dim3(1), dim3(a.rows > 4 * kMaxBatch ? kSetupThreads : kMaxBatch), 0, st, a);
}

// Append n positions of precomputed (post-RoPE) keys and values for every layer.
// k, v: [n_layers][n][nkv][hd].  Positions start at the slot's current length.
template <typename T>
__global__ void k_kv_append(T* kv, const T* k, const T* v, int n_layers, int n, int nkv, int hd,
                            int kv_block, const int32_t* block_table, int slot, int max_blocks,
                            const int32_t* slot_len) {
  const long total = (long)n_layers * n * nkv * hd;
  const long blk_elems = kv_block_elems(n_layers, nkv, kv_block, hd);
  const int len = slot_len[slot];
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < total;
       i += (long)gridDim.x * blockDim.x) {
    long t = i;
    const int e = t % hd; t /= hd;
    const int g = t % nkv; t /= nkv;
    const int p = t % n; t /= n;
    const int l = (int)t;
    const int pos = len + p;
    const int blk = pos / kv_block, within = pos - blk * kv_block;
    if (blk >= max_blocks) continue;
    const long phys = block_table[(long)slot * max_blocks + blk];
    T* base = kv + phys * blk_elems;
    base[(((long)l * 2 + 0) * nkv + g) * kv_block * hd + kv_k_at(within, e, hd)] = k[i];
    base[(((long)l * 2 + 1) * nkv + g) * kv_block * hd + kv_v_at(within, e, kv_block)] = v[i];
  }
}

__global__ void k_add_len(int32_t* slot_len, int slot, int n) { slot_len[slot] += n; }

void launch_kv_append(int kvdtype, void* kv, const void* k, const void* v, int n_layers, int n,
                      int nkv, int hd, int kv_block, const int32_t* block_table, int slot,
                      int max_blocks, const int32_t* slot_len, int32_t* slot_len_out,
                      hipStream_t st) {
  const long total = (long)n_layers * n * nkv * hd;
  const int grid = (int)std::min<long>((total + 255) / 256, 4096);
  if (total > 0) {
    if (kvdtype == 1)
      hipLaunchKernelGGL(k_kv_append<bf16_t>, dim3(grid), dim3(256), 0, st,
                         reinterpret_cast<bf16_t*>(kv), reinterpret_cast<const bf16_t*>(k),
                         reinterpret_cast<const bf16_t*>(v), n_layers, n, nkv, hd, kv_block,
                         block_table, slot, max_blocks, slot_len);
    else
      hipLaunchKernelGGL(k_kv_append<float>, dim3(grid), dim3(256), 0, st,
                         reinterpret_cast<float*>(kv), reinterpret_cast<const float*>(k),
                         reinterpret_cast<const float*>(v), n_layers, n, nkv, hd, kv_block,
                         block_table, slot, max_blocks, slot_len);
  }
  hipLaunchKernelGGL(k_add_len, dim3(1), dim3(1), 0, st, slot_len_out, slot, n);
}

// Shorten a slot to min(length, len) and drop its pending ingest.
__global__ void k_set_len(int32_t* slot_len, int32_t* pend_n, int slot, int len) {
  slot_len[slot] = min(slot_len[slot], len);
  pend_n[slot] = 0;
}

void launch_set_len(int32_t* slot_len, int32_t* pend_n, int slot, int len, hipStream_t st) {
  hipLaunchKernelGGL(k_set_len, dim3(1), dim3(1), 0, st, slot_len, pend_n, slot, len);
}

__global__ void k_fill_i32(int32_t* p, int32_t v, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    p[i] = v;
}

void launch_fill_i32(int32_t* p, int32_t v, long n, hipStream_t st) {
  if (n <= 0) return;
  const int grid = (int)std::min<long>((n + 255) / 256, 1024);
  hipLaunchKernelGGL(k_fill_i32, dim3(grid), dim3(256), 0, st, p, v, n);
}

}  // namespace osp
