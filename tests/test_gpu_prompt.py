"""Prompts and further turns on the GPU against the oracle: passes of many new rows per
sequence (the tiled products, attention by blocks of query vectors, the row setup), at
the sizes where their tiles and context splits begin and end."""
import numpy as np
import pytest
import torch

import synth
from oracle import harness as OH

from . import parity
from .test_gpu_tree import _path_keys

pytestmark = pytest.mark.gpu

# name -> body, head dim and group; rows per sequence over each cached context.  A block
# holds 64 or 128 query vectors (rows x group), a step 64 positions, a product tile 128 rows.
CASES = {
    "one_row": ("p_single64", [(5, 1)]),       # the vector body of bf16 weights
    "group2_hd64": ("p_qwen_small", [(0, 9), (0, 33), (47, 64)]),
    "group2_hd64_ragged": ("p_qwen_small", [(0, 128), (129, 1), (16, 200)]),
    "group4_hd64_one": ("p_single64", [(300, 37)]),
    "group2_hd128": ("p_single128", [(0, 129)]),
    "group2_hd128_turn": ("p_single128", [(1000, 65)]),
    "group4_hd128": ("p_inject", [(0, 70), (511, 17)]),
    # products by blocks of 256 rows (where they fill the chip's rounds as well as 128 rows
    # do): taps and down projection, gate/up with K splits, gate/up with SwiGLU in the block
    "wide_tile_store": ("p_ffn8192_wide_taps", [(0, 700), (0, 700), (5, 649)]),
    "wide_tile_splits": ("p_ffn4096", [(0, 300), (9, 213)]),
    "wide_tile_swiglu": ("p_ffn8192", [(0, 300), (9, 213)]),
    "many": ("p_qwen_small", [(b, 4 + b % 3) for b in range(18)]),
    # more than 64 sequences: nothing to narrow (a row each), too little, and kept rows that
    # take more than one streaming pass
    "one_each_b70": ("p_qwen_small", [(b % 5, 1) for b in range(70)]),
    "two_each_b66": ("p_qwen_small", [(b % 5, 2) for b in range(66)]),
    "four_each_b66": ("p_qwen_small", [(b % 5, 4) for b in range(66)]),
    "odd_taps": ("p_odd_taps", [(5, 100), (0, 60)]),
    "wide_taps": ("p_wide_taps", [(0, 65), (3, 2), (64, 63)]),
    # three and five query heads per kv head; widths that are no multiple of 256
    "group3": ("p_group3", [(0, 70), (130, 45)]),
    "group5_d320": ("p_group5_d320", [(0, 90), (31, 77)]),
    "group5_d320_r80": ("p_group5_d320", [(3, 80)]),
    "group5_d320_b70": ("p_group5_d320", [(b % 3, 1) for b in range(70)]),
    "f32": ("p_tiny_f32", [(0, 65)]),
    "f32_turn": ("p_tiny_f32", [(70, 3)]),
    # fp32 products go by groups of eight rows
    "f32_group": ("p_tiny_f32", [(0, 8)]),
    "f32_two_groups": ("p_f32_two_layers", [(3, 1), (0, 8)]),
    "f32_groups": ("p_f32_two_layers", [(0, 100), (20, 33)]),
}


@pytest.mark.parametrize("K", [0, 3])
@pytest.mark.parametrize("name", list(CASES))
def test_prompt_matches_oracle(name, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_09338_amd import _lib as L
    from paper_2609_09338_amd import workload as WL
    from paper_2609_09338_amd.binding import Drafter, make_config
    body, seqs = CASES[name]
    # (taps of 3 x 200 columns: not a whole number of 32-column steps)
    if body == "p_odd_taps":
        w = synth.get("p_qwen_small").with_(target_hidden=200)
    elif body == "p_group3":
        w = synth.get("p_qwen_small").with_(n_q_heads=6)
    elif body == "p_group5_d320":
        w = synth.get("p_single64").with_(d_model=320, n_q_heads=5, n_kv_heads=1, d_ffn=448)
    elif body == "p_f32_two_layers":
        w = synth.get("p_tiny_f32").with_(n_layers=2)
    elif body.startswith("p_ffn"):
        w = synth.get("p_wide_taps" if "taps" in body else "p_qwen_small").with_(d_ffn=int(body[5:9]))
    else:
        w = synth.get(body)
    w = w.with_(name="prompt_" + name, batch=len(seqs), K=max(K, 1), temps=(0.0,), draft_temps=())
    weights, d2t = synth.make_weights(w), synth.make_d2t(w)
    dr_o = OH.build_drafter(w, weights, d2t)
    ctx, rows = [c for c, _ in seqs], [n for _, n in seqs]
    blocks = synth.block_ids(w, [synth.blocks_needed(w, c + n + K + 1) for c, n in seqs])
    cfg = make_config(n_layers=w.n_layers, d_model=w.d_model, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads,
                      head_dim=w.head_dim, d_ffn=w.d_ffn, vocab_draft=w.vocab_draft, vocab_target=w.vocab_target,
                      target_hidden=w.target_hidden, n_taps=w.n_taps,
                      dtype=L.OSPREY_BF16 if w.dtype == "bf16" else L.OSPREY_F32, qk_norm=w.qk_norm,
                      rms_eps=w.rms_eps, rope_theta=w.rope_theta, max_batch=w.batch, max_k=3,
                      max_seq_len=max(c + n for c, n in seqs) + K + 1, kv_num_blocks=sum(map(len, blocks)),
                      max_new_rows=max(sum(rows), 1))
    dev = "cuda:0"
    dr = Drafter(cfg, {k: WL.to_dev(v, w, dev) for k, v in weights.items()}, torch.from_numpy(d2t).to(dev))
    dr.kv.fill_(0xFF)          # unwritten cache memory is NaN: nothing may read it
    toks, taps, ref, caches = [], [], [], []
    for b, (c, n) in enumerate(seqs):
        dr.seq_reset(b, blocks[b])
        seq = OH.Sequence(w, c + n + K + 1)
        if c:
            k, v = synth.context_kv(w, b, c)
            dr.kv_append(b, WL.to_dev(k, w, dev), WL.to_dev(v, w, dev))
            seq.k[:, :c], seq.v[:, :c], seq.length = k, v, c
        t, tp = synth.prompt_tokens(w, b, n), synth.taps(w, 0, b, n)
        toks.append(t)
        taps.append(tp)
        ref.append(dr_o.draft(seq, t, tp, K, 0.0, np.zeros(max(K, 1))))
        caches.append(seq)
    logits = torch.empty((w.batch, max(K, 1), w.vocab_draft), device=dev)
    drafts = torch.empty((w.batch, max(K, 1)), dtype=torch.int32, device=dev)
    print(f"[prompt] {name} K {K}", flush=True)
    dr.draft_step(list(range(w.batch)), K, WL.to_dev(np.concatenate(taps), w, dev), torch.zeros(w.batch, device=dev),
                  n_new=rows, new_tokens=torch.from_numpy(np.concatenate(toks).astype(np.int32)).to(dev),
                  draft_tokens=drafts if K else None, draft_logits=logits if K else None)
    torch.cuda.synchronize()
    assert dr.device_errors() == 0
    kv = dr.kv.view(torch.bfloat16 if w.dtype == "bf16" else torch.float32).float().cpu().numpy()
    kv = kv.reshape(cfg.kv_num_blocks, w.n_layers, 2, w.n_kv_heads, 16 * w.head_dim)
    # stored values: half a bf16 ulp (2^-9 of the value) plus the 2e-2 that the parity tests
    # allow a logit, at the size of a key or value; fp32 as its logits, 1e-4
    rel, tol = (2.0 ** -8, 2e-2) if w.dtype == "bf16" else (0.0, 1e-4)
    for b, (c, n) in enumerate(seqs):
        assert dr.seq_length(b) == c + n
        for j, cache in enumerate((caches[b].k, caches[b].v)):
            pages = kv[blocks[b], :, j].reshape(len(blocks[b]), w.n_layers, w.n_kv_heads, *((16, w.head_dim) if j == 0 else (w.head_dim, 16)))
            got = pages if j == 0 else pages.swapaxes(-1, -2)
            got = got.transpose(1, 0, 3, 2, 4).reshape(w.n_layers, -1, w.n_kv_heads, w.head_dim)[:, c:c + n]
            want = cache[:, c:c + n]
            assert np.all(np.abs(got - want) <= rel * np.abs(want) + tol)
        if K:
            _, lo, _, _ = ref[b]
            g = logits[b].cpu().numpy()
            m = np.isfinite(lo)
            assert np.array_equal(m, np.isfinite(g))
            assert np.max(np.abs(g[m] - lo[m])) < tol
            assert drafts[b].cpu().tolist() == ref[b][0].tolist()


@pytest.mark.parametrize("rows", [70, 140, 141])
def test_tree_after_a_prompt_matches_oracle(rows):
    """A tree whose root is the last row of a long ingest."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle.tree import draft_tree
    from paper_2609_09338_amd import workload as WL
    w = synth.get("p_single128")
    from paper_2609_09338_amd import _lib as L
    from paper_2609_09338_amd.binding import Drafter, make_config
    weights, d2t = synth.make_weights(w), synth.make_d2t(w)
    n_blocks = (rows + 24) // 16
    cfg = make_config(n_layers=w.n_layers, d_model=w.d_model, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads,
                      head_dim=w.head_dim, d_ffn=w.d_ffn, vocab_draft=w.vocab_draft, vocab_target=w.vocab_target,
                      target_hidden=w.target_hidden, dtype=L.OSPREY_BF16, qk_norm=w.qk_norm, max_batch=1, max_k=4,
                      max_seq_len=n_blocks * 16, kv_num_blocks=n_blocks, max_new_rows=rows)
    dev = "cuda:0"
    dr = Drafter(cfg, {k: WL.to_dev(v, w, dev) for k, v in weights.items()}, torch.from_numpy(d2t).to(dev))
    dr.seq_reset(0, list(range(n_blocks)))
    toks, taps = synth.prompt_tokens(w, 0, rows), synth.taps(w, 0, 0, rows)
    tk = torch.empty((1, 12), dtype=torch.int32, device=dev)
    pr = torch.empty_like(tk)
    sc = torch.empty((1, 12), dtype=torch.float64, device=dev)
    dr.draft_tree([0], 3, 3, 12, WL.to_dev(taps, w, dev), torch.zeros(1, device=dev), tk, pr, n_new=[rows],
                  new_tokens=torch.from_numpy(toks).to(dev), scores=sc)
    torch.cuda.synchronize()
    assert dr.device_errors() == 0
    o = OH.build_drafter(w, weights, d2t)
    t = draft_tree(o, OH.Sequence(w, rows + 8), toks, taps.astype(np.float64), 3, 3, 12)
    # scores agree on every node both trees hold, and nodes differ only where a selection
    # was closer than four times that measured difference (the rule of test_gpu_tree.py)
    g_tok, g_par, g_sc = tk.cpu().numpy()[0], pr.cpu().numpy()[0], sc.cpu().numpy()[0]
    gk, ok = _path_keys(g_tok, g_par), _path_keys(t.tokens, t.parents)
    want = dict(zip(ok, t.scores))
    err = max(abs(v - want[k]) for k, v in zip(gk, g_sc) if k in want)
    print(f"[tree after a prompt] {rows} rows: score error {err:.2e}, equal {gk == ok}", flush=True)
    assert err < 2e-2
    if gk != ok:
        near = parity.tree_near_tie_keys(t, 4.0 * err + 1e-9)
        assert parity.tree_mismatch_excused(gk, ok, near), (g_tok, t.tokens)


@pytest.mark.parametrize("rows", [(100, 120), (20, 40), (300, 150)])
def test_values_that_are_no_numbers_stay_in_their_sequence(rows):
    """A prompt whose taps are NaN (and one with infinities) beside a sound one, whose cache
    must come out bit for bit as without them."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_09338_amd import _lib as L
    from paper_2609_09338_amd import workload as WL
    from paper_2609_09338_amd.binding import Drafter, make_config
    w = synth.get("p_qwen_small").with_(batch=3, n_layers=3)
    dev, ns = "cuda:0", [rows[0], rows[1], rows[0]]
    nb = max(ns) // 16 + 2
    cfg = make_config(n_layers=w.n_layers, d_model=w.d_model, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads,
                      head_dim=w.head_dim, d_ffn=w.d_ffn, vocab_draft=w.vocab_draft, vocab_target=w.vocab_target,
                      target_hidden=w.target_hidden, dtype=L.OSPREY_BF16, qk_norm=w.qk_norm, max_batch=3, max_k=1,
                      max_seq_len=16 * nb, kv_num_blocks=3 * nb, max_new_rows=sum(ns))
    dr = Drafter(cfg, {k: WL.to_dev(v, w, dev) for k, v in synth.make_weights(w).items()},
                 torch.from_numpy(synth.make_d2t(w)).to(dev))
    toks = torch.from_numpy(np.concatenate([synth.prompt_tokens(w, b, n) for b, n in enumerate(ns)])).to(dev)
    got = []
    for bad in (False, True):
        taps = [WL.to_dev(synth.taps(w, 0, b, n), w, dev) for b, n in enumerate(ns)]
        if bad:
            taps[0][1:] = float("nan")
            taps[2][::2] = float("inf")
        for b in range(3):
            dr.seq_reset(b, range(b * nb, (b + 1) * nb))
        dr.kv.zero_()
        print(f"[prompt] NaN {bad} rows {ns}", flush=True)
        dr.draft_step([0, 1, 2], 0, torch.cat(taps), torch.zeros(3, device=dev), n_new=ns, new_tokens=toks)
        torch.cuda.synchronize()
        assert dr.device_errors() == 0
        got.append(dr.kv.view(torch.int16).view(3, -1)[1].clone())
    assert torch.equal(*got)
    assert bool((got[0] != 0).any())


def test_taps_past_two_gigabytes():
    """Tap rows further apart than a 31-bit byte offset reaches take the other product."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_09338_amd import _lib as L
    from paper_2609_09338_amd import workload as WL
    from paper_2609_09338_amd.binding import Drafter, make_config
    w = synth.get("p_qwen_small").with_(batch=2)
    dev, rows = "cuda:0", [100, 61]
    stride = (1 << 31) // (2 * 2 * w.tap_width) + 1
    weights, d2t = synth.make_weights(w), synth.make_d2t(w)
    cfg = make_config(n_layers=w.n_layers, d_model=w.d_model, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads,
                      head_dim=w.head_dim, d_ffn=w.d_ffn, vocab_draft=w.vocab_draft, vocab_target=w.vocab_target,
                      target_hidden=w.target_hidden, dtype=L.OSPREY_BF16, qk_norm=w.qk_norm, max_batch=2, max_k=1,
                      max_seq_len=112, kv_num_blocks=14, max_new_rows=sum(rows))
    dr = Drafter(cfg, {k: WL.to_dev(v, w, dev) for k, v in weights.items()}, torch.from_numpy(d2t).to(dev))
    toks = [synth.prompt_tokens(w, b, n) for b, n in enumerate(rows)]
    taps = [synth.taps(w, 0, b, n) for b, n in enumerate(rows)]
    far = torch.empty((2, stride, w.tap_width), dtype=torch.bfloat16, device=dev)
    for b, n in enumerate(rows):
        dr.seq_reset(b, range(7 * b, 7 * b + 7))
        far[b, :n] = WL.to_dev(taps[b], w, dev)
    logits = torch.empty((2, 1, w.vocab_draft), device=dev)
    print("[prompt] taps past 2 GB", flush=True)
    dr.draft_step([0, 1], 1, far, torch.zeros(2, device=dev), n_new=rows, taps_stride=stride, draft_logits=logits,
                  new_tokens=torch.from_numpy(np.concatenate(toks).astype(np.int32)).to(dev))
    torch.cuda.synchronize()
    assert dr.device_errors() == 0
    o = OH.build_drafter(w, weights, d2t)
    for b, n in enumerate(rows):
        _, want, _, _ = o.draft(OH.Sequence(w, n + 1), toks[b], taps[b].astype(np.float64), 1, 0.0, np.zeros(1))
        assert np.max(np.abs(logits[b].cpu().numpy() - want)) < 2e-2


@pytest.mark.parametrize("body,rows,K,launches", [("p_qwen_small", 70, 1, 3), ("p_qwen_small", 64, 1, 2),
                                                  ("p_qwen_small", 70, 0, 2), ("p_tiny_f32", 20, 1, 2)])
def test_every_qkv_product_of_an_ingest_is_timed(body, rows, K, launches):
    """A narrowed last layer has two: the keys and values of every row, and the used rows'."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_09338_amd import _lib as L
    from paper_2609_09338_amd import workload as WL
    from paper_2609_09338_amd.binding import KERNEL_QKV, Drafter, make_config
    w = synth.get(body)
    n = rows // 16 + 2
    cfg = make_config(n_layers=w.n_layers, d_model=w.d_model, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads,
                      head_dim=w.head_dim, d_ffn=w.d_ffn, vocab_draft=w.vocab_draft, vocab_target=w.vocab_target,
                      target_hidden=w.target_hidden, dtype=L.OSPREY_BF16 if w.dtype == "bf16" else L.OSPREY_F32,
                      qk_norm=w.qk_norm, max_batch=1, max_k=1, max_seq_len=16 * n, kv_num_blocks=n, max_new_rows=rows)
    dev = "cuda:0"
    dr = Drafter(cfg, {k: WL.to_dev(v, w, dev) for k, v in synth.make_weights(w).items()},
                 torch.from_numpy(synth.make_d2t(w)).to(dev))
    dr.seq_reset(0, range(n))
    dr.kernel_timing((KERNEL_QKV,))
    print(f"[timing] {body} {rows} rows K {K}", flush=True)
    dr.draft_step([0], K, WL.to_dev(synth.taps(w, 0, 0, rows), w, dev), torch.zeros(1, device=dev), n_new=[rows],
                  new_tokens=torch.from_numpy(synth.prompt_tokens(w, 0, rows)).to(dev))
    ms, got = dr.kernel_time(KERNEL_QKV)
    assert got == launches and ms > 0
