"""osprey_graph_*: one steady-state iteration (pending draft call + verification)
captured as a HIP graph over fixed buffers and replayed.

Every replay must give bit-for-bit the results of the same iteration launched call
by call (the kernels and their order are the same), with the program's own eager
work (copying the next iteration's inputs into the captured buffers) between
replays.  The host state must advance as the two calls would, and misuse must be
refused before anything is enqueued."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _require_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_09338_amd import _lib
    _lib.load()


def _say(*a):
    print(*a, flush=True)


def _reference(w, n_it):
    """Stream launches: per iteration the inputs, the target logits and the outputs."""
    from paper_2609_09338_amd import workload as WL
    s = WL.make_drafter(w, n_it)
    WL.reset_sequences(s)
    out = WL.alloc_outputs(s)
    rec = []
    for it in range(n_it):
        inp = WL.iter_inputs(s, it)
        WL.draft(s, it, inp, out)
        tl = WL.synthetic_target(s, it, out.logits)
        WL.verify(s, inp, tl, out)
        torch.cuda.synchronize()
        rec.append((inp, tl, [t.clone() for t in (out.drafts, out.logits, out.accept_len,
                                                   out.mask, out.tokens)]))
    return s, out, rec


# (twelve sequences: an ingest of 72 planned rows narrows its last layer, as 17 fp32 rows do; contexts of 1100:
# ingests that attend by blocks of query vectors over several splits, planned for the longer
# contexts of a graph)
@pytest.mark.parametrize("name,change", [("p_qwen_small", {}), ("p_single128", {}), ("p_block", {}),
                                         ("p_qwen_small", dict(batch=12)), ("p_tiny_f32", dict(K=16)), ("p_block", dict(ctx_lo=1090, ctx_hi=1100)),
                                         ("p_single64", dict(ctx_lo=1100, ctx_hi=1100)),
                                         ("p_block", dict(batch=1, ctx_lo=2040, ctx_hi=2040)),
                                         # (merged by the O projection, by the merge kernel in the graph)
                                         ("p_block", dict(batch=2, ctx_lo=990, ctx_hi=990)),
                                         ("p_single64", dict(ctx_lo=100, ctx_hi=100))])
def test_graph_replays_equal_stream_launches(name, change):
    _require_gpu()
    from paper_2609_09338_amd import workload as WL
    w = synth.get(name).with_(**change)
    n_it = 5
    _say(f"[graph] {name}: stream reference")
    s, out, rec = _reference(w, n_it)
    B = w.batch
    # back to the start, on a stream of its own, iteration 0 (explicit) call by call
    st = torch.cuda.Stream()
    s.drafter.set_stream(st)
    for b in range(B):
        s.drafter.seq_truncate(b, int(s.ctx[b]) - 1)
    inp0, tl0, _ = rec[0]
    WL.draft(s, 0, inp0, out)
    WL.verify(s, inp0, tl0, out)
    # fixed input buffers the graph reads
    fx_taps = torch.empty_like(inp0.taps)
    fx_ud, fx_ua, fx_ub = (torch.empty_like(inp0.u_draft), torch.empty_like(inp0.u_accept),
                           torch.empty_like(inp0.u_bonus))
    fx_tl = torch.empty_like(tl0)
    mask = synth.mask_token(w) if w.drafting == "block" else None
    _say(f"[graph] {name}: capture")
    g = s.drafter.capture_iteration(list(range(B)), w.K, fx_taps, s.draft_temperature, fx_ud,
                                    out.drafts, out.logits, fx_tl, s.temperature, fx_ua, fx_ub,
                                    out.accept_len, out.mask, out.tokens,
                                    max_context=int(s.drafter.cfg.max_seq_len),
                                    taps_stride=w.K + 1, mask_token=mask)
    for it in range(1, n_it):
        inp, tl, ref = rec[it]
        with torch.cuda.stream(st):
            for dst, src in ((fx_taps, inp.taps), (fx_ud, inp.u_draft), (fx_ua, inp.u_accept),
                             (fx_ub, inp.u_bonus), (fx_tl, tl)):
                dst.copy_(src)
        g.launch()
        st.synchronize()
        _say(f"[graph] {name}: replay {it}")
        for got, want in zip((out.drafts, out.logits, out.accept_len, out.mask, out.tokens), ref):
            assert torch.equal(got, want), (name, it)
    assert s.drafter.device_errors() == 0
    # the host state advanced as the calls would: the next call-by-call iteration is allowed
    # and lands where the recorded trajectory says
    lengths = [s.drafter.seq_length(b) for b in range(B)]
    want = [int(s.ctx[b]) + sum(int(rec[j][2][2][b]) + 1 for j in range(n_it - 1))
            for b in range(B)]
    assert lengths == want, (lengths, want)
    g.close()


def test_graph_misuse_is_refused():
    _require_gpu()
    from paper_2609_09338_amd import _lib as L
    from paper_2609_09338_amd import workload as WL
    from paper_2609_09338_amd.binding import OspreyError
    w = synth.get("p_single128")
    s, out, rec = _reference(w, 2)
    inp, tl, _ = rec[1]
    args = ([0], w.K, inp.taps, s.draft_temperature, inp.u_draft, out.drafts, out.logits, tl,
            s.temperature, inp.u_accept, inp.u_bonus, out.accept_len, out.mask, out.tokens)
    kw = dict(max_context=int(s.drafter.cfg.max_seq_len), taps_stride=w.K + 1)

    def code(fn):
        with pytest.raises(OspreyError) as e:
            fn()
        return e.value.status

    # the null stream cannot be captured
    assert code(lambda: s.drafter.capture_iteration(*args, **kw)) == L.OSPREY_E_INVALID
    st = torch.cuda.Stream()
    s.drafter.set_stream(st)
    # kernel timing on
    s.drafter.kernel_timing((0,))
    assert code(lambda: s.drafter.capture_iteration(*args, **kw)) == L.OSPREY_E_STATE
    s.drafter.kernel_timing(())
    # a context bound the slot already exceeds
    assert code(lambda: s.drafter.capture_iteration(*args, max_context=8,
                                                    taps_stride=w.K + 1)) == L.OSPREY_E_CAPACITY
    g = s.drafter.capture_iteration(*args, **kw)
    # capturing ran nothing and changed no state: the slot is still VERIFIED and a
    # call-by-call iteration still works
    WL.draft(s, 1, inp, out)
    # DRAFTED now: a graph launch needs VERIFIED slots
    assert code(g.launch) == L.OSPREY_E_STATE
    WL.verify(s, inp, tl, out)
    g.launch()
    st.synchronize()
    assert s.drafter.device_errors() == 0
    g.close()


@pytest.mark.parametrize("name,k0", [("p_single128", 1), ("p_qwen_small", 2), ("p_tiny_f32", 1)])
def test_graph_captured_after_a_shorter_draft(name, k0):
    """A graph of K drafts captured while the slots hold what a call with fewer drafts left
    pending: its later launches ingest up to K + 1 tokens each.  (The calls plan fewer rows
    for the first iteration, so logits are compared within the parity tests' tolerances.)"""
    _require_gpu()
    from paper_2609_09338_amd import workload as WL
    w = synth.get(name).with_(temps=(0.0,), draft_temps=(), sigma=0.01)
    n_it, B = 5, w.batch
    s = WL.make_drafter(w, n_it)
    out = WL.alloc_outputs(s)
    inps = [WL.iter_inputs(s, it) for it in range(n_it)]
    short = dict(drafts=torch.empty((B, k0), dtype=torch.int32, device=s.device),
                 mask=torch.empty((B, k0), dtype=torch.uint8, device=s.device),
                 tokens=torch.empty((B, k0 + 1), dtype=torch.int32, device=s.device),
                 logits=torch.empty((B, k0, w.vocab_draft), device=s.device))
    targets = []

    def first():
        WL.reset_sequences(s)
        dr, i = s.drafter, inps[0]
        dr.draft_step(list(range(B)), k0, i.taps, s.draft_temperature, i.u_draft[:, :k0].contiguous(), n_new=[1] * B,
                      new_tokens=i.new_tokens, taps_stride=w.K + 1, draft_tokens=short["drafts"],
                      draft_logits=short["logits"])
        if not targets:
            full = torch.cat([short["logits"], short["logits"][:, -1:].expand(-1, w.K - k0, -1)], 1)
            targets.append(WL.synthetic_target(s, 0, full.contiguous())[:, :k0 + 1].contiguous())
        dr.verify(list(range(B)), k0, targets[0], s.temperature, i.u_accept[:, :k0].contiguous(), i.u_bonus,
                  out.accept_len, short["mask"], short["tokens"], draft_temperature=s.draft_temperature)

    first()
    ref = []
    for it in range(1, n_it):
        WL.draft(s, it, inps[it], out)
        targets.append(WL.synthetic_target(s, it, out.logits))
        WL.verify(s, inps[it], targets[it], out)
        torch.cuda.synchronize()
        ref.append([t.clone() for t in (out.drafts, out.logits, out.accept_len, out.mask, out.tokens)])
    accepted = [int(r[2].max()) for r in ref]
    assert max(accepted[:-1]) > k0, accepted        # (else nothing would be cut short)
    st = torch.cuda.Stream()
    s.drafter.set_stream(st)
    first()
    st.synchronize()
    fx = [torch.empty_like(t) for t in (inps[1].taps, inps[1].u_draft, targets[1], inps[1].u_accept, inps[1].u_bonus)]
    _say(f"[graph] {name}: capture after {k0} drafts, accepted {accepted}")
    g = s.drafter.capture_iteration(list(range(B)), w.K, fx[0], s.draft_temperature, fx[1], out.drafts, out.logits, fx[2],
                                    s.temperature, fx[3], fx[4], out.accept_len, out.mask, out.tokens,
                                    max_context=int(s.drafter.cfg.max_seq_len), taps_stride=w.K + 1)
    for it in range(1, n_it):
        i = inps[it]
        with torch.cuda.stream(st):
            for dst, src in zip(fx, (i.taps, i.u_draft, targets[it], i.u_accept, i.u_bonus)):
                dst.copy_(src)
        g.launch()
        st.synchronize()
        for got, want in zip((out.drafts, out.accept_len, out.mask, out.tokens), ref[it - 1][:1] + ref[it - 1][2:]):
            assert torch.equal(got, want), (name, it)
        m = torch.isfinite(ref[it - 1][1])
        assert torch.equal(m, torch.isfinite(out.logits))
        assert float((out.logits - ref[it - 1][1])[m].abs().max()) < (2e-2 if w.dtype == "bf16" else 1e-4)
    assert s.drafter.device_errors() == 0
    g.close()
