"""Small calls: a float32 step whose attention and LM head share a launch and whose acceptance forms the rows' statistics from the
logits, against the same step in its three stages (statistics by a kernel of their own) and against the oracle."""
import numpy as np
import pytest

import gen
import oracle

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("temps", [False, True])
@pytest.mark.parametrize("batch,num_q,vocab,hidden,lens,dim", [(1, 1, 1, 8, (1, 9), 64), (4, 5, 1024, 256, (256, 256), 64), (3, 7, 1023, 64, (7, 300), 64), (3, 4, 2048, 64, (9, 99), 64), (3, 4, 2049, 64, (9, 99), 64),
                                                           (8, 2, 2003, 72, (64, 512), 64), (2, 5, 8192, 96, (30, 60), 64),
                                                           # past one slice; past the small LM-head tiles; past one split
                                                           (2, 5, 8193, 32, (30, 60), 64), (40, 8, 2048, 64, (20, 40), 64), (2, 4, 500, 64, (500, 700), 64), (4, 5, 2001, 64, (7, 300), 128), (2, 4, 500, 64, (500, 700), 128),
                                                           # several rows a wavefront: formed in the sweep up to three tiles each, ..
                                                           (2, 9, 1000, 32, (30, 60), 64), (3, 24, 1024, 32, (30, 60), 64), (130, 17, 1100, 32, (30, 60), 64),
                                                           # .. or by the launch
                                                           (2, 25, 1000, 32, (30, 60), 64), (3, 9, 1100, 32, (30, 60), 64), (127, 9, 1100, 32, (30, 60), 64),
                                                           # long contexts: in one launch with the head, and in two
                                                           (1, 1, 500, 64, (40000, 40000), 128), (1, 1, 8000, 64, (40000, 40000), 128),
                                                           (2, 8, 100, 64, (34000, 34000), 64),
                                                           # the head's tiles past one round of the shared kernel
                                                           (3, 11, 8000, 1028, (60, 64), 128)])
def test_float32_step_equals_its_stages(gpu_lib, batch, num_q, vocab, hidden, lens, dim, temps):
    from paper_2602_06932_amd.device import DeviceVerify
    from parity_util import check_accept, check_attention, check_logits
    kw = {}
    if temps:
        kw = dict(draft="noisy_target", temperatures=np.array([0.0, 0.6, 1.0, 0.8] * batch, np.float32)[:batch])
    seq = np.linspace(lens[0], lens[1], batch).astype(np.int32)
    w = gen.make_workload(name="small", seed=40 + vocab, seq_lens=np.maximum(seq, num_q).astype(np.int32), recipe="", batch=batch, num_q=num_q,
                          num_q_heads=8, num_kv_heads=2, head_dim=dim, page_size=256, hidden_size=hidden, vocab=vocab,
                          temperature=1.0, dtype=gen.F32, **{"draft": "independent", **kw})
    one, parts = DeviceVerify(w), DeviceVerify(w)
    one.workspace.fill_(255)  # (statistics that are read before they are written would be NaN)
    parts.workspace.fill_(255)
    one.verify()
    parts.attn(), parts.lmhead(), parts.accept_logits()
    torch.cuda.synchronize()
    assert np.array_equal(one.attn_out_host(), parts.attn_out_host())
    ref_o, ref_a = oracle.verify(w, want_cdf=True, want_logits=True)
    check_attention(one.attn_out_host(), ref_o, w.dtype)
    check_logits(one.logits_host(), ref_a.logits, w.dtype)
    check_accept(one.results_host(), ref_a, w)
    a, b = one.results_host(), parts.results_host()
    for n in a:
        assert np.array_equal(a[n], b[n]), n
    # the step leaves the statistics behind as the stages do: acceptance alone, on its part of the workspace
    attn_bytes = gpu_lib.aurora_verify_logits_ptr(one.attn_desc, one.accept_desc, one.workspace) - \
        gpu_lib.aurora_verify_logits_ptr(None, one.accept_desc, one.workspace)
    one.accept_len.fill_(-1), one.next_token.fill_(-1)
    gpu_lib.aurora_verify_accept_logits(one.accept_desc, one.draft_tokens, one.draft_probs, one.uniforms, None, one.accept_len,
                                        one.next_token, one.accept_mask, one.p_at_draft, one.row_lse, one.workspace[attn_bytes:])
    torch.cuda.synchronize()
    c = one.results_host()
    for n in a:
        assert np.array_equal(a[n], c[n]), n


@pytest.mark.gpu
@pytest.mark.parametrize("temps", [False, True])
@pytest.mark.parametrize("kind", ["nan_entry", "nan_row", "inf_entry"])
@pytest.mark.parametrize("vocab", [1, 1000, 1024, 2001, 2048])
def test_logits_that_are_not_finite(gpu_lib, vocab, kind, temps):
    """A NaN logit reaches the row's logsumexp, and with it the accept tests, wherever the statistics are formed."""
    from paper_2602_06932_amd.device import DeviceVerify
    kw = dict(temperatures=np.array([0.0, 0.6, 1.0, 0.8], np.float32)) if temps else {}
    w = gen.make_workload(name="small", seed=60 + vocab, seq_lens=np.full(4, 20, np.int32), recipe="", batch=4, num_q=5, num_q_heads=4,
                          num_kv_heads=2, head_dim=64, page_size=16, hidden_size=64, vocab=vocab, temperature=1.0, dtype=gen.F32,
                          draft="noisy_target", **kw)
    dv = DeviceVerify(w)
    if kind == "nan_row":  # every logit of a request's third row
        dv.hidden.view(4, 5, 64)[1, 2, 7] = float("nan")
    else:                  # one logit of every row: the vocabulary's last
        dv.lm_head.view(vocab, 64)[-1, 3] = float(kind[:3])
    dv.accept()
    torch.cuda.synchronize()
    one = {n: x.copy() for n, x in dv.results_host().items()}
    dv.workspace.fill_(255)
    for t in (dv.accept_len, dv.next_token, dv.accept_mask):
        t.fill_(9)
    dv.lmhead(), dv.accept_logits()
    torch.cuda.synchronize()
    two = dv.results_host()
    for n in one:
        assert np.array_equal(one[n], two[n], equal_nan=True), n
    if kind == "nan_entry" and vocab > 1:  # (a row of nothing else has no maximum: its logsumexp is -inf)
        assert np.isnan(one["row_lse"]).all()
        sampled = np.arange(4) > 0 if temps else np.full(4, True)
        assert (one["accept_len"][sampled] == 0).all()


@pytest.mark.gpu
@pytest.mark.parametrize("where", ["hidden", "hidden_part", "lm_head"])
def test_head_that_reads_what_attention_writes(gpu_lib, where):
    """Hidden states (or W) that lie in attention's output: the step is attention, then the LM head, as its stages are."""
    from paper_2602_06932_amd.device import DeviceVerify
    w = gen.make_workload(name="small", seed=70, seq_lens=np.full(4, 300, np.int32), recipe="", batch=4, num_q=5, num_q_heads=8,
                          num_kv_heads=2, head_dim=64, page_size=64, hidden_size=512, vocab=20 if where == "lm_head" else 1000,
                          temperature=1.0, dtype=gen.F32, draft="noisy_target")
    dv = DeviceVerify(w)
    room = torch.zeros(3 * 20 * 512, device="cuda")
    attn_out = room[20 * 512:40 * 512]
    hidden, lm_head = dv.hidden, dv.lm_head
    if where == "lm_head":
        lm_head = attn_out
    else:  # the same rows, or rows that begin in the output's last quarter
        hidden = attn_out if where == "hidden" else room[35 * 512:55 * 512]

    def step(*stages):
        room.zero_()
        dv.workspace.fill_(255)
        for t in (dv.accept_len, dv.next_token, dv.accept_mask):
            t.fill_(9)
        torch.cuda.synchronize()
        kv = (dv.q, dv.k_pages, dv.v_pages, dv.block_table, dv.seq_lens, None, attn_out)
        acc = (hidden, lm_head, dv.draft_tokens, dv.draft_probs, dv.uniforms)
        res = (dv.accept_len, dv.next_token, dv.accept_mask, dv.p_at_draft, dv.row_lse, dv.workspace)
        if stages:
            gpu_lib.aurora_verify_attn(dv.attn_desc, *kv, dv.workspace)
            torch.cuda.synchronize()
            gpu_lib.aurora_verify_accept(dv.accept_desc, *acc, None, *res)
        else:
            gpu_lib.aurora_verify(dv.attn_desc, dv.accept_desc, *kv, *acc, *res)
        torch.cuda.synchronize()
        return {**{n: x.copy() for n, x in dv.results_host().items()}, "out": attn_out.cpu().numpy()}

    one, two = step(), step("attention", "accept")
    assert np.abs(one["out"]).max() > 0
    for n in one:
        assert np.array_equal(one[n], two[n]), n
