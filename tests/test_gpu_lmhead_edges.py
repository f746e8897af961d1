"""LM head on the matrix cores at the sizes where its tiles and rings end: hidden sizes of one stage and a few (fewer than the rings
hold, odd numbers of them), token rows at the borders between kernels and column widths, vocabularies that end anywhere in a
tile.  Logits against float64 products, row statistics and group maxima against the logits themselves."""
import pytest

torch = pytest.importorskip("torch")

ROWS = [1, 16, 17, 33, 65, 97, 128, 129, 160, 161, 193, 225, 256, 257, 320, 321, 353, 385, 417, 449, 512, 513, 641]


def _check(av, rows, vocab, hidden, fp8, seed):
    print(f"[case] rows {rows} vocab {vocab} hidden {hidden} fp8 {fp8}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(seed)
    h = torch.randn((rows, hidden), device="cuda", generator=g)
    w = torch.randn((vocab, hidden), device="cuda", generator=g) * 0.05
    kw = {}
    if fp8:
        sh, sw = (x.abs().amax(1) / 448 for x in (h, w))
        h8, w8 = ((x / s[:, None]).to(torch.float8_e4m3fn) for x, s in ((h, sh), (w, sw)))
        hd, wd = h8.double() * sh.double()[:, None], w8.double() * sw.double()[:, None]
        h, w = h8.view(torch.uint8), w8.view(torch.uint8)
        kw = dict(hidden_scale=sh.data_ptr(), lm_head_scale=sw.data_ptr())
    else:
        h, w = h.to(torch.bfloat16), w.to(torch.bfloat16)
        hd, wd = h.double(), w.double()
    # greedy, one position a request: the token is the row's arg-max, the row's logsumexp is taken at T = 1
    d = av.aurora_accept_desc(batch=rows, num_q=1, hidden=hidden, vocab=vocab, dtype=av.AURORA_FP8_E4M3 if fp8 else av.AURORA_BF16,
                              temperature=0.0, **kw)
    # what lies behind the workspace's end of use must not matter: fill it with NaN
    ws = torch.full((av.aurora_verify_workspace_bytes(None, d),), 255, dtype=torch.uint8, device="cuda")
    av.aurora_verify_lmhead(d, h, w, ws)
    off = av.aurora_verify_logits_ptr(None, d, ws) - ws.data_ptr()
    z = ws[off:off + 4 * rows * vocab].view(torch.float32).view(rows, vocab).clone()
    gptr, n_groups = av.aurora_verify_group_max_ptr(None, d, ws)
    off = gptr - ws.data_ptr()
    gm = ws[off:off + 4 * rows * n_groups].view(torch.float32).view(rows, n_groups).clone()
    tok = torch.zeros((rows, 1), dtype=torch.int32, device="cuda")
    out = {n: torch.empty(s, dtype=t, device="cuda") for n, s, t in
           (("len", rows, torch.int32), ("next", rows, torch.int32), ("mask", (rows, 1), torch.uint8),
            ("p", (rows, 1), torch.float32), ("lse", (rows, 1), torch.float32))}
    av.aurora_verify_accept_logits(d, tok, None, None, None, out["len"], out["next"], out["mask"], out["p"], out["lse"], ws)
    torch.cuda.synchronize()
    err = (z.double() - hd @ wd.T).abs()
    if fp8:
        # the 8-bit instruction adds the products of a step in fixed point under the largest of them (seen: 2^-17 of the sum of
        # magnitudes at 128 products); each product loses at most 2^-16 of the row's largest
        bound = hidden * 2.0 ** -16 * hd.abs().amax(1)[:, None] * wd.abs().amax(1)[None]
    else:  # sums of H exact products in float32, in any order
        bound = hidden * 2.0 ** -24 * (hd.abs() @ wd.abs().T)
    assert bool((err <= bound).all()), float((err / bound).max())
    # group maxima and arg-max are those of the stored logits, the logsumexp theirs up to float32 sums of exponentials
    pad = torch.nn.functional.pad(z, (0, 32 * n_groups - vocab), value=float("-inf")).view(rows, n_groups, 32).amax(2)
    assert torch.equal(gm, pad)
    assert torch.equal(out["next"].long(), z.argmax(1))
    assert float((out["lse"][:, 0].double() - torch.logsumexp(z.double(), 1)).abs().max()) <= 2e-5


@pytest.mark.gpu
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("rows", ROWS)
def test_lmhead_at_the_edges(gpu_lib, rows, fp8):
    unit = 128 if fp8 else 64  # hidden elements of a stage
    for i, (vocab, stages) in enumerate([(256, 1), (257, 2), (1000, 3), (63, 4), (2085, 5), (516, 7)]):
        _check(gpu_lib, rows, vocab, unit * stages, fp8, 1000 * rows + i)


@pytest.mark.gpu
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("rows", [161, 192, 193, 225, 256, 321, 352, 383])
def test_tiled_lmhead_of_one_round_less(gpu_lib, rows, fp8):
    """171 vocabulary tiles: enough that the tiled kernel takes these rows from the W-streaming one, which has the small
    vocabularies above."""
    unit = 128 if fp8 else 64
    for i, (vocab, stages) in enumerate([(43525, 1), (43776, 2), (43522, 3), (43772, 5)]):
        _check(gpu_lib, rows, vocab, unit * stages, fp8, 2000 * rows + i)
