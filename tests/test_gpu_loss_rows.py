"""Drafter loss where its row kernel can go wrong: rows that do not start at 16 bytes (elements before and after the vectors),
base pointers that are aligned differently, vocabularies at the edges of the register paths, kept tokens on every side of the LDS turns, and class counts formed by the
rows' workgroups or by a kernel of their own - against the float64 oracle."""
import numpy as np
import pytest

import gen
import oracle

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("rows,vd,k", [(5, 8, 4), (6, 9, 9), (7, 11, 3), (9, 16385, 1000), (5, 16387, 1024), (4, 32767, 1024),
                                       (3, 32768, 700), (3, 32769, 64), (8193, 40, 8), (8192, 41, 8), (4099, 33, 33),
                                       (5, 4095, 1024), (5, 4096, 1024), (6, 4097, 1024), (5, 8191, 64), (4, 8192, 1024),
                                       (5, 8193, 500), (2048, 37, 5), (2049, 37, 5), (8193, 4200, 4), (4, 1, 1), (9, 7, 7)])
def test_rows_of_any_alignment_and_length(gpu_lib, rows, vd, k):
    _check_rows(gpu_lib, rows, vd, k)


@pytest.mark.gpu
@pytest.mark.parametrize("z_off,grad_off,traj_off", [(1, 1, 0), (2, 2, 1), (3, 3, 0), (0, 1, 0), (3, 0, 2), (0, 0, 3)])
@pytest.mark.parametrize("rows,vd,k", [(6, 1000, 64), (5, 4100, 1024), (4, 20000, 700)])
def test_base_pointers_of_any_alignment(gpu_lib, rows, vd, k, z_off, grad_off, traj_off):
    """draft_logits and grad off a 16-byte boundary by the same number of floats (registers) or by different ones (three
    passes), and trajectory codes off a 4-byte boundary (counted by a kernel of its own)."""
    _check_rows(gpu_lib, rows, vd, k, z_off, grad_off, traj_off)


def _shifted(t, off):
    """The tensor's values `off` elements into a larger buffer."""
    buf = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
    out = buf[off:off + t.numel()].view(t.shape)
    out.copy_(t)
    return out


def _check_rows(gpu_lib, rows, vd, k, z_off=0, grad_off=0, traj_off=0):
    av = gpu_lib
    z, ids, bits, traj = gen.loss_inputs(7 + vd, rows, vd, top_k=k)
    keep = min(k, vd)
    if vd > 40:  # the first and last entries of the row, and both sides of the turns' edge, among the kept tokens
        for m in range(rows):
            want = [v for v in dict.fromkeys((0, 2, 3, vd - 1, vd - 4, 16383, 16384, 16387)) if 0 <= v < vd][:keep]
            rest = [i for i in ids[m, :keep].tolist() if i not in want]
            ids[m, :keep] = (want + rest)[:keep]
    ref = oracle.draft_loss(z, ids, bits, traj, 0.5, None)
    d = av.aurora_loss_desc(rows=rows, draft_vocab=vd, top_k=k, discard_top_k=0, lambda_discard=0.5)
    dev = [_shifted(torch.from_numpy(a), off) for a, off in ((z, z_off), (ids, 0), (bits.view(np.int16), 0), (traj, traj_off))]
    kl, loss = torch.empty(rows, device="cuda"), torch.empty(5, device="cuda")
    grad = _shifted(torch.full((rows, vd), float("nan")), grad_off)
    av.aurora_draft_loss(d, *dev, kl, loss, grad)
    torch.cuda.synchronize()
    w = max(1.0 / max(1, ref["n_accept"]), 0.5 / max(1, ref["n_discard"]))
    # fp32 exponentials (a few ulp of a probability of at most 1) in both terms, times the row's weight
    assert np.abs(grad.cpu().numpy() - ref["grad"]).max() <= 4e-6 * w
    assert (np.abs(kl.cpu().numpy() - ref["row_kl"]) <= 2e-5 + 1e-5 * np.abs(ref["row_kl"])).all()
    assert loss[3].item() == ref["n_accept"] and loss[4].item() == ref["n_discard"]
    assert abs(loss[0].item() - ref["loss"]) <= 2e-5 * max(1.0, abs(ref["loss"]))


def _many_rows(gpu_lib, rows, accepted, unused, want_grad):
    """`rows` rows, eight prototypes over and over: `accepted` of them accepted, `unused` unused, the rest discarded."""
    av = gpu_lib
    z, ids, bits, _ = gen.loss_inputs(3, 8, 8, top_k=4)
    reps = -(-rows // 8)
    traj = torch.full((rows,), 2, dtype=torch.int8, device="cuda")
    traj[accepted] = 1
    traj[unused] = 0
    dev = [torch.from_numpy(a).cuda().repeat(reps, 1)[:rows] for a in (z, ids, bits.view(np.int16))]
    kl, loss = torch.empty(rows, device="cuda"), torch.empty(5, device="cuda")
    grad = torch.full((rows, 8), float("nan"), device="cuda") if want_grad else None
    d = av.aurora_loss_desc(rows=rows, draft_vocab=8, top_k=4, discard_top_k=0, lambda_discard=0.5)
    print(f"[case] rows={rows} grad={want_grad}", flush=True)
    av.aurora_draft_loss(d, *dev, traj, kl, loss, grad)
    torch.cuda.synchronize()
    # the oracle on the prototypes, each in either class (no discard filter: a row's KL does not depend on its class)
    per_row = oracle.draft_loss(z, ids, bits, np.ones(8, np.int8), 0.5)["row_kl"]
    n_a, n_d = len(accepted), rows - len(accepted) - len(unused)
    count = np.bincount(np.arange(rows) % 8, minlength=8).astype(np.float64)
    gone = np.bincount(np.array(accepted + unused, np.int64) % 8, minlength=8)
    mean_a = float(np.mean([per_row[i % 8] for i in accepted]))
    mean_d = float((per_row * (count - gone)).sum() / n_d)
    assert loss[3].item() == np.float32(n_a) and loss[4].item() == np.float32(n_d)
    for got, want in ((loss[0], mean_a + 0.5 * mean_d), (loss[1], mean_a), (loss[2], mean_d)):
        assert abs(got.item() - want) <= 2e-5 + 1e-5 * abs(want)
    return per_row, traj, kl, grad, n_a, n_d


@pytest.mark.gpu
@pytest.mark.parametrize("rows,n_accept,want_grad", [(2_200_000, 1, False), (2_200_000, 1, True), (4_300_000, 5, False)])
def test_class_counts_of_millions_of_rows(gpu_lib, rows, n_accept, want_grad):
    """Both class counts are exact whatever the number of discarded rows (their sum is a whole number of up to 62 bits)."""
    _many_rows(gpu_lib, rows, [7 + 411_111 * i for i in range(n_accept)], [5, rows - 1], want_grad)


@pytest.mark.gpu
def test_more_rows_than_one_grid_dimension_holds(gpu_lib):
    """A grid dimension takes fewer than 2^32 threads: above 2^23 rows of 512 threads the rows run on in a second one."""
    rows = (1 << 23) + 1037
    per_row, traj, kl, grad, n_a, n_d = _many_rows(gpu_lib, rows, [11, (1 << 22) + 3, rows - 2], [5, rows - 1], True)
    at = torch.arange(rows, device="cuda") % 8
    want = torch.tensor(per_row, device="cuda")[at]
    assert ((kl.double() - want).abs() <= 2e-5 + 1e-5 * want.abs()).all()
    assert torch.isfinite(grad).all() and (grad[5] == 0).all() and (grad[rows - 1] == 0).all()
    # equal rows of a class have equal gradients, bit for bit
    first = torch.full((8,), -1, device="cuda")
    for i in range(8, 16):
        first[i % 8] = i if traj[i] == 2 else i + 8
    same = (grad == grad[first[at]]).all(1) | (traj != 2)
    assert same.all()
