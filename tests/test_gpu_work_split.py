"""How the work is split, where a split changes: attention batches of so few tiles that every workgroup takes one run of one
pair and a row's partials are merged by several groups of threads (and the first sizes past either), their backward, and tree
walks whose slices are held in registers or not.  Against the float64 oracle, at the tolerances of parity_util."""
import numpy as np
import pytest

import gen
import oracle

torch = pytest.importorskip("torch")


def _workload(batch, context, nodes, kv8, hq=8, hkv=2):
    kw = dict(batch=batch, vocab=64, hidden_size=64, num_q_heads=hq, num_kv_heads=hkv, kv_fp8=kv8)
    if nodes:
        return gen.llama_tree(300 + batch + context, num_q=nodes, context=context, **kw)
    return gen.llama_chain(300 + batch + context, len_lo=max(5, context - 40), len_hi=context, **kw)


@pytest.mark.gpu
@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("batch,context,nodes,hkv", [(1, 5, 0, 2), (1, 33, 0, 2), (1, 700, 0, 1), (1, 2777, 0, 2), (3, 1500, 7, 2),
                                                     (12, 300, 0, 2), (24, 200, 0, 2), (1, 40, 24, 1), (1, 2777, 32, 2),
                                                     (9, 500, 32, 2), (2, 900, 61, 2),
                                                     # as many runs as workgroups, and one request more
                                                     (256, 40, 0, 2), (257, 40, 0, 2), (128, 60, 24, 2), (129, 60, 24, 2),
                                                     (40, 400, 0, 2), (16, 300, 24, 1)])
def test_attention_of_few_tiles(gpu_lib, batch, context, nodes, hkv, kv8):
    from paper_2602_06932_amd.device import DeviceVerify
    from parity_util import check_attention
    w = _workload(batch, context, nodes, kv8, hq=4 * hkv, hkv=hkv)
    dv = DeviceVerify(w)
    dv.attn_out.fill_(float("nan"))
    dv.attn()
    torch.cuda.synchronize()
    check_attention(dv.attn_out_host(), oracle.attn_workload(w), w.dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("batch,hq", [(1024, 4), (1030, 4), (1030, 16)])
def test_attention_of_many_short_requests(gpu_lib, batch, hq, kv8):
    """The last size whose split the workgroups build themselves, and past it, where it is read from the planning kernel's prefix."""
    from paper_2602_06932_amd.device import DeviceVerify
    from parity_util import check_attention
    w = gen.llama_chain(170, batch=batch, num_q=5, num_q_heads=hq, num_kv_heads=2, len_lo=5, len_hi=70, vocab=64, hidden_size=64,
                        kv_fp8=kv8)
    dv = DeviceVerify(w)
    dv.attn_out.fill_(float("nan"))
    dv.attn()
    torch.cuda.synchronize()
    check_attention(dv.attn_out_host(), oracle.attn_workload(w), w.dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("num_q,tiles,batch", [(8, 1, 1), (8, 4, 1), (8, 5, 3), (8, 87, 1), (8, 10, 12), (32, 1, 1), (32, 4, 1), (32, 5, 2),
                                               (32, 86, 1), (32, 5, 12)])
def test_infinities_at_nodes_a_row_does_not_see(gpu_lib, num_q, tiles, batch, kv8):
    """The last tile of 32 tokens holds only the later nodes of the chunk, and the last of them has infinities (NaN codes in an
    8-bit cache) in K and V: rows that see nothing of that tile come out as if it were not there.  (So few tiles that no wavefront
    multiplies another tile into the same sums; where one does, the product's 0 x infinity stays in them.)"""
    from paper_2602_06932_amd.device import DeviceVerify
    from parity_util import check_attention
    first = {8: 4, 32: 16}[num_q]  # the first node in the last tile
    length = 32 * tiles + num_q - first
    w = gen.llama_chain(300 + batch + length, len_lo=length, len_hi=length, num_q=num_q, batch=batch, vocab=64, hidden_size=64,
                        num_q_heads=8, num_kv_heads=2, kv_fp8=kv8)
    assert (w.seq_lens == length).all()
    ref = oracle.attn_workload(w)
    dv = DeviceVerify(w)
    at = (length - 1) // w.page_size
    for pool in (dv.k_pages, dv.v_pages):
        for b in range(batch):
            pool[int(w.block_table[b, at]), :, (length - 1) % w.page_size, :] = 0x7F if kv8 else float("inf")
    dv.attn()
    torch.cuda.synchronize()
    check_attention(dv.attn_out_host()[:, :first], ref[:, :first], w.dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("batch,context,nodes", [(1, 40, 0), (1, 1500, 0), (1, 1500, 12), (1, 1500, 32), (5, 333, 32),
                                                 # as many runs as workgroups, one request more, short pairs in fours
                                                 (128, 60, 0), (129, 60, 0), (129, 60, 12), (300, 60, 5), (128, 60, 32), (129, 60, 32)])
def test_backward_of_few_tiles(gpu_lib, batch, context, nodes):
    from test_gpu_attn_bwd import _check
    _check(_workload(batch, context, nodes, False), 11)


@pytest.mark.gpu
@pytest.mark.parametrize("batch,num_q,vocab,wor", [(130, 6, 9000, False), (130, 6, 9000, True),   # 36 groups: held, not held
                                                   (130, 6, 12288, False), (130, 6, 12289, False), # one slice of 48 groups: held; 49
                                                   (130, 6, 13000, False),                      # one workgroup, not held
                                                   (130, 6, 40000, False), (130, 4, 70000, True),  # ... in several slices
                                                   (50, 8, 70000, False),                       # five slices of 55 groups: not held
                                                   (64, 8, 49152, False),                       # four slices of 48 groups: held
                                                   (12, 16, 8192, True), (12, 16, 8193, True),  # 32 groups: the first split in two
                                                   (12, 16, 12288, False), (12, 16, 12289, False),  # 48: one workgroup; 49: split
                                                   (3, 64, 20011, False), (3, 64, 20011, True)])  # as many sweeps as there can be
def test_tree_walk_slices(gpu_lib, batch, num_q, vocab, wor):
    from test_gpu_parity import _full_check
    w = gen.llama_tree(400 + batch, batch=batch, num_q=num_q, vocab=vocab, hidden_size=64, context=70, num_q_heads=2,
                       num_kv_heads=1, draft_noise=1.5, siblings_without_replacement=wor)
    _, a = _full_check(gpu_lib, w)
    assert 0 < np.mean(a.accept_len) < num_q - 1
