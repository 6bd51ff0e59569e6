"""GPU parity of attention over key tiles shared by a block of query rows
(dense attention of many rows per sequence) against the fp64 oracle: the edges
of its 32-row blocks and 64-key tiles, every GQA group, key ranges merged
afterwards, rows without keys, and values that are not finite outside a row's
keys.  Tolerances as for every attention output (tests/gpu_util.py)."""
import numpy as np
import pytest

import oracle as orc
from paper_2606_06467_amd import inputs
from tests import gpu_util as U
from tests.test_gpu_dense import _case, _full_sets

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,n,ps", [(17, 4161, 0), (32, 2113, 16), (33, 2048, 0), (97, 769, 64),
                                     (250, 321, 0), (288, 288, 64)])
@pytest.mark.parametrize("qh,kvh", [(4, 4), (4, 2), (32, 8), (10, 2), (16, 2)])
def test_tile_edges(nq, n, ps, qh, kvh):
    """Causal rows that end with their sequence; the second sequence is shorter
    than the block of rows (its first rows see nothing), the third is empty.  As often
    as it takes for the tiles to be chosen."""
    for times in (1, 2, 4, 8, 16):
        w = inputs.small_workload(batch=3 * times, lens=(n, nq // 2, 0) * times, n_q=nq, causal=True,
                                  q_pos0=(n - nq, nq // 2 - nq, -nq) * times, q_heads=qh,
                                  kv_heads=kvh, page_size=ps, n_layers=1, wid=81)
        if U.dense_in_tiles(w):
            break
    assert U.dense_in_tiles(w)
    _case(w, f"tiles {nq} rows {n} keys Hq={qh} Hkv={kvh} page={ps}")


@pytest.mark.parametrize("nq,n", [(16, 3000), (40, 5000)])
def test_not_causal_split_by_key_range(nq, n):
    """Few row blocks: the key range is split and merged; every row sees every key."""
    w = inputs.small_workload(batch=2, lens=(n, n // 3), n_q=nq, n_layers=1, wid=82)
    assert U.dense_in_tiles(w)
    _case(w, f"tiles {nq} rows {n} keys, split")


def test_large_logits():
    """Logits of hundreds: the running maximum moves far, in both directions."""
    w = inputs.small_workload(batch=1, lens=(1300,), n_q=40, causal=True, q_pos0=(1260,),
                              n_layers=1, wid=83)
    assert U.dense_in_tiles(w)
    x = inputs.make_inputs(w, layers=[0])
    k = inputs.f32_from_bf16_bits(x["k_cache"])
    k *= np.linspace(-30, 30, 1300)[None, :, None, None]
    x["k_cache"] = inputs.bf16_bits_from_f32(k)
    _run_and_compare(w, x)


def _run_and_compare(w, x, mask_rows=None):
    import torch
    from paper_2606_06467_amd import binding as B
    d = U.to_dev(x)
    q = B.bf16_from_bits(x["q_layers"][0])
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full(q.shape[:-1], float("nan"), device="cuda")
    sh = U.shape_of(w)
    B.clsa_dense_attn(sh, q, d["k_cache"], d["v_cache"], d["page_table"], d["seq_lens"],
                      d["q_pos"], out, lse, B.workspace(sh, B.CLSA_OP_DENSE))
    torch.cuda.synchronize()
    osh, idx, n = _full_sets(w, x["seq_lens"], x["q_pos"])
    ref_o, ref_l = orc.sparse_attn(osh, x["q_layers"][0], x["k_cache"], x["v_cache"], idx, n,
                                   x["page_table"])
    o = B.bits_from_bf16(out)
    ls = lse.cpu().numpy().astype(np.float64)
    U.compare_attn(o, ls, ref_o, ref_l, mask_rows=mask_rows)
    return inputs.f32_from_bf16_bits(o), ls


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("which", ["k_cache", "v_cache"])
def test_values_not_finite_stay_with_the_rows_that_see_them(which, bad):
    """A token whose key or value is not finite changes no row before it."""
    w = inputs.small_workload(batch=1, lens=(1500,), n_q=70, causal=True, q_pos0=(1430,),
                              n_layers=1, wid=84)
    assert U.dense_in_tiles(w)
    x = inputs.make_inputs(w, layers=[0])
    x["k_cache"] = x["k_cache"].copy()
    x["v_cache"] = x["v_cache"].copy()
    x[which][0, 1450, :, 5] = inputs.bf16_bits_from_f32(np.float32([bad]))[0]
    before = np.zeros((1, 70), bool)
    before[0, :20] = True  # positions 1430 .. 1449
    o, ls = _run_and_compare(w, x, mask_rows=before)
    if which == "v_cache":  # the others carry it, in that dimension alone
        assert not np.isfinite(o[0, 20:, :, 5]).any()
        assert np.isfinite(np.delete(o[0, 20:], 5, axis=-1)).all()
        assert np.isfinite(ls).all()


@pytest.mark.parametrize("qh,kvh,ps", [(32, 8, 0), (20, 4, 64), (16, 8, 16), (64, 8, 64)])
@pytest.mark.parametrize("top_k", [300, 950])
def test_step_with_selection_masks(qh, kvh, ps, top_k):
    """Chunked prefill over few keys: every layer attends in tiles with a
    selection mask.  Rows that select everything (words of ones, and a word cut
    at the row's own position), a part, or nothing (rows before a shorter
    sequence's first token)."""
    from tests.test_gpu_decode_step import _check_step
    w = inputs.small_workload(batch=2, lens=(1000, 610), n_q=1000, causal=True,
                              q_pos0=(0, 610 - 1000), q_heads=qh, kv_heads=kvh, page_size=ps,
                              top_k=top_k, n_layers=2, wid=85)
    assert U.step_in_tiles(w)
    _check_step(w, inputs.make_inputs(w), [1], f"masked tiles k={top_k} Hq={qh} Hkv={kvh}")


@pytest.mark.parametrize("ps", [0, 64])
def test_step_selection_excludes_values_not_finite(ps):
    """An infinite value of one token reaches the rows that select it, no other."""
    from tests.test_gpu_decode_step import _gpu_step
    w = inputs.small_workload(batch=1, lens=(960,), n_q=960, causal=True, q_pos0=(0,), top_k=400,
                              page_size=ps, n_layers=1, wid=86)
    assert U.step_in_tiles(w)
    x = inputs.make_inputs(w)
    at = (int(x["page_table"][0, 500 // ps]), 500 % ps) if ps else (0, 500)
    x["v_cache"][at][:, 7] = inputs.bf16_bits_from_f32(np.float32([np.inf]))[0]
    out, lse, idx, ns = _gpu_step(w, x, 1)
    has = (idx[0] == 500).any(-1)
    assert has[500:].any() and not has.all() and not has[500:].all()
    o = inputs.f32_from_bf16_bits(out[0, 0])
    assert np.isfinite(o[~has]).all() and np.isfinite(lse).all()
    assert np.isposinf(o[has][:, :, 7]).all()
    ro, rl = orc.sparse_attn(orc.shape_of(w), x["q_layers"][0], x["k_cache"], x["v_cache"], idx,
                             ns, x["page_table"])
    U.compare_attn(out[0], lse[0], ro, rl, mask_rows=~has[None])


@pytest.mark.parametrize("scale", [0.0, -0.09])
def test_scale_not_positive(scale):
    """Dense rows in tiles and in the per-row kernel, and a step with selection masks."""
    import torch
    from paper_2606_06467_amd import binding as B
    for nq, n, top_k in ((70, 1900, 64), (5, 1900, 64), (1000, 1000, 600)):
        w = inputs.small_workload(batch=1, lens=(n,), n_q=nq, causal=True, q_pos0=(n - nq,),
                                  top_k=top_k, n_layers=1, wid=89)
        x = inputs.make_inputs(w)
        sh = U.shape_of(w)
        sh.softmax_scale = scale
        d = U.to_dev(x)
        q = d["q_layers"]
        out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full(q.shape[:-1], float("nan"), device="cuda")
        if nq < 1000:
            B.clsa_dense_attn(sh, q[0], d["k_cache"], d["v_cache"], None, d["seq_lens"],
                              d["q_pos"], out[0], lse[0], B.workspace(sh, B.CLSA_OP_DENSE))
            osh, idx, ns = _full_sets(w, x["seq_lens"], x["q_pos"])
        else:
            idx = torch.empty((1, nq, top_k), dtype=torch.int32, device="cuda")
            ns = torch.empty((1, nq), dtype=torch.int32, device="cuda")
            B.clsa_decode_step(sh, d["q_idx"], d["k_idx"], d["k_cache"], d["v_cache"], None,
                               d["seq_lens"], d["q_pos"], q, out, lse, idx, ns,
                               B.workspace(sh, B.CLSA_OP_DECODE, 1))
            osh, idx, ns = orc.shape_of(w), idx.cpu().numpy(), ns.cpu().numpy()
        torch.cuda.synchronize()
        osh.softmax_scale = scale
        ref_o, ref_l = orc.sparse_attn(osh, x["q_layers"][0], x["k_cache"], x["v_cache"], idx, ns)
        U.compare_attn(B.bits_from_bf16(out[0]), lse[0].cpu().numpy().astype(np.float64), ref_o,
                       ref_l, what=f"scale {scale}, {nq} rows")


@pytest.mark.parametrize("top_k", [300, 700])
def test_masked_step_grouped_and_replayed(top_k):
    """The mask lies in the scores of its index set: sets made afresh for every layer
    give the shared step's results, and so does every replay of a captured step."""
    import torch
    from paper_2606_06467_amd import binding as B
    w = inputs.small_workload(batch=2, lens=(1000, 410), n_q=600, causal=True,
                              q_pos0=(400, 410 - 600), top_k=top_k, n_layers=3, wid=93)
    assert U.step_in_tiles(w)
    d = U.to_dev(inputs.make_inputs(w))
    sh, q = U.shape_of(w), d["q_layers"]
    ws = B.workspace(sh, B.CLSA_OP_DECODE, 3)

    def outputs(sets):
        return (torch.empty(q.shape, dtype=torch.bfloat16, device="cuda"),
                torch.empty(q.shape[:-1], device="cuda"),
                torch.empty((sets, 2, 600, top_k), dtype=torch.int32, device="cuda"),
                torch.empty((sets, 2, 600), dtype=torch.int32, device="cuda"))

    def shared(o):
        B.clsa_decode_step(sh, d["q_idx"], d["k_idx"], d["k_cache"], d["v_cache"], None,
                           d["seq_lens"], d["q_pos"], q, *o, ws)

    def same(a, b):
        return all(torch.equal(x.view(torch.int16) if x.dtype == torch.bfloat16 else x,
                               y.view(torch.int16) if y.dtype == torch.bfloat16 else y)
                   for x, y in zip(a, b))

    ref = outputs(1)
    shared(ref)
    got = outputs(3)
    B.clsa_decode_step_grouped(sh, d["q_idx"], 0, d["k_idx"], 0, d["k_cache"], d["v_cache"], None,
                               d["seq_lens"], d["q_pos"], 1, q, *got, ws)
    torch.cuda.synchronize()
    assert same(got[:2], ref[:2])
    assert all(torch.equal(got[2][s], ref[2][0]) and torch.equal(got[3][s], ref[3][0]) for s in range(3))
    rep = outputs(1)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        shared(rep)
    for _ in range(3):
        for t in rep:
            t.fill_(0)
        g.replay()
        torch.cuda.synchronize()
        assert same(rep, ref)
        shared(outputs(1))  # eager work between replays
        torch.cuda.synchronize()
