"""The key-tile attention kernel run on the CPU, wave by wave: its results must not
depend on which wave of a workgroup runs first.  Tolerances as on the GPU."""
import ctypes

import numpy as np
import pytest

import oracle as orc
from paper_2606_06467_amd import inputs
from tests import emu_util
from tests import gpu_util as U

_WRAPPERS = """
extern "C" void emu_tile(int batch, int n_q, int max_len, int page_shift, int max_pages, int causal,
                         int q_heads, int kv_heads, float scale, const void *q, const void *k,
                         const void *v, const int32_t *pt, const int32_t *sl, const int32_t *qp,
                         const uint32_t *mask, int splits, int span, void *out, float *lse,
                         float *po, float *pml, int order) {
    clsa::Geometry g{batch, n_q, batch * n_q, max_len, page_shift, max_pages, 1, causal,
                     q_heads, kv_heads, q_heads / kv_heads, scale};
    emu::wave_order = order;
    emu::wave_ops = 0;
    clsa::launch_tile_attn(g, q, k, v, pt, sl, qp, mask, splits, span, out, lse, po, pml, nullptr);
}
extern "C" void emu_mask(int batch, int n_q, int max_len, int top_k, const int32_t *idx,
                         const int32_t *n_sel, const int32_t *sl, uint32_t *mask) {
    clsa::Geometry g{batch, n_q, batch * n_q, max_len, -1, 0, top_k, 1, 8, 8, 1, 0.1f};
    clsa::launch_attn_mask(g, idx, n_sel, sl, mask, nullptr);
}
extern "C" int emu_masked(int batch, int n_q, int max_len, int top_k, int q_heads, int kv_heads,
                           int splits) {
    clsa::Geometry g{batch, n_q, batch * n_q, max_len, -1, 0, top_k, 1, q_heads, kv_heads,
                     q_heads / kv_heads, 0.1f};
    return clsa::tile_attn_masked(g, splits);
}
extern "C" int emu_dense(int batch, int n_q, int max_len, int causal, int q_heads, int kv_heads, int splits) {
    clsa::Geometry g{batch, n_q, batch * n_q, max_len, -1, 0, 1, causal, q_heads, kv_heads,
                     q_heads / kv_heads, 0.1f};
    return clsa::tile_attn_dense(g, splits);
}
extern "C" long emu_wave_ops() { return emu::wave_ops; }
"""


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    return emu_util.build(str(tmp_path_factory.mktemp("emu")), "tile_attn.hip", _WRAPPERS)


def _p(a):
    return None if a is None else a.ctypes.data_as(ctypes.c_void_p)


def _run(emu, w, x, order, mask=None, scale=None):
    """(out bits, lse) of one layer, one key range."""
    q = np.ascontiguousarray(x["q_layers"][0])
    out = np.zeros(q.shape, np.uint16)
    lse = np.zeros(q.shape[:-1], np.float32)
    emu.emu_tile(w.batch, w.n_q, w.max_len, w.page_size.bit_length() - 1, w.max_pages,
                 int(w.causal), w.q_heads, w.kv_heads,
                 ctypes.c_float(w.softmax_scale if scale is None else scale), _p(q),
                 _p(x["k_cache"]), _p(x["v_cache"]), _p(x["page_table"]), _p(x["seq_lens"]),
                 _p(x["q_pos"]), _p(mask), 1, -(-w.max_len // 64) * 64, _p(out), _p(lse), None,
                 None, order)
    return out, lse


def _sets(w, x):
    sh = orc.shape_of(w, top_k=w.max_len)
    n = orc.valid_lens(sh, x["seq_lens"], x["q_pos"]).astype(np.int32)
    j = np.arange(w.max_len, dtype=np.int32)
    return sh, np.where(j < n[..., None], j, -1), n


def _compare(w, x, out, lse, sets, what, rows=None, scale=None):
    sh, idx, n = sets
    if scale is not None:
        sh.softmax_scale = scale
    ref_o, ref_l = orc.sparse_attn(sh, x["q_layers"][0], x["k_cache"], x["v_cache"], idx, n,
                                   x["page_table"])
    U.compare_attn(out, lse.astype(np.float64), ref_o, ref_l, mask_rows=rows, what=what)


def _mask(idx, n, max_len):
    """The selection words of the kernel: two per 64 keys and row."""
    bits = np.zeros(idx.shape[:2] + (-(-max_len // 64) * 64,), np.uint8)
    for r in np.ndindex(n.shape):
        bits[r][idx[r][:n[r]]] = 1
    return np.ascontiguousarray(np.packbits(bits, axis=-1, bitorder="little").view(np.uint32))


def _thirds(idx, n):
    """A third of every row's keys."""
    g = np.random.default_rng(88)
    idx, n = np.full_like(idx, -1), n // 3
    for r in np.ndindex(n.shape):
        idx[r][:n[r]] = np.sort(g.choice(3 * n[r], n[r], replace=False))
    return idx, n


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("page", [0, 16])
def test_wave_order_dense(emu, order, page):
    """Three key tiles, two (row block, head) pairs per KV head: a wave far ahead of
    the others stores tile after tile while they still read."""
    w = inputs.small_workload(batch=1, lens=(170,), n_q=40, causal=True, q_pos0=(130,), q_heads=4,
                              kv_heads=1, page_size=page, n_layers=1, wid=87)
    x = inputs.make_inputs(w)
    out, lse = _run(emu, w, x, order)
    _compare(w, x, out, lse, _sets(w, x), f"waves in order {order}, page {page}")


@pytest.mark.parametrize("order", [0, 1])
def test_wave_order_masked(emu, order):
    w = inputs.small_workload(batch=1, lens=(150,), n_q=36, causal=True, q_pos0=(114,), q_heads=4,
                              kv_heads=1, n_layers=1, wid=88)
    x = inputs.make_inputs(w)
    sh, idx, n = _sets(w, x)
    idx, n = _thirds(idx, n)
    out, lse = _run(emu, w, x, order, mask=_mask(idx, n, w.max_len))
    _compare(w, x, out, lse, (sh, idx, n), f"masked, waves in order {order}")


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("scale", [0.0, -0.09])
def test_scale_not_positive(emu, scale, masked):
    """A scale of zero weighs every key alike, a negative one turns the order round; both
    take the same work as a positive one."""
    w = inputs.small_workload(batch=1, lens=(150,), n_q=36, causal=True, q_pos0=(114,), q_heads=4,
                              kv_heads=1, n_layers=1, wid=88)
    x = inputs.make_inputs(w)
    sh, idx, n = _sets(w, x)
    mask = None
    if masked:
        idx, n = _thirds(idx, n)
        mask = _mask(idx, n, w.max_len)
    _run(emu, w, x, 0, mask=mask)
    usual = emu.emu_wave_ops()
    out, lse = _run(emu, w, x, 0, mask=mask, scale=scale)
    _compare(w, x, out, lse, (sh, idx, n), f"scale {scale}", scale=scale)
    assert emu.emu_wave_ops() <= 1.1 * usual


def _one_hot(n, z):
    """A row of 4 heads whose logit of key j is z[j] in log2 units, up to the rounding of
    the keys to bf16; the values of keys with z < 0 or the last key are random, others 0."""
    w = inputs.small_workload(batch=1, lens=(n,), n_q=33, q_heads=4, kv_heads=1, n_layers=1, wid=90)
    x = inputs.make_inputs(w)
    q = np.zeros((1, 1, 33, 4, 128), np.float32)
    q[..., 0] = 8.0
    k = np.zeros((1, n, 1, 128), np.float32)
    k[0, :, 0, 0] = np.asarray(z) / (8.0 * w.softmax_scale * np.log2(np.e))
    x["q_layers"], x["k_cache"] = inputs.bf16_bits_from_f32(q), inputs.bf16_bits_from_f32(k)
    return w, x


@pytest.mark.parametrize("level", [7.4, 1.3, -2.3, -5.7])
def test_largest_weight_of_a_tile_is_exact(emu, level):
    """Tile 1 holds one key that counts, above or below the keys of tile 0 (whose values
    are zero): its weight must not be rounded, or every output is off by the same part.
    The outputs' own rounding averages out over 128 dimensions: 0.0017 / 11."""
    z = np.full(128, -60.0)
    z[:64] = 0.0
    z[100] = level
    w, x = _one_hot(128, z)
    x["v_cache"] = x["v_cache"].copy()
    x["v_cache"][0, np.arange(128) != 100] = 0
    out, lse = _run(emu, w, x, 0)
    sh, idx, n = _sets(w, x)
    ref, ref_l = orc.sparse_attn(sh, x["q_layers"][0], x["k_cache"], x["v_cache"], idx, n)
    o = inputs.f32_from_bf16_bits(out).astype(np.float64)
    v = inputs.f32_from_bf16_bits(x["v_cache"])[0, 100, 0].astype(np.float64)
    part = ref[0, 0, 0, 0] / v[0]                       # weight of key 100 in 64 bits
    got = (o[0, 0, 0] * v).sum() / (v * v).sum()
    assert abs(got / part - 1) < 6e-4, (got, part)
    assert np.abs(lse - ref_l).max() < 1e-5


def test_short_rows_are_as_exact_as_their_outputs(emu):
    """Rows of at most 64 keys: the weights' own rounding does not show beside that of the
    bf16 outputs (2-norm 0.00166; with weights of 8 bits 0.0020)."""
    w = inputs.small_workload(batch=1, lens=(64,), n_q=64, causal=True, q_pos0=(0,), q_heads=4,
                              kv_heads=1, n_layers=1, wid=91)
    x = inputs.make_inputs(w)
    out, _ = _run(emu, w, x, 0)
    sh, idx, n = _sets(w, x)
    ref, _ = orc.sparse_attn(sh, x["q_layers"][0], x["k_cache"], x["v_cache"], idx, n)
    d = inputs.f32_from_bf16_bits(out).astype(np.float64) - ref
    rel = float(np.sqrt((d * d).sum() / (ref * ref).sum()))
    assert rel < 0.00175, rel


def _float_model(w, x, idx, n):
    """Attention with every value as it is: out, in float64 (infinities and NaN included)."""
    q, k, v = (inputs.f32_from_bf16_bits(x[i]).astype(np.float64) for i in ("q_layers", "k_cache", "v_cache"))
    if w.page_size:
        k, v = (c[x["page_table"][0]].reshape((-1,) + c.shape[2:])[None] for c in (k, v))
    out = np.zeros(q[0].shape)
    with np.errstate(all="ignore"):
        for t in range(w.n_q):
            s = idx[0, t, :n[0, t]]
            z = q[0, 0, t] @ k[0, s, 0].T * w.softmax_scale
            e = np.exp(z - z.max(-1, keepdims=True))
            out[0, t] = (e[:, :, None] * v[0, s, 0][None]).sum(1) / e.sum(-1, keepdims=True)
    return out


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 3.3e38])
def test_values_not_finite(emu, bad, masked, page):
    """One value of three keys (the first of the sequence, one that some rows see, the
    last) is not finite, or so large that sums of a lagging base overflow: the outputs
    are those of every value as it is, for at most a few times the work."""
    w = inputs.small_workload(batch=1, lens=(176,), n_q=70, causal=True, q_pos0=(106,), q_heads=4,
                              kv_heads=1, page_size=page, n_layers=1, wid=92)
    x = inputs.make_inputs(w)
    sh, idx, n = _sets(w, x)
    mask = None
    if masked:
        idx, n = _thirds(idx, n)
        mask = _mask(idx, n, w.max_len)
    _run(emu, w, x, 0, mask=mask)
    usual = emu.emu_wave_ops()
    x["v_cache"] = x["v_cache"].copy()
    for j, d in ((0, 3), (130, 77), (175, 127)):
        at = (x["page_table"][0, j // page], j % page) if page else (0, j)
        x["v_cache"][at][0, d] = inputs.bf16_bits_from_f32(np.float32([bad]))[0]
    out, lse = _run(emu, w, x, 0, mask=mask)
    assert emu.emu_wave_ops() <= 4 * usual
    o, ref = inputs.f32_from_bf16_bits(out).astype(np.float64), _float_model(w, x, idx, n)
    fin = np.isfinite(ref)
    assert np.array_equal(np.isnan(o), np.isnan(ref))
    assert np.array_equal(o[~fin & ~np.isnan(ref)], ref[~fin & ~np.isnan(ref)])
    assert np.all(np.abs(o[fin] - ref[fin]) <= 0.02 * np.maximum(1, np.abs(ref[fin])))
    _, ref_l = orc.sparse_attn(sh, x["q_layers"][0], x["k_cache"], x["v_cache"], idx, n,
                               x["page_table"])
    assert np.abs(lse - ref_l).max() < 1e-4


@pytest.mark.parametrize("batch,n_q,n,k,qh,kvh,splits,tiles", [
    (2, 137, 137, 512, 32, 8, 1, False), (2, 122, 122, 2048, 64, 8, 1, False),  # the mask's launch
    (2, 138, 138, 1024, 64, 8, 1, True), (4, 125, 125, 1720, 20, 4, 4, True),   # ... and a merge
    (1, 287, 287, 1024, 32, 8, 2, True), (4, 167, 167, 1024, 20, 4, 2, True),
    (3, 473, 1674, 512, 32, 8, 2, True), (2, 2054, 5500, 512, 16, 8, 2, True),
    (1, 179, 1002, 512, 32, 8, 2, False), (1, 4096, 32768, 2048, 32, 8, 8, False),  # few of the keys
    (1, 15, 15, 512, 32, 8, 1, False)])
def test_masked_tiles_where_they_measured_faster(emu, batch, n_q, n, k, qh, kvh, splits, tiles):
    assert bool(emu.emu_masked(batch, n_q, n, k, qh, kvh, splits)) == tiles


@pytest.mark.parametrize("batch,n_q,n,qh,kvh,splits,tiles", [
    (4, 32, 600, 64, 8, 1, False), (3, 64, 300, 64, 8, 1, False), (1, 150, 600, 64, 8, 1, False),
    (1, 64, 1000, 64, 8, 2, False), (4, 64, 600, 20, 4, 1, False), (1, 500, 600, 20, 4, 1, False),
    (1, 1000, 1000, 20, 4, 3, True), (3, 500, 600, 64, 8, 8, True), (1, 500, 1000, 64, 8, 1, True),
    (1, 500, 600, 8, 8, 1, True), (8, 16, 4096, 32, 8, 1, True), (1, 16, 32768, 32, 8, 8, True),
    (1, 8192, 8192, 20, 4, 8, True), (1, 15, 65536, 32, 8, 9, False), (1, 64, 600, 32, 8, 2, False)])
def test_dense_tiles_where_they_measured_faster(emu, batch, n_q, n, qh, kvh, splits, tiles):
    assert bool(emu.emu_dense(batch, n_q, n, 1, qh, kvh, splits)) == tiles


def test_mask_of_long_rows(emu):
    """Rows of more than 65536 keys take several passes: runs of entries that cross a
    pass, entries in one pass alone, none; nothing is written past a sequence's words."""
    max_len, k = 140000, 3000
    g = np.random.default_rng(5)
    lens = np.array([140000, 70001], np.int32)
    rows = [np.sort(g.choice(140000, 3000, replace=False)), np.arange(64000, 67000),
            np.sort(g.choice(70001, 700, replace=False)), np.arange(65530, 65545)[:0],
            np.arange(66000, 66100), np.array([0, 31, 32, 65535, 65536, 70000])]
    idx, n = np.full((2, 3, k), -1, np.int32), np.zeros((2, 3), np.int32)
    for r, s in zip(np.ndindex(2, 3), (rows[0], rows[1], rows[5], rows[2], rows[3], rows[4])):
        idx[r][:s.size], n[r] = s, s.size
    words = 2 * -(-max_len // 64)
    mask = np.full((2, 3, words), 0xabcdabcd, np.uint32)
    emu.emu_mask(2, 3, max_len, k, _p(idx), _p(n), _p(lens), _p(mask))
    ref = _mask(idx, n, max_len)
    used = 2 * -(-70001 // 64)
    assert np.array_equal(mask[0], ref[0]) and np.array_equal(mask[1, :, :used], ref[1, :, :used])
    assert (mask[1, :, used:] == 0xabcdabcd).all()
