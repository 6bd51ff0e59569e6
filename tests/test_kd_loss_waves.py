"""The distillation loss run on the CPU, wave by wave: the same results whichever wave
of a workgroup runs first, and nothing written outside the workspace that the library
asks for.  Bounds as on the GPU."""
import ctypes

import numpy as np
import pytest

import oracle as orc
from paper_2606_06467_amd import inputs
from tests import emu_util

_WRAPPERS = """
static clsa::Geometry geometry(int batch, int n_q, int max_len, int page_shift, int max_pages, int causal) {
    return clsa::Geometry{batch, n_q, batch * n_q, max_len, page_shift, max_pages, 1, causal, 8, 8, 1, 1.0f};
}
extern "C" void emu_kd(int batch, int n_q, int max_len, int page_shift, int max_pages, int causal,
                       const float *abar, const void *q, const void *k, const int32_t *pt,
                       const int32_t *sl, const int32_t *qp, float *loss, float *dq, float *dk,
                       float *ws, int order) {
    emu::wave_order = order;
    emu::wave_ops = 0;
    clsa::launch_kd_loss(geometry(batch, n_q, max_len, page_shift, max_pages, causal), abar, q, k,
                         pt, sl, qp, loss, dq, dk, ws, nullptr);
}
extern "C" long emu_wave_ops() { return emu::wave_ops; }
extern "C" size_t emu_kd_carved(int batch, int n_q, int max_len) {
    return clsa::kd_loss_plan(geometry(batch, n_q, max_len, -1, 0, 0)).floats;
}
extern "C" size_t emu_kd_ws(int batch, int n_q, int max_len) {
    return clsa::kd_loss_ws_floats(geometry(batch, n_q, max_len, -1, 0, 0));
}
"""


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    lib = emu_util.build(str(tmp_path_factory.mktemp("emu")), "kd_loss.hip", _WRAPPERS)
    lib.emu_kd_ws.restype = lib.emu_kd_carved.restype = ctypes.c_size_t
    return lib


def _p(a):
    return None if a is None else a.ctypes.data_as(ctypes.c_void_p)


_GUARD = 4096  # floats on either side of the workspace


def _run(emu, w, x, abar, order=0):
    """(loss, dq, dk); the workspace lies between guards that must stay as they are."""
    n_ws = -(-emu.emu_kd_ws(w.batch, w.n_q, w.max_len) // 64) * 64
    buf = np.full(n_ws + 2 * _GUARD + 64, 7.25, np.float32)
    first = _GUARD + (-(buf.ctypes.data // 4 + _GUARD)) % 64  # 256-byte aligned
    ws = buf[first:first + n_ws]
    loss = np.zeros(1, np.float32)
    dq = np.zeros(x["q_idx"].shape, np.float32)
    dk = np.zeros(x["k_idx"].shape, np.float32)
    emu.emu_kd(w.batch, w.n_q, w.max_len, w.page_size.bit_length() - 1, w.max_pages,
               int(w.causal), _p(abar), _p(x["q_idx"]), _p(x["k_idx"]), _p(x["page_table"]),
               _p(x["seq_lens"]), _p(x["q_pos"]), _p(loss), _p(dq), _p(dk), _p(ws), order)
    assert (buf[:first] == 7.25).all() and (buf[first + n_ws:] == 7.25).all()
    return float(loss[0]), dq, dk


def _inputs(w):
    """Index tensors, and a peaked random distribution over each row's keys."""
    x = inputs.make_inputs(w, index_only=True)
    nv = orc.valid_lens(orc.shape_of(w), x["seq_lens"], x["q_pos"])
    z = np.random.default_rng(w.wid).standard_normal((w.batch, w.n_q, w.max_len)) * 2
    e = np.exp(z) * (np.arange(w.max_len) < nv[..., None])
    return x, np.ascontiguousarray(e / np.maximum(e.sum(-1, keepdims=True), 1e-300), np.float32)


def _compare(w, x, abar, got):
    loss, dq, dk = got
    r_loss, r_q, r_k = orc.kd_loss(orc.shape_of(w), abar, x["q_idx"], x["k_idx"], x["seq_lens"],
                                   x["q_pos"], x["page_table"])
    assert abs(loss - r_loss) <= 1e-5 * abs(r_loss) + 1e-7
    for g, r in ((dq, r_q), (dk, r_k)):
        ok = ~np.isnan(r)
        assert np.abs(g[ok] - r[ok]).max() <= 1e-5 * np.abs(r[ok]).max() + 1e-7


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("page", [0, 16])
def test_wave_order(emu, order, page):
    w = inputs.small_workload(batch=2, lens=(300, 70), n_q=150, causal=True, q_pos0=(150, -80),
                              page_size=page, n_layers=1, q_heads=8, kv_heads=8, wid=103)
    x, abar = _inputs(w)
    _compare(w, x, abar, _run(emu, w, x, abar, order))


def test_more_rows_than_a_tile_list(emu):
    """More than 16384 rows of one sequence take two ranges of rows however small the
    workspace is."""
    w = inputs.small_workload(batch=1, lens=(1,), n_q=16385, n_layers=1, q_heads=8, kv_heads=8,
                              wid=104)
    x, abar = _inputs(w)
    _compare(w, x, abar, _run(emu, w, x, abar))


def test_carved_within_the_workspace(emu):
    """Every batch, row count (around the multiples of a tile, a block and a list of
    tiles) and small to large capacity: what a call lays out fits what it asks for."""
    near = [m + d for m in (64, 128, 512, 2048, 16384, 32768, 49152, 1 << 20) for d in (-1, 0, 1, 70)]
    for batch in (1, 2, 3, 7):
        for n_q in [1, 2, 31, 33] + near:
            for max_len in (1, 2, 3, 5, 16, 63, 64, 65, 127, 129, 257, 258, 300, 513, 514, 515,
                            700, 1100, 4096, 33000, 262144):
                have, need = emu.emu_kd_ws(batch, n_q, max_len), emu.emu_kd_carved(batch, n_q, max_len)
                assert need <= have, (batch, n_q, max_len, need, have)


def _float_model(w, x, abar):
    """dq and dk in float64 from the pairs that count alone, every value as it is."""
    q, k = (inputs.f32_from_bf16_bits(x[i]).astype(np.float64).reshape(-1, 256) for i in ("q_idx", "k_idx"))
    if w.page_size:
        row = (x["page_table"][0][:, None] * w.page_size + np.arange(w.page_size)).ravel()
        k = k[row]
    n = orc.valid_lens(orc.shape_of(w), x["seq_lens"], x["q_pos"])[0]
    dq, dk = np.zeros(q.shape), np.zeros(k.shape)
    with np.errstate(all="ignore"):
        for t in range(w.n_q):
            z = q[t] @ k[:n[t]].T
            p = np.exp(z - z.max(initial=-np.inf))
            d = (p / p.sum() - abar[0, t, :n[t]]) / max(1, int((n > 0).sum()))
            dq[t] = (d[:, None] * k[:n[t]]).sum(0)
            dk[:n[t]] += d[:, None] * q[t]
    if w.page_size:
        out = np.zeros(dk.shape)
        out[row] = dk
        dk = out
    return dq.reshape(x["q_idx"].shape), dk.reshape(x["k_idx"].shape)


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("side,bad", [("q_idx", np.inf), ("q_idx", np.nan), ("k_idx", np.inf),
                                      ("k_idx", np.nan), ("k_idx", -np.inf)])
def test_values_not_finite(emu, side, bad, page):
    """An index vector that is not finite reaches the gradients of the pairs it is in,
    for at most a few times the work."""
    w = inputs.small_workload(batch=1, lens=(144,), n_q=150, causal=True, q_pos0=(-6,), n_layers=1,
                              page_size=page, q_heads=8, kv_heads=8, wid=105)
    x, abar = _inputs(w)
    _run(emu, w, x, abar)
    usual = emu.emu_wave_ops()
    x[side] = x[side].copy()
    at = 70 if side == "q_idx" or not page else int(x["page_table"][0, 70 // page]) * page + 70 % page
    x[side].reshape(-1, 256)[at, [3, 200]] = inputs.bf16_bits_from_f32(np.float32([bad]))[0]
    _, dq, dk = _run(emu, w, x, abar)
    assert emu.emu_wave_ops() <= 4 * usual
    for got, ref in zip((dq, dk), _float_model(w, x, abar)):
        assert np.array_equal(np.isfinite(got), np.isfinite(ref))
        ok = np.isfinite(ref)
        assert np.abs(got[ok] - ref[ok]).max(initial=0) <= 1e-5 * np.abs(ref[ok]).max(initial=0) + 1e-7


def test_row_term_of_equal_parts(emu):
    """1000 equal terms a row, whose sum one after another in fp32 rounds the same way at
    every step (500 a lane: an error of 6e-6): sums of 32 lose 32 + 16 roundings at most."""
    w = inputs.small_workload(batch=1, lens=(1000,), n_q=1, n_layers=1, q_heads=8, kv_heads=8, wid=106)
    x, abar = _inputs(w)
    x["q_idx"] = np.zeros_like(x["q_idx"])
    worst = 0.0
    for p in np.float32([1.1171, 1.3701, 1.6117]):
        abar[:] = p
        loss, _, _ = _run(emu, w, x, abar)
        exact = 1000 * float(p) * (np.log(float(p)) + np.log(1000.0))
        worst = max(worst, abs(loss / exact - 1))
    assert worst < 50 * 2.0 ** -25, worst


def test_target_not_a_number(emu):
    """A target that is not a number has no term in the loss (only P > 0 has), and makes
    the gradients of its row and key NaN."""
    w = inputs.small_workload(batch=1, lens=(100,), n_q=3, n_layers=1, q_heads=8, kv_heads=8, wid=107)
    x, abar = _inputs(w)
    abar[0, 1, 70] = 0.0
    without, _, _ = _run(emu, w, x, abar)
    abar[0, 1, 70] = np.nan
    loss, dq, dk = _run(emu, w, x, abar)
    assert loss == without
    assert np.isnan(dq[0, 1]).all() and np.isfinite(dq[0, [0, 2]]).all()
    assert np.isnan(dk[0, 70]).all() and np.isfinite(np.delete(dk[0], 70, axis=0)).all()


def test_target_infinite(emu):
    """An infinite target makes the gradients of its row and key infinite, as one product
    of each value with Q - P does."""
    w = inputs.small_workload(batch=1, lens=(100,), n_q=40, n_layers=1, q_heads=8, kv_heads=8, wid=108)
    x, abar = _inputs(w)
    for bad in (np.inf, -np.inf):
        abar[0, 33, 70] = bad
        _, dq, dk = _run(emu, w, x, abar)
        for got, ref in zip((dq, dk), _float_model(w, x, abar)):
            assert np.array_equal(np.isnan(got), np.isnan(ref))
            hit = np.isinf(ref)
            assert hit.sum() >= 250 and np.array_equal(got[hit], ref[hit])
            ok = np.isfinite(ref)
            assert np.abs(got[ok] - ref[ok]).max() <= 1e-5 * np.abs(ref[ok]).max() + 1e-7
