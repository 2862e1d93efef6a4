"""A small fp32 model's step as one kernel (k_step_small) against the separate
kernels, bit for bit (same MFMA in the same order of k, same attention order),
on every output and intermediate: one and several rows per block, a last block
with fewer rows, widths off the 32-column tiles and 64-unit packing, a last k
group of 4, the largest widths, ids out of range, aliased states, a one-
sentence source, states gathered from a pool.  Where some queries are beyond
the keys' factors the separate kernels choose the formula per tile and this
one per row, so there the two agree to rounding only.  Both are held to the
oracle elsewhere (tiny and ragged cases)."""
import numpy as np
import pytest

from paper_1605_04809_amd.workloads import Config, random_annotations, unit_gain

pytestmark = pytest.mark.gpu

BASE = Config("small", V=300, V_src=40, E=32, H=64, A=64, B=8, S=3, len_lo=1, len_hi=21, Tpad=21,
              sigma_w=1.0, sigma_emb=1.0, seed=101)


@pytest.fixture(scope="module")
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_cases
    return gpu_cases


def both(fn):
    from paper_1605_04809_amd import binding as nb
    prev = nb.debug_small_step(0)
    try:
        apart = fn()
    finally:
        nb.debug_small_step(prev)
    return fn(), apart


@pytest.mark.parametrize("kw", [
    dict(), dict(B=1, S=1), dict(B=300), dict(B=601, H=100, E=52, A=76), dict(B=1025, H=128, E=256, A=256),
    dict(B=2048, H=36, E=104, A=100, S=1), dict(B=17, H=128, E=4, A=4, S=7, Tpad=130, len_hi=130),
    dict(B=70, H=4, E=12, A=132)], ids=lambda kw: "_".join(f"{k}{v}" for k, v in kw.items()) or "base")
def test_one_kernel_equals_the_separate_ones(gpu, kw):
    wl = unit_gain(BASE.replace(**kw))
    wl.y_prev[::5] = -1
    g = gpu.GpuRun(wl)
    y, s = wl.y_prev.copy(), wl.sent_id.copy()
    if len(y) > 20 and wl.cfg.S > 1:   # flagged rows: everything but log p is still defined
        y[3], s[11], s[12] = wl.cfg.V, -1, wl.cfg.S
    one, apart = both(lambda: g.step(wl.s_prev, y, s, wl.req))
    for k in apart:
        np.testing.assert_array_equal(one[k], apart[k], err_msg=k)
    alias = g.step(wl.s_prev, y, s, wl.req, debug=False, alias=True)
    np.testing.assert_array_equal(alias["s_new"], apart["s_new"])
    g.close()


def test_longest_sentences(gpu):
    """Eight rows a block with the scores of 1,024 positions: 82 KB of LDS."""
    wl = unit_gain(BASE.replace(B=1100, H=128, E=256, A=256, S=2, Tpad=1024, len_hi=1024))
    wl.src_len[0] = 1024
    g = gpu.GpuRun(wl, ctx_f32=random_annotations(wl.cfg, seed=104))
    one, apart = both(lambda: g.step(wl.s_prev, wl.y_prev, wl.sent_id, wl.req))
    for k in apart:
        np.testing.assert_array_equal(one[k], apart[k], err_msg=k)
    g.close()


@pytest.mark.parametrize("shift", [1, 37, -1, -37])
@pytest.mark.parametrize("B", [300, 2000])
def test_new_states_over_a_part_of_the_old_ones(gpu, B, shift):
    """New states shifted against the old ones in one buffer: the separate
    kernels have read every old state before they write a new one."""
    import torch
    from paper_1605_04809_amd import binding as nb
    wl = unit_gain(BASE.replace(B=B))
    g = gpu.GpuRun(wl)
    want = g.step(wl.s_prev, wl.y_prev, wl.sent_id, wl.req)
    H, pad = wl.cfg.H, 40
    buf = torch.zeros((B + 2 * pad, H), device="cuda")
    old, new = buf[pad:pad + B], buf[pad + shift:pad + shift + B]
    old.copy_(gpu.cuda(wl.s_prev))
    lp = torch.empty(B, device="cuda")
    nb.nmt_score_batch(g.model, g.src, old, gpu.cuda(wl.y_prev), gpu.cuda(wl.sent_id), gpu.cuda(wl.req), lp, new)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(new.cpu().numpy(), want["s_new"])
    np.testing.assert_array_equal(lp.cpu().numpy(), want["logp"])
    g.close()


def test_keys_beyond_the_factors_range(gpu):
    cfg = BASE.replace(B=40, A=128)
    wl = unit_gain(cfg, key_scale=40.0, query_scale=60.0)
    ctx = random_annotations(cfg, seed=102)
    g, o = gpu.GpuRun(wl, ctx_f32=ctx), gpu.OracleRun(wl, ctx_f32=ctx)
    args = (wl.s_prev, wl.y_prev, wl.sent_id, wl.req)
    got, ref = g.step(*args), o.step(*args)
    assert gpu.max_abs(got["alpha"], ref["alpha"]) <= 1e-4
    g.close()


@pytest.mark.parametrize("B", [40, 520, 1100])
def test_some_queries_beyond_the_factors_range(gpu, B):
    """A third of the rows have a query beyond the keys' factors: rows of one
    tile may take another formula than alone, each within a few 1e-7."""
    cfg = BASE.replace(B=B)
    wl = unit_gain(cfg, key_scale=40.0, query_scale=16.0)
    g = gpu.GpuRun(wl, ctx_f32=random_annotations(cfg, seed=103))
    one, apart = both(lambda: g.step(wl.s_prev, wl.y_prev, wl.sent_id, wl.req))
    for k in apart:
        assert gpu.max_abs(one[k], apart[k]) <= (1e-4 if k.startswith("log") else 1e-5), k
    g.close()


def test_states_from_a_pool(gpu):
    import torch
    from paper_1605_04809_amd import binding as nb
    wl = unit_gain(BASE.replace(B=50))
    g = gpu.GpuRun(wl)
    row = np.random.default_rng(5).integers(-1, 51, size=90).astype(np.int32)   # both ends out of range
    y, s = np.resize(wl.y_prev, 90), np.resize(wl.sent_id, 90)
    off = np.arange(0, 181, 2, dtype=np.int32)
    req = np.resize(wl.req, 180)

    def run():
        lp, sn = torch.empty(180, device="cuda"), torch.empty((90, wl.cfg.H), device="cuda")
        nb.nmt_score_forest_step(g.model, g.src, gpu.cuda(wl.s_prev), gpu.cuda(row), gpu.cuda(y), gpu.cuda(s),
                                 gpu.cuda(off), gpu.cuda(req), lp, sn)
        torch.cuda.synchronize()
        return lp.cpu().numpy(), sn.cpu().numpy()
    one, apart = both(run)
    np.testing.assert_array_equal(one[0], apart[0])
    np.testing.assert_array_equal(one[1], apart[1])
    g.close()
