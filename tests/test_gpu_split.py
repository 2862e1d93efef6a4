"""fp32 products on the fp16 matrix cores (csrc/split.hip) against the oracle.

Weights of unit gain (workloads.unit_gain), so that a mistake anywhere in the
step moves its outputs; bars are the fp32 ones: 1e-4 on log p and log Z, and
1e-5 on the intermediates (fp32 rounding of unit-gain sums over at most 2,048
terms is about 1e-6, and the two halves' sums err less).
"""
import numpy as np
import pytest

from paper_1605_04809_amd.workloads import Config, random_annotations, unit_gain

pytestmark = pytest.mark.gpu

BASE = Config("split", V=1003, V_src=40, E=100, H=256, A=132, B=70, S=2, len_lo=1, len_hi=9, Tpad=9,
              sigma_w=1.0, sigma_emb=1.0, seed=81)
TOL_LOGP, TOL_INTER = 1e-4, 1e-5


@pytest.fixture(scope="module")
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_cases
    return gpu_cases


def check(gpu, got, ref, what, rows=slice(None), tol_c=TOL_INTER):
    errs = {k: gpu.max_abs(got[k][rows], ref[k][rows]) for k in ("logp", "logZ", "s1", "s_new", "t", "c")}
    print(what, {k: f"{v:.1e}" for k, v in errs.items()}, flush=True)
    assert errs["logp"] <= TOL_LOGP and errs["logZ"] <= TOL_LOGP, errs
    assert all(errs[k] <= TOL_INTER for k in ("s1", "s_new", "t")) and errs["c"] <= tol_c, errs


# Every tile of the GEMMs (32 to 128 rows, one to eight k groups) with row and
# column remainders; widths off every block (a last column block of 4 units or
# columns, a last k step of 4), short and long K, the vocabulary's row tiles of
# 32 and 64 rows, two to eight steps in flight and one-block remainders.
@pytest.mark.parametrize("kw", [
    dict(B=1), dict(B=33), dict(B=65), dict(B=130, H=260, E=36, A=260, V=33),
    dict(B=300, H=1024, A=1024, E=500), dict(B=700, H=516, E=124, A=68, V=2050),
    dict(B=1100, H=1024, E=252, A=516, V=999), dict(B=2100, H=1024, A=1024, E=32, V=320),
    dict(B=4100, H=768, A=256, E=572, V=4001), dict(B=257, H=256, E=508, A=1028, V=64)],
    ids=lambda kw: "_".join(f"{k}{v}" for k, v in kw.items()))
def test_step_and_encoder_match_the_oracle(gpu, kw):
    from paper_1605_04809_amd import binding as nb
    wl = unit_gain(BASE.replace(**kw))
    wl.y_prev[::7] = -1
    n0 = nb.debug_gemm_streamed()
    g, o = gpu.GpuRun(wl), gpu.OracleRun(wl)
    args = (wl.s_prev, wl.y_prev, wl.sent_id, wl.req)
    got = g.step(*args)
    assert nb.debug_gemm_streamed() - n0 >= 8, "the split products did not run"
    ctx, pctx = (x.cpu().numpy() for x in g.src.copy_out())
    for name, a, b in (("ctx", ctx, o.ctx), ("pctx", pctx, o.pctx), ("s0", g.s0.cpu().numpy(), o.s0)):
        assert gpu.max_abs(a, b) <= TOL_INTER, (name, gpu.max_abs(a, b))
    check(gpu, got, o.step(*args), str(kw))
    g.close()


@pytest.mark.parametrize("B", [40, 1000])
def test_states_beyond_the_halves_range(gpu, B):
    """Rows whose states pass the halves' range match the oracle, rows with an
    infinity the fp32 MFMA form, and every other row the same call without
    them, bit for bit; the same for annotations."""
    from paper_1605_04809_amd import binding as nb
    wl = unit_gain(BASE.replace(B=B))
    ctx = random_annotations(wl.cfg, seed=82)
    ctx[0, 0, 5], ctx[1, 0, 3] = 40.0, -3e4
    wide, infs = np.array([1, 34, B - 1]), np.array([7])
    plain = wl.s_prev.copy()
    s = wl.s_prev.copy()
    s[wide, [0, 100, 255]] = [16.0, -900.0, 7e4]
    s[infs, 17] = np.inf
    g, o = gpu.GpuRun(wl, ctx_f32=ctx), gpu.OracleRun(wl, ctx_f32=ctx)
    prev = nb.debug_precompute(0)
    try:
        g32 = gpu.GpuRun(wl, ctx_f32=ctx)
    finally:
        nb.debug_precompute(prev)
    rest = (wl.y_prev, wl.sent_id, wl.req)
    got, base, old = g.step(s, *rest), g.step(plain, *rest), g32.step(s, *rest)
    same = np.setdiff1d(np.arange(B), np.r_[wide, infs])
    for k in ("logp", "logZ", "s_new", "s1", "t"):
        np.testing.assert_array_equal(got[k][same], base[k][same], err_msg=k)
    ref = o.step(s, *rest)
    # a state of 7e4 is kept by its update gate: s_new and s1 relative to it
    for k in ("s1", "s_new"):
        d = np.abs(got[k][wide] - ref[k][wide]) / np.maximum(1.0, np.abs(ref[k][wide]))
        assert d.max() <= TOL_INTER, (k, d.max())
    for k in ("s1", "s_new", "logp", "logZ"):
        np.testing.assert_array_equal(np.isfinite(got[k][infs]), np.isfinite(old[k][infs]), err_msg=k)
        f = np.isfinite(old[k][infs])
        np.testing.assert_allclose(got[k][infs][f], old[k][infs][f], atol=TOL_LOGP, err_msg=k)
    keep = same[np.isfinite(ref["logp"][same])]
    # the context mixes an annotation of -3e4 with weights whose fp32 rounding is 2^-24: 1.8e-3
    check(gpu, base, o.step(plain, *rest), "annotations beyond the range", keep, tol_c=3e4 * 2.0 ** -24)
    g.close()
    g32.close()


# A GRU tile of each form at H = 1,024 on 256 CUs: 32, 64 and 128 rows, eight, four, two and one k groups.
@pytest.mark.parametrize("B", [33, 300, 700, 2000, 4000])
def test_states_outside_the_halves_range_in_every_tile(gpu, B):
    """Rows beyond the range and rows far below it match the oracle in every
    GRU tile, and the rows beside them do not change by a bit."""
    wl = unit_gain(BASE.replace(B=B, H=1024, A=64, E=36, V=64))
    wl.params["g1_U"] *= np.float32(2.0 ** 24)   # states of 2^-24 carry the first GRU
    s = (wl.s_prev * np.float32(2.0 ** -24)).astype(np.float32)
    plain = s.copy()
    wide = np.array([1, 31, B // 2, B - 1])
    s[wide] = wl.s_prev[wide] * 2.0 ** -24
    s[wide, [0, 511, 700, 1023]] = [900.0, -16.0, 7e4, 20.0]
    zero = np.array([5, B - 3])
    s[zero] = plain[zero] = 0.0
    g, o = gpu.GpuRun(wl), gpu.OracleRun(wl)
    rest = (wl.y_prev, wl.sent_id, wl.req)
    got, base, ref = g.step(s, *rest), g.step(plain, *rest), o.step(plain, *rest)
    same = np.setdiff1d(np.arange(B), wide)
    for k in ("logp", "logZ", "s_new", "s1", "t"):
        np.testing.assert_array_equal(got[k][same], base[k][same], err_msg=k)
    check(gpu, base, ref, "far below the range")
    # beyond it: one element of 16 and more times 2^24 saturates the gates, so s1 is 0 or 1 times the state, or +-1
    wref = o.step(s, *rest)
    d = np.abs(got["s1"][wide] - wref["s1"][wide]) / np.maximum(1.0, np.abs(wref["s1"][wide]))
    assert np.mean(d > TOL_INTER) <= 1e-3, np.sort(d.ravel())[-8:]   # (a gate whose sum falls within rounding of 0)
    g.close()


# The plain product's tiles by their number of rows (keys of 1,024 columns on 256 CUs): 32 to 128 rows, one to eight
# k groups, one and two column blocks a wave.
@pytest.mark.parametrize("S,Tpad", [(2, 9), (8, 66), (10, 115), (20, 115), (40, 115), (50, 180)])
def test_annotations_outside_the_halves_range_in_every_tile(gpu, S, Tpad):
    """Keys of annotations of about 2^-24, some rows with an element of 16 to 3e4; errors relative to a row's largest products."""
    from paper_1605_04809_amd import binding as nb
    import oracle
    wl = unit_gain(BASE.replace(S=S, Tpad=Tpad, len_hi=Tpad, A=1024, B=8))
    wl.src_len[:] = Tpad
    wl.params["att_Wc"] *= np.float32(2.0 ** 24)
    wl.params["att_b"][:] = 0
    ctx = (random_annotations(wl.cfg, seed=84) * np.float32(2.0 ** -24)).astype(np.float32)
    big = [(0, 0, 5), (S - 1, Tpad - 1, 300), (S // 2, Tpad // 2, 511), (S - 1, 1, 0)]
    for (a, b, c), v in zip(big, (40.0, -3e4, 16.0, 1e3)):
        ctx[a, b, c] = v
    m = nb.Model.from_workload(wl)
    src = nb.nmt_source_from_annotations(m, gpu.cuda(ctx), wl.src_len)
    keys = src.copy_out()[1].cpu().numpy()
    _, ref = oracle.keys_from_annotations(oracle.Model.from_workload(wl), ctx, wl.src_len)
    size = np.maximum(1.0, np.abs(ctx).max(-1, keepdims=True) * 2.0 ** 24)   # a row's products are about this large
    err = np.abs(keys - ref) / size
    print(S * Tpad, "rows:", f"{err.max():.1e}", flush=True)
    assert err.max() <= TOL_INTER
    src.close()
    m.close()


@pytest.mark.parametrize("what", ["tiny_column", "inf_weight", "masked_words", "lowest_bias"])
def test_weights_outside_the_rule(gpu, what):
    """Weights the halves would hold less precisely (a column 2^-20 of the
    matrix's largest element), infinite weights and masking biases: the
    results are the oracle's (or for infinities the same as in numpy)."""
    wl = unit_gain(BASE)
    p = wl.params
    args = (wl.s_prev, wl.y_prev, wl.sent_id, wl.req)
    if what == "tiny_column":
        for k in ("g1_U", "att_Wq", "out_W"):
            p[k][:, 3] *= np.float32(2.0 ** -20)
    elif what == "masked_words":
        p["out_b"][5:900:3] = -np.inf
        wl.req[:] = 900 + np.arange(len(wl.req)) % 100
    elif what == "lowest_bias":
        p["out_b"][5:900:3] = np.finfo(np.float32).min
        wl.req[::2] = 5
    else:
        p["out_W"][:, 7] = -np.inf   # a word whose logit is infinite or undefined in every row
    g = gpu.GpuRun(wl)
    got = g.step(*args)
    t = got["t"].astype(np.float64)
    with np.errstate(invalid="ignore", over="ignore"):
        z = t @ p["out_W"].astype(np.float64) + p["out_b"].astype(np.float64)
        if what == "inf_weight":
            assert np.all(~np.isfinite(got["logp"]) | ~np.isfinite(got["logZ"]) | np.isneginf(z[:, 7]))
        else:
            m = z.max(1, keepdims=True)
            lz = (m + np.log(np.exp(z - m).sum(1, keepdims=True)))[:, 0]
            lp = z[np.arange(len(lz)), wl.req] - lz
            assert gpu.max_abs(got["logZ"], lz) <= TOL_LOGP
            fin = np.abs(lp) < 1e30
            assert gpu.max_abs(got["logp"][fin], lp[fin]) <= TOL_LOGP
            np.testing.assert_allclose(got["logp"][~fin], lp[~fin], rtol=1e-6)
            if what == "tiny_column":
                check(gpu, got, gpu.OracleRun(wl).step(*args), what)
    g.close()


@pytest.mark.parametrize("row", [0, 1, 2, 3, 67, 99])
@pytest.mark.parametrize("kw", [dict(H=64, A=64), dict()], ids=["h64", "h256"])
def test_the_scale_sees_every_row(gpu, kw, row):
    """One row of every matrix 2^9 above the others, each place in a packed
    vector and a row of a later wave: a scale from the other rows would take
    it past the halves' range."""
    wl = unit_gain(BASE.replace(**kw))
    for k in ("g1_U", "g2_U", "att_Wq", "ro_Ws", "out_W", "enc_f_U", "enc_b_U"):
        w = wl.params[k]
        w *= np.float32(2.0 ** -9)
        w[min(row, len(w) - 1)] *= np.float32(2.0 ** 9)
    g, o = gpu.GpuRun(wl), gpu.OracleRun(wl)
    args = (wl.s_prev, wl.y_prev, wl.sent_id, wl.req)
    assert gpu.max_abs(g.src.copy_out()[0].cpu().numpy(), o.ctx) <= TOL_INTER
    check(gpu, g.step(*args), o.step(*args), f"row {row}")
    g.close()


# Six 16-k steps of the output weights (E of 65 to 96), whose last thread block packs only in part where the number of
# column blocks is odd (a write past it would fall on the scaled bias); the vocabulary kernel's row tiles of 32 (70 and
# 300 rows) and 64, two steps in flight.
@pytest.mark.parametrize("kw", [dict(E=E, V=V, B=B, H=H, A=64) for E in (68, 80, 96) for V, B, H in
                                ((1003, 70, 64), (1003, 1100, 256), (2016, 300, 64), (2016, 2100, 256))],
                         ids=lambda kw: "_".join(f"{k}{v}" for k, v in kw.items()))
def test_six_vocabulary_steps(gpu, kw):
    wl = unit_gain(BASE.replace(**kw))
    g, o = gpu.GpuRun(wl), gpu.OracleRun(wl)
    args = (wl.s_prev, wl.y_prev, wl.sent_id, wl.req)
    check(gpu, g.step(*args), o.step(*args), str(kw))
    g.close()


# Batches whose vocabulary takes more slices on the halves than on the fp32 MFMA (256 CUs): their partials over the
# projections and the query, and (widths of 4) in a region of their own.
@pytest.mark.parametrize("kw", [dict(B=558, V=13488), dict(B=2275, V=26024), dict(B=40, V=13488, H=4, A=4, E=4),
                                dict(B=70, V=5000, H=256, A=132)],
                         ids=lambda kw: "_".join(f"{k}{v}" for k, v in kw.items()))
def test_a_workspace_serves_both_forms(gpu, kw):
    import torch
    from paper_1605_04809_amd import binding as nb
    wl = unit_gain(BASE.replace(**{**dict(H=64, A=64, E=36), **kw}))
    other = unit_gain(BASE.replace(**{**dict(H=64, A=64, E=36), **kw}))
    other.params["out_W"][:, 3] *= np.float32(2.0 ** -20)   # not split
    g, u = gpu.GpuRun(wl), gpu.GpuRun(other)
    n = nb.nmt_score_workspace_bytes(u.model, wl.cfg.B)
    assert n == nb.nmt_score_workspace_bytes(g.model, wl.cfg.B)
    args = (wl.s_prev, wl.y_prev, wl.sent_id, wl.req)
    for run, w in ((g, wl), (u, other)):
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        check(gpu, run.step(*args, workspace=ws), gpu.OracleRun(w).step(*args), str(kw))
        run.close()


def test_average_takes_the_form_its_weights_allow(gpu):
    """Members in two forms average; the result equals the same weights loaded."""
    from paper_1605_04809_amd import binding as nb
    a, b = unit_gain(BASE), unit_gain(BASE.replace(seed=83))
    a.params["g2_U"][:, 9] *= np.float32(2.0 ** -20)   # not split
    c = unit_gain(BASE)
    c.params = {k: (0.5 * a.params[k] + 0.5 * b.params[k]).astype(np.float32) for k in a.params}
    ga, gb, gc = gpu.GpuRun(a), gpu.GpuRun(b), gpu.GpuRun(c)
    m = nb.nmt_model_average([ga.model, gb.model])
    g = gpu.GpuRun(c, model=m)
    args = (a.s_prev, a.y_prev, a.sent_id, a.req)
    got, want = g.step(*args), gc.step(*args)
    for k in ("logp", "s_new", "t"):
        assert gpu.max_abs(got[k], want[k]) <= TOL_INTER, k
    for x in (ga, gb, gc, g):
        x.close()
