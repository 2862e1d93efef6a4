"""The encoder's one-launch recurrence (csrc/encode.hip) against the oracle:
one and two row tiles of 16 sentences, two groups of 32, two launches, more
sentences than it takes (the chain of launches), a single position, lengths
from 1 to Tpad, units off the 16-unit blocks and 32-k steps, more units than
it takes, and both weight types.

fp32 bars as in test_gpu_split.py; bf16 weights of unit gain: each state
enters the products rounded to bf16 (2^-9 relative), the recurrence passes on
less than it adds, so annotations stay within a few 1e-3 and the attention's
keys (2H of them summed at unit gain) within 2e-2.
"""
import numpy as np
import pytest

from paper_1605_04809_amd.workloads import Config, unit_gain

pytestmark = pytest.mark.gpu

BASE = Config("scan", V=64, V_src=90, E=36, H=64, A=64, B=4, S=1, len_lo=1, len_hi=7, Tpad=7,
              sigma_w=1.0, sigma_emb=1.0, seed=91)


@pytest.mark.parametrize("wtype", ["f32", "bf16"])
@pytest.mark.parametrize("kw", [dict(), dict(S=17), dict(S=33, H=100), dict(S=70, H=260), dict(S=130),
                                dict(S=3, Tpad=1, len_hi=1), dict(S=2, H=1024, Tpad=5, len_hi=5),
                                dict(S=40, H=1024, Tpad=4, len_hi=4), dict(S=2, H=1028, Tpad=3, len_hi=3),
                                dict(S=5, H=4, E=4, A=4)],
                         ids=lambda kw: "_".join(f"{k}{v}" for k, v in kw.items()) or "one")
def test_annotations_keys_and_states_match_the_oracle(kw, wtype):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_cases
    from paper_1605_04809_amd import binding as nb
    wl = unit_gain(BASE.replace(wtype=wtype, **kw))
    wl.src_len[-1] = wl.cfg.Tpad
    g, o = gpu_cases.GpuRun(wl), gpu_cases.OracleRun(wl)
    ctx, pctx = (x.cpu().numpy() for x in g.src.copy_out())
    errs = {n: gpu_cases.max_abs(a, b) for n, a, b in (("ctx", ctx, o.ctx), ("pctx", pctx, o.pctx),
                                                       ("s0", g.s0.cpu().numpy(), o.s0))}
    print(kw, wtype, {k: f"{v:.1e}" for k, v in errs.items()}, flush=True)
    tol = {"f32": (1e-5, 1e-5), "bf16": (1e-2, 2e-2)}[wtype]
    assert errs["ctx"] <= tol[0] and errs["pctx"] <= tol[1] and errs["s0"] <= tol[1], errs
    # positions past each length are zeros, and a second source is the same bit for bit
    for s, n in enumerate(wl.src_len):
        assert not ctx[s, n:].any()
    again = nb.nmt_encode(g.model, gpu_cases.cuda(wl.src_ids), wl.src_len)
    torch.cuda.synchronize()
    assert nb.nmt_stream_status(g.model) == nb.NMT_OK
    np.testing.assert_array_equal(again.copy_out()[0].cpu().numpy(), ctx)
    again.close()
    g.close()


# The chain's K splits at S of at most 64 and more: one of a few steps, seven with a longer last one, eight, four of
# eight steps; a last step and a last chunk that are not full; position and mask edges.
@pytest.mark.parametrize("kw", [dict(S=1, H=1024), dict(S=20, H=1024), dict(S=64, H=960), dict(S=65, H=1024),
                                dict(S=128, H=1000), dict(S=7, H=64), dict(S=7, H=100), dict(S=9, H=192),
                                dict(S=33, H=320), dict(S=5, H=36), dict(S=90, H=896), dict(S=70, H=704),
                                dict(S=40, H=512, Tpad=40, len_hi=40)],
                         ids=lambda kw: "_".join(f"{k}{v}" for k, v in kw.items()))
def test_bf16_states_are_the_chains_bit_for_bit(kw):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_cases
    from paper_1605_04809_amd import binding as nb
    wl = unit_gain(BASE.replace(wtype="bf16", **kw))
    g = gpu_cases.GpuRun(wl)
    one = [x.cpu().numpy() for x in g.src.copy_out()] + [g.s0.cpu().numpy()]
    prev = nb.debug_encode_form(0)
    try:
        c = gpu_cases.GpuRun(wl, model=g.model)
    finally:
        nb.debug_encode_form(prev)
    chain = [x.cpu().numpy() for x in c.src.copy_out()] + [c.s0.cpu().numpy()]
    for name, a, b in zip(("ctx", "pctx", "s0"), one, chain):
        np.testing.assert_array_equal(a.view(np.int32), b.view(np.int32), err_msg=name)
    c.src.close()
    g.close()


@pytest.mark.parametrize("wtype", ["f32", "bf16"])
@pytest.mark.parametrize("kw", [dict(), dict(S=17, H=100), dict(S=33, H=260), dict(S=70, H=1024), dict(S=5, H=4, E=4, A=4),
                                dict(S=3, Tpad=1, len_hi=1), dict(S=20, H=960, Tpad=12, len_hi=12)],
                         ids=lambda kw: "_".join(f"{k}{v}" for k, v in kw.items()) or "one")
def test_a_wait_that_runs_out_changes_nothing(kw, wtype):
    """With no wait waited out, the kernel that needs no other block computes
    the states the one launch gives, and the call is not an error."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_cases
    from paper_1605_04809_amd import binding as nb
    wl = unit_gain(BASE.replace(wtype=wtype, **kw))
    g = gpu_cases.GpuRun(wl)
    prev = nb.debug_encode_form(2)
    try:
        c = gpu_cases.GpuRun(wl, model=g.model)
    finally:
        nb.debug_encode_form(prev)
    for a, b in zip([*g.src.copy_out(), g.s0], [*c.src.copy_out(), c.s0]):
        np.testing.assert_array_equal(a.cpu().numpy().view(np.int32), b.cpu().numpy().view(np.int32))
    assert nb.nmt_stream_status(g.model) == nb.NMT_OK
    c.src.close()
    g.close()


def test_sources_on_two_streams_at_once():
    """Two recurrences in flight together give what each gives alone."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_cases
    from paper_1605_04809_amd import binding as nb
    wl = unit_gain(BASE.replace(S=20, H=1024, Tpad=7))
    g = gpu_cases.GpuRun(wl)
    want = g.src.copy_out()[0].cpu().numpy()
    ids = gpu_cases.cuda(wl.src_ids)
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    srcs = [nb.nmt_encode(g.model, ids, wl.src_len, stream=s) for s in streams for _ in range(2)]
    torch.cuda.synchronize()
    for s in srcs:
        np.testing.assert_array_equal(s.copy_out()[0].cpu().numpy(), want)
        s.close()
    assert nb.nmt_stream_status(g.model) == nb.NMT_OK
    g.close()


def test_source_blocks_come_back_and_outlive_their_model():
    """A source set up in another source's old block (larger, smaller, equal)
    is the one a fresh block gives; a source may be destroyed after its model."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_cases
    from paper_1605_04809_amd import binding as nb
    live = nb.debug_alloc_hook(-1)
    wl = unit_gain(BASE.replace(S=9, H=100))
    g = gpu_cases.GpuRun(wl)
    ids = gpu_cases.cuda(wl.src_ids)
    first = {}
    for n in (9, 4, 9, 1, 5, 4, 9):
        src = nb.nmt_encode(g.model, ids[:n].contiguous(), wl.src_len[:n])
        ctx, pctx = (x.cpu().numpy() for x in src.copy_out())
        want = first.setdefault(n, (ctx, pctx))
        np.testing.assert_array_equal(ctx, want[0])
        np.testing.assert_array_equal(pctx, want[1])
        src.close()
    g.model.close()
    g.src.close()
    assert nb.debug_alloc_hook(-1) == live


def test_more_idle_blocks_than_the_pool_keeps():
    """100 sources of growing size at once, then destroyed and set up again."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_cases
    from paper_1605_04809_amd import binding as nb
    live = nb.debug_alloc_hook(-1)
    wl = unit_gain(BASE.replace(S=1, H=32, Tpad=100, len_hi=100))
    m = nb.Model.from_workload(wl)
    ids = gpu_cases.cuda(wl.src_ids)
    want = {}
    for turn in range(2):
        srcs = [(n, nb.nmt_encode(m, ids[:, :n].contiguous(), np.array([n], np.int32))) for n in range(1, 101)]
        for n, s in srcs:
            ctx = s.copy_out()[0].cpu().numpy()
            np.testing.assert_array_equal(ctx, want.setdefault(n, ctx))
        for _, s in srcs:
            s.close()
    m.close()
    assert nb.debug_alloc_hook(-1) == live
