"""Kernels whose workgroups take the end of one head and the start of the next (make_deal's even deal): a whole step in every mode at a
number of heads that does not divide the compute units, with a ragged last unit.  129 heads of 600 tokens are 3 units of 8 blocks and 5
tiles each: one workgroup a head would leave half of the compute units idle, so units are dealt evenly, 1 to 2 (2 to 3 tiles) a workgroup.

Bars: 1e-2 element by element for bf16 results, 1e-5 for fp32 ones (2e-5 for their weight gradients, sums over all tokens)."""
import functools

import numpy as np
import pytest

from oracle import linattn_oracle as O
from oracle import relu_oracle as R
from paper_2510_08318_amd import synth

pytestmark = pytest.mark.gpu
REL_R = 0.37
SHARED = (43, 3, 600)          # heads, batch items, tokens


@functools.lru_cache(None)
def _case(d, dtype, shape):
    H, B, n = shape
    return synth.generate("C5", n=n, H=H, B=B, d=d, dtype=dtype)


def _softmax_branch(x):
    return synth._pack((np.random.default_rng(x.d).standard_normal(x.q.shape) * 0.1).astype(np.float32), x.dtype)


@functools.lru_cache(None)
def _reference(d, dtype, form, shape):
    x = _case(d, dtype, shape)
    if form == "relu":
        return (("out", R.relu_fwd_bh(x.q, x.k, x.v)), *zip(("dq", "dk", "dv"), R.relu_bwd_bh(x.q, x.k, x.v, x.dout)))
    names = ("dq", "dk", "dv", "dwq", "dwk")
    if form == "blend":
        s = _softmax_branch(x)
        *grads, _, dr = O.blend_bwd_bh(x.q, x.k, x.v, x.wq, x.wk, s, REL_R, x.dout)
        return (("out", O.blend_fwd_bh(x.q, x.k, x.v, x.wq, x.wk, s, REL_R)), ("dr", dr), *zip(names, grads))
    return (("out", O.fwd_bh(x.q, x.k, x.v, x.wq, x.wk)), *zip(names, O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)))


@pytest.mark.parametrize("layout", ["bhnd", "bnhd"])
@pytest.mark.parametrize("form", ["weight gradients", "frozen map", "blend", "centred", "relu"])
@pytest.mark.parametrize("mode,d", [("bf16", 64), ("bf16", 128), ("f32math", 64), ("f32math", 128), ("f32", 64), ("f32", 128)])
def test_step_with_heads_that_share_workgroups(mode, d, form, layout):
    if form == "centred" and mode != "bf16":
        pytest.skip("the flag belongs to the bf16 mode")
    if layout == "bnhd" and form in ("frozen map", "centred"):
        pytest.skip("covered by the other forms")
    _step(mode, d, form, layout, SHARED)


# The bf16 query pass, whose rounds on a part of the compute units cost less, has 600 tokens dealt head by head (the blended one of width 128
# evenly); 1050 tokens, five units a head, it deals evenly: 2 to 3 a workgroup.
@pytest.mark.parametrize("form", ["frozen map", "blend", "relu"])
@pytest.mark.parametrize("d", [64, 128])
def test_query_pass_with_heads_that_share_workgroups(d, form):
    _step("bf16", d, form, "bhnd", (43, 3, 1050))


# The same of the fp32 query passes that are bound by the memory system.
@pytest.mark.parametrize("form", ["blend", "relu"])
def test_fp32_query_pass_with_heads_that_share_workgroups(form):
    _step("f32", 128, form, "bhnd", (43, 3, 1050))


# 100 heads of 640 tokens: two workgroups a head, two rounds of 8 wavefronts or one of 12, which the query pass takes then
@pytest.mark.parametrize("form", ["frozen map", "blend", "relu"])
@pytest.mark.parametrize("d", [64, 128])
def test_query_pass_of_twelve_wavefronts(d, form):
    _step("bf16", d, form, "bhnd", (50, 2, 640 - 3))


# Twelve wavefronts in the forms that these miss.  103 heads of 1140 tokens, width 64: nine tiles, so the state comes from a reduction; two
# workgroups a head, three rounds of 8 wavefronts or two of 12.  155 heads of 1019 tokens with blend, width 128: three units of 12 to a
# head, the last with 8 blocks, dealt evenly over all compute units.
@pytest.mark.parametrize("d,form,shape", [(64, "frozen map", (103, 1, 1140)), (64, "blend", (103, 1, 1140)), (64, "relu", (103, 1, 1140)),
                                          (128, "blend", (31, 5, 1019))])
def test_other_query_passes_of_twelve_wavefronts(d, form, shape):
    _step("bf16", d, form, "bhnd", shape)


def _step(mode, d, form, layout, shape):
    import torch
    from paper_2510_08318_amd import torch_glue as G
    relu, f32_math = form == "relu", mode == "f32math"
    x = _case(d, "f32" if mode == "f32" else "bf16", shape)
    perm = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if layout == "bnhd" else (lambda t: t)
    back = (lambda t: t.permute(0, 2, 1, 3)) if layout == "bnhd" else (lambda t: t)
    q, k, v, do = [perm(G.to_device(t)) for t in (x.q, x.k, x.v, x.dout)]
    if relu:
        lay = G.ReluLayer(x.H, x.d, x.B, x.n, q.dtype, layout=layout, f32_math=f32_math)
    else:
        lay = G.Layer(G.to_device(x.wq), G.to_device(x.wk), x.B, x.n, want_wgrads=form != "frozen map", layout=layout, f32_math=f32_math,
                      centred=form == "centred")
    if form == "blend":
        s = _softmax_branch(x)
        dr = torch.zeros(1, device="cuda")
        lay.set_blend(perm(G.to_device(s)), torch.tensor([REL_R], device="cuda"), dr)
    got = {"out": back(lay.forward(q, k, v))}
    got.update(zip(("dq", "dk", "dv"), (back(t) for t in lay.backward(q, k, v, do))))
    if not relu and form != "frozen map":
        got.update(dwq=lay.dwq, dwk=lay.dwk)
    got = {name: G.to_host_f64(t) for name, t in got.items()}
    ref = dict(_reference(d, x.dtype, form if form in ("relu", "blend") else "plain", shape))
    if form == "blend":
        # dL/dr is a sum of products of random sign: 1e-2 of its spread
        assert abs(float(dr) - ref.pop("dr")) <= 1e-2 * np.sqrt(np.square(O.to_f64(x.dout) * O.to_f64(s)).sum())
    lay.close()
    for name, r in ref.items():
        if name in got:
            bar = (2e-5 if name in ("dwq", "dwk") else 1e-5) if mode == "f32" or (f32_math and name in ("dwq", "dwk")) else 1e-2
            assert O.err_metric(got[name], r)[0] <= bar, name


# 45 heads of 3870 tokens without blend: 16 units of 8 blocks or 11 of 12 a head, both dealt evenly, three rounds or two; a head's last unit of 12 has one block
@pytest.mark.parametrize("d,form", [(64, "frozen map"), (128, "frozen map"), (128, "relu")])
def test_twelve_wavefronts_dealt_evenly(d, form):
    _step("bf16", d, form, "bhnd", (45, 1, 3870))
