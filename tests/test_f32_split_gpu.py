"""The fp32-arithmetic kernels (fp32 tensors, and bf16 tensors with fp32 arithmetic), whose products are sums of bf16 piece
products on the matrix cores: sizes around their 16-, 32- and 128-token steps, more heads than workgroups, both maps, both
layouts, against the fp64 oracle.

Bar, 2-norm: 32 units of 2^-24 (1.9e-6).  A contraction of K = 128 takes 8 steps of 6 piece products, each rounding the
accumulator by 0.4 unit rms (3 units together); five contractions follow one another in a gradient (projection, state, dS,
dL/dphi, dx), and outputs and gradients are differences of terms about twice their size.  Largest error: 1e-5, the bar of the mode.
bf16 results carry the rounding of their store on top: 2^-9 in the 2-norm, 2^-8 for the largest."""
import numpy as np
import pytest

from oracle import linattn_oracle as O
from oracle import relu_oracle as R
from paper_2510_08318_amd import synth

pytestmark = pytest.mark.gpu
REL, MAX = 32 * 2.0 ** -24, 1e-5


def _run(x, relu, layout, blend=None):
    import torch
    from paper_2510_08318_amd import torch_glue as G
    perm = (lambda t: t.permute(0, 2, 1, 3).contiguous()) if layout == "bnhd" else (lambda t: t)
    back = (lambda t: t.permute(0, 2, 1, 3)) if layout == "bnhd" else (lambda t: t)
    q, k, v, do = [perm(G.to_device(t)) for t in (x.q, x.k, x.v, x.dout)]
    bf16 = x.dtype == "bf16"
    if relu:
        lay = G.ReluLayer(x.H, x.d, x.B, x.n, q.dtype, layout=layout, f32_math=bf16)
    else:
        lay = G.Layer(G.to_device(x.wq), G.to_device(x.wk), x.B, x.n, want_wgrads=True, layout=layout, f32_math=bf16)
    if blend is not None:
        dr = torch.zeros(1, device="cuda")
        lay.set_blend(perm(G.to_device(blend[0])), torch.tensor([blend[1]], device="cuda"), dr)
    got = {"out": back(lay.forward(q, k, v)), "state": lay.state}
    got.update(zip(("dq", "dk", "dv"), (back(t) for t in lay.backward(q, k, v, do))))
    if not relu:
        got.update(dwq=lay.dwq, dwk=lay.dwk)
    if blend is not None:
        got["dr"] = dr
    torch.cuda.synchronize()
    got = {name: G.to_host_f64(t) for name, t in got.items()}
    lay.close()
    return got


def _reference(x, relu):
    if relu:
        ref = {"out": R.relu_fwd_bh(x.q, x.k, x.v)}
        ref.update(zip(("dq", "dk", "dv"), R.relu_bwd_bh(x.q, x.k, x.v, x.dout)))
    else:
        ref = {"out": O.fwd_bh(x.q, x.k, x.v, x.wq, x.wk), "state": O.state_bh(x.k, x.v, x.wk)}
        ref.update(zip(("dq", "dk", "dv", "dwq", "dwk"), O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)))
    return ref


@pytest.mark.parametrize("relu", [False, True], ids=["hedgehog", "relu"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,H,B,d,layout", [(16, 2, 1, 128, "bhnd"), (17, 2, 1, 64, "bnhd"), (127, 2, 1, 64, "bhnd"), (128, 1, 2, 128, "bnhd"),
                                            (129, 3, 1, 128, "bhnd"), (257, 2, 1, 64, "bhnd"), (130, 150, 2, 64, "bnhd"), (3000, 1, 1, 128, "bhnd")])
def test_edges_of_steps_and_tiles(n, H, B, d, layout, dtype, relu):
    x = synth.generate("C5", n=n, H=H, B=B, d=d, dtype=dtype)
    _compare(_run(x, relu, layout), _reference(x, relu), dtype)


def _compare(got, ref, dtype, largest=MAX):
    for name, r in ref.items():
        rounding = 2.0 ** -9 if dtype == "bf16" and name in ("out", "dq", "dk", "dv") else 0.0
        rel = float(np.linalg.norm(got[name] - r) / np.linalg.norm(r))
        assert rel <= REL + rounding, (name, rel)
        if name != "state":
            err = O.err_metric(got[name], r)[0]
            assert err <= largest + 2 * rounding, (name, err)


@pytest.mark.parametrize("kind", ["hedgehog", "relu", "mixed"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,H,d,layout", [(6200, 12, 128, "bhnd"), (2900, 30, 64, "bnhd")])
def test_wavefronts_of_several_blocks(n, H, d, layout, dtype, kind):
    """21 (8) workgroups a head of eight wavefronts for 194 (91) blocks of 32 tokens: a wavefront takes a second block, prefetched during
    the first; 588 (690) tiles dealt to 256 workgroups: two and more a workgroup, some across a head's end.

    Largest error: 2e-5.  In the head of scale 2 the pre-softmax features of some of 6200 tokens reach 8, and three roundings of 2^-24 of
    that move a probability by 1.4e-6; where two or three features carry a token's du, which is a difference of terms twice
    its size, the nine million elements of dk go three deviations of 4e-6 out (plain fp32 FMA: 1.4e-5)."""
    largest = 2 * MAX
    x = synth.generate("C5", n=n, H=H, d=d, dtype=dtype)
    if kind != "mixed":
        return _compare(_run(x, kind == "relu", layout), _reference(x, kind == "relu"), dtype, largest)
    s = synth._pack((np.random.default_rng(n).standard_normal(x.q.shape) * 0.1).astype(np.float32), dtype)
    got = _run(x, False, layout, (s, 0.37))
    ref = {"out": O.blend_fwd_bh(x.q, x.k, x.v, x.wq, x.wk, s, 0.37), "state": O.state_bh(x.k, x.v, x.wk)}
    grads = O.blend_bwd_bh(x.q, x.k, x.v, x.wq, x.wk, s, 0.37, x.dout)
    ref.update(zip(("dq", "dk", "dv", "dwq", "dwk"), grads))
    _compare(got, ref, dtype, largest)
    # dr sums n H d products of independent signs, each rounded: 2^-24 of their root sum of squares per rounding, a few of them
    scale = np.sqrt(np.sum((O.to_f64(x.dout) * O.to_f64(s)) ** 2))
    assert abs(float(got["dr"][0]) - grads[6]) <= 1e-5 * scale


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
def test_mixed_backward_reads_s_for_the_mixing_gradient_alone(d, dtype):
    import torch
    from paper_2510_08318_amd import torch_glue as G
    x = synth.generate("C5", n=500, H=2, d=d, dtype=dtype)
    q, k, v, do = [G.to_device(t) for t in (x.q, x.k, x.v, x.dout)]
    s, r, dr = torch.randn_like(q) * 0.1, torch.tensor([0.37], device="cuda"), torch.zeros(1, device="cuda")
    grads = []
    for want in (True, False):
        lay = G.Layer(G.to_device(x.wq), G.to_device(x.wk), x.B, x.n, want_wgrads=True, f32_math=dtype == "bf16")
        lay.set_blend(s, r, dr if want else None)
        lay.forward(q, k, v)
        if not want:
            s.fill_(float("nan"))
        grads.append([t.clone() for t in lay.backward(q, k, v, do)] + [lay.dwq.clone(), lay.dwk.clone()])
        torch.cuda.synchronize()
        lay.close()
    assert torch.isfinite(dr).all()
    for a, b in zip(*grads):
        assert torch.equal(a, b) and torch.isfinite(a).all()


def test_long_sum_has_no_common_error():
    """The matrix instruction cuts the low end of a step's sum, always downwards; tiles summed with alternating sign keep that
    out of S.  Errors that are independent over the 128 features leave REL / sqrt(128) in their mean; the bias of 300 tiles
    summed alike is five times that (it is the part of the error that phi(q) S does not average out)."""
    x = synth.generate("C5", n=38400, H=1, d=128, dtype="f32")
    S = _run(x, False, "bhnd")["state"][0, 0, :128]
    ref = O.state_bh(x.k, x.v, x.wk)[0, 0, :128]
    common = np.sqrt(np.mean(np.mean(S - ref, axis=0) ** 2)) / np.sqrt(np.mean(ref ** 2))
    assert common <= REL / np.sqrt(128), common
