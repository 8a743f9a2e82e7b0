"""The bf16 kernels where a workgroup's share changes its form: several heads' worth of tiles to a workgroup in the backward, the
lengths at which the query pass stops summing the partial states itself, and the numbers of partial states at which the
reduction changes its threads per element.

Bar: 1e-2 element by element for the bf16 tensors and weight gradients, the bar of the mode.  For the fp32 state, 2-norm: phi and W~
enter its matrix products rounded to 2^-11 (fp16), or 2^-9 (bf16 rows, exact); independent roundings of n terms leave 2^-11 of the norm,
and two of them (phi, and the softmax argument's products) stay below 2^-10."""
import numpy as np
import pytest

from oracle import linattn_oracle as O
from oracle import relu_oracle as R
from paper_2510_08318_amd import synth

pytestmark = pytest.mark.gpu


def _run(x, relu, wgrads, centred=False):
    import torch
    from paper_2510_08318_amd import torch_glue as G
    q, k, v, do = [G.to_device(t) for t in (x.q, x.k, x.v, x.dout)]
    if relu:
        lay = G.ReluLayer(x.H, x.d, x.B, x.n, q.dtype)
    else:
        lay = G.Layer(G.to_device(x.wq), G.to_device(x.wk), x.B, x.n, want_wgrads=wgrads, centred=centred)
    got = {"out": lay.forward(q, k, v), "state": lay.state}
    got.update(zip(("dq", "dk", "dv"), lay.backward(q, k, v, do)))
    if wgrads and not relu:
        got.update(dwq=lay.dwq, dwk=lay.dwk)
    torch.cuda.synchronize()
    got = {name: G.to_host_f64(t) for name, t in got.items()}
    lay.close()
    return got


def _check(x, relu=False, wgrads=True, centred=False):
    got = _run(x, relu, wgrads, centred)
    if relu:
        ref = {"out": R.relu_fwd_bh(x.q, x.k, x.v), "state": R.relu_state_bh(x.k, x.v)}
        ref.update(zip(("dq", "dk", "dv"), R.relu_bwd_bh(x.q, x.k, x.v, x.dout)))
    else:
        ref = {"out": O.fwd_bh(x.q, x.k, x.v, x.wq, x.wk), "state": O.state_bh(x.k, x.v, x.wk)}
        ref.update(zip(("dq", "dk", "dv", "dwq", "dwk"), O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)))
    for name, r in ref.items():
        if name not in got:
            continue
        if name == "state":
            assert np.linalg.norm(got[name] - r) <= 2.0 ** -10 * np.linalg.norm(r), name
        else:
            assert O.err_metric(got[name], r)[0] <= 1e-2, name


@pytest.mark.parametrize("mode", ["weight gradients", "frozen map", "centred", "relu"])
@pytest.mark.parametrize("d", [64, 128])
def test_backward_workgroups_of_several_tiles(d, mode):
    # 300 heads: one workgroup a head, four tiles (the last ragged) each
    _check(synth.generate("C5", n=400, H=100, B=3, d=d, dtype="bf16"), relu=mode == "relu",
           wgrads=mode != "frozen map", centred=mode == "centred")


@pytest.mark.parametrize("relu", [False, True], ids=["hedgehog", "relu"])
@pytest.mark.parametrize("n,H,d", [(1, 1, 64), (129, 2, 64), (300, 3, 64), (640, 2, 64), (1024, 5, 64), (1025, 5, 64), (1000, 100, 64), (768, 6, 64), (769, 6, 64), (1024, 4, 64),
                                   (1000, 64, 64), (1000, 65, 64), (500, 33, 64),
                                   (128, 3, 128), (256, 3, 128), (257, 3, 128), (200, 300, 128)])
def test_query_pass_that_sums_the_partials(n, H, d, relu):
    if n == 1:        # one token: the state is phi(k)^T v; out is v whatever q and k are, so dq and dk vanish (ReLU: up to its eps)
        x = synth.generate("C5", n=n, H=H, B=1, d=d, dtype="bf16")
        got = _run(x, relu, False)
        state = R.relu_state_bh(x.k, x.v) if relu else O.state_bh(x.k, x.v, x.wk)
        out = R.relu_fwd_bh(x.q, x.k, x.v) if relu else O.fwd_bh(x.q, x.k, x.v, x.wq, x.wk)
        dq, dk, dv = (R.relu_bwd_bh(x.q, x.k, x.v, x.dout) if relu else O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout))[:3]
        assert np.linalg.norm(got["state"] - state) <= 2.0 ** -10 * np.linalg.norm(state)
        assert O.err_metric(got["out"], out)[0] <= 1e-2 and O.err_metric(got["dv"], dv)[0] <= 1e-2
        for name, r in (("dq", dq), ("dk", dk)):
            assert np.abs(got[name] - r).max() <= 1e-2 * np.abs(dv).max(), name
        return
    _check(synth.generate("C5", n=n, H=H, B=1, d=d, dtype="bf16"), relu=relu)


# eight tiles a head, a slot each: summed by the query pass up to 12 heads, by a launch for 13 to 32, by the query pass again beyond
@pytest.mark.parametrize("H", [12, 13, 32, 33])
def test_query_pass_at_eight_tiles_a_head(H):
    _check(synth.generate("C5", n=1001, H=H, B=1, d=64, dtype="bf16"), wgrads=False)


@pytest.mark.parametrize("n,d", [(100, 128), (200, 128), (257, 128), (1000, 64)])
def test_mixed_attention_where_the_query_pass_sums_the_partials(n, d):
    import torch
    from paper_2510_08318_amd import torch_glue as G
    x = synth.generate("C5", n=n, H=3, B=1, d=d, dtype="bf16")
    s = synth._pack((np.random.default_rng(n).standard_normal(x.q.shape) * 0.1).astype(np.float32), x.dtype)
    lay = G.Layer(G.to_device(x.wq), G.to_device(x.wk), x.B, x.n)
    lay.set_blend(G.to_device(s), torch.tensor([0.37], device="cuda"))
    out = G.to_host_f64(lay.forward(*[G.to_device(t) for t in (x.q, x.k, x.v)]))
    state = G.to_host_f64(lay.state)
    lay.close()
    assert O.err_metric(out, O.blend_fwd_bh(x.q, x.k, x.v, x.wq, x.wk, s, 0.37))[0] <= 1e-2
    ref = O.state_bh(x.k, x.v, x.wk)
    assert np.linalg.norm(state - ref) <= 2.0 ** -10 * np.linalg.norm(ref)


@pytest.mark.parametrize("n,H", [(129 * 8, 1), (129 * 9, 1), (128 * 32, 1), (128 * 33, 1), (128 * 150, 1), (5000, 7)])
def test_reduction_of_few_and_many_partials(n, H):
    _check(synth.generate("C5", n=n, H=H, B=1, d=128, dtype="bf16"))
