"""The bf16 backward stores dq and dv (ReLU: dq and dk) through the caches where the three gradients fit half of the last-level cache (3 x 2 bytes x 128 channels x
174762 tokens are the most) and past them above; the fp32-arithmetic one its dL/du rows (2 sides x 4 bytes x 64 features x 262144
tokens): one head of width 128 on both sides of the lines, the last block ragged.

Bar: 1e-2 element by element, as for every bf16 result; weight gradients of the fp32-arithmetic modes 2e-5, as elsewhere."""
import numpy as np
import pytest

from oracle import linattn_oracle as O
from oracle import relu_oracle as R
from paper_2510_08318_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [174762, 174763])
@pytest.mark.parametrize("relu", [False, True], ids=["hedgehog", "relu"])
def test_gradients_on_both_sides_of_the_line(relu, n):
    from paper_2510_08318_amd import torch_glue as G
    x = synth.generate("C5", n=n, H=1)
    q, k, v, do = [G.to_device(t) for t in (x.q, x.k, x.v, x.dout)]
    if relu:
        lay = G.ReluLayer(x.H, x.d, x.B, x.n, q.dtype)
    else:
        lay = G.Layer(G.to_device(x.wq), G.to_device(x.wk), x.B, x.n, want_wgrads=True)
    lay.forward(q, k, v)
    got = [G.to_host_f64(t) for t in lay.backward(q, k, v, do)]
    if relu:
        ref = R.relu_bwd_bh(x.q, x.k, x.v, x.dout)
    else:
        got += [G.to_host_f64(lay.dwq), G.to_host_f64(lay.dwk)]
        ref = O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)
    lay.close()
    for name, a, b in zip(("dq", "dk", "dv", "dwq", "dwk"), got, ref):
        assert np.isfinite(a).all() and O.err_metric(a, b)[0] <= 1e-2, name


@pytest.mark.parametrize("mode,n", [("f32math", 262144), ("f32math", 262145), ("f32", 262145)])
def test_du_rows_on_both_sides_of_the_line(mode, n):
    from paper_2510_08318_amd import torch_glue as G
    x = synth.generate("C5", n=n, H=1, dtype="f32" if mode == "f32" else "bf16")
    q, k, v, do = [G.to_device(t) for t in (x.q, x.k, x.v, x.dout)]
    lay = G.Layer(G.to_device(x.wq), G.to_device(x.wk), x.B, x.n, want_wgrads=True, f32_math=mode == "f32math")
    lay.forward(q, k, v)
    got = [G.to_host_f64(t) for t in lay.backward(q, k, v, do)] + [G.to_host_f64(lay.dwq), G.to_host_f64(lay.dwk)]
    lay.close()
    for name, a, b in zip(("dq", "dk", "dv", "dwq", "dwk"), got, O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)):
        bar = 2e-5 if name.startswith("dw") else 1e-5 if mode == "f32" else 1e-2
        assert np.isfinite(a).all() and O.err_metric(a, b)[0] <= bar, (name, O.err_metric(a, b)[0])
