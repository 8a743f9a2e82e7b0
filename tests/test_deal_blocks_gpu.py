"""Short calls, whose units are of two or four blocks, beside one with units of eight: a whole step in every mode.

Bars: those of the modes, 1e-2 element by element for bf16 tensors, 1e-5 for fp32 ones and 2e-5 for their weight gradients."""
import pytest

from oracle import linattn_oracle as O
from oracle import relu_oracle as R
from paper_2510_08318_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["bf16", "relu", "f32", "f32 relu", "f32math"])
@pytest.mark.parametrize("H,n,d", [(2, 333, 64), (2, 333, 128), (20, 200, 64), (50, 333, 64), (40, 200, 128), (100, 333, 64)])
def test_step(H, n, d, mode):
    from paper_2510_08318_amd import torch_glue as G
    f32, relu = mode.startswith("f32") and mode != "f32math", "relu" in mode
    x = synth.generate("C5", n=n, H=H, B=1, d=d, dtype="f32" if f32 else "bf16")
    q, k, v, do = [G.to_device(t) for t in (x.q, x.k, x.v, x.dout)]
    if relu:
        lay = G.ReluLayer(H, d, 1, n, q.dtype)
        ref = [R.relu_fwd_bh(x.q, x.k, x.v), *R.relu_bwd_bh(x.q, x.k, x.v, x.dout)[:3]]
    else:
        lay = G.Layer(G.to_device(x.wq), G.to_device(x.wk), 1, n, want_wgrads=True, f32_math=mode == "f32math")
        ref = [O.fwd_bh(x.q, x.k, x.v, x.wq, x.wk), *O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)]
    got = [lay.forward(q, k, v), *lay.backward(q, k, v, do)] + ([] if relu else [lay.dwq, lay.dwk])
    for name, g, r in zip(("out", "dq", "dk", "dv", "dwq", "dwk"), got, ref):
        bar = (2e-5 if name.startswith("dw") else 1e-5) if f32 else 1e-2
        assert O.err_metric(G.to_host_f64(g), r)[0] <= bar, name
    lay.close()
