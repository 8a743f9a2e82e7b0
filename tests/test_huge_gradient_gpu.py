"""bf16 matrix-core path: any finite bf16 gradient is in the domain, up to the largest (3.39e38).  The power of two that brings a token's
largest gradient into the range of fp16 has to stay a normal fp32 number with a normal reciprocal."""
import numpy as np
import pytest

from oracle import linattn_oracle as O
from oracle import relu_oracle as R
from paper_2510_08318_amd import synth
from tests.test_bf16_paths_gpu import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["plain", "centred", "relu"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("value", [1e37, 1.5e38, 2.5e38, 3.38e38])
def test_huge_gradient_row(value, d, mode):
    x = synth.generate("C5", n=300, H=2, d=d, dtype="bf16")
    v = O.to_f64(x.v).astype(np.float32) * np.float32(0.01)      # nothing the gradients are made of leaves the range of fp32
    x.v = synth._pack(v, x.dtype)
    do = O.to_f64(x.dout).astype(np.float32)
    do[0, 0, 130, 5] = value
    x.dout = synth._pack(do, x.dtype)
    relu = mode == "relu"
    got = _run(x, relu, True, mode == "centred")
    ref = dict(zip(("dq", "dk", "dv", "dwq", "dwk"), R.relu_bwd_bh(x.q, x.k, x.v, x.dout) if relu
                   else O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)))
    # the head with the huge row (dq: that row; the others are as ever), relative to its largest magnitude; and the other head
    for name, r in ref.items():
        g, r0 = got[name], r
        assert np.isfinite(g).all(), name
        a, b = (g[0, 0], r0[0, 0]) if name in ("dq", "dk", "dv") else (g[0], r0[0])
        assert np.abs(a - b).max() <= 1e-2 * np.abs(b).max(), (name, np.abs(a - b).max() / np.abs(b).max())
        a, b = (g[0, 1], r0[0, 1]) if name in ("dq", "dk", "dv") else (g[1], r0[1])
        assert np.abs(a - b).max() <= 1e-2 * np.abs(b).max(), name
