"""bf16 backward: the sum dS = sum phi(q)^T dO / den takes phi rounded to fp16, and its normaliser is formed from the same rounded values, so
a rounding that a token's features have in common drops out of phi / den."""
import numpy as np
import pytest

from oracle import linattn_oracle as O
from paper_2510_08318_amd import synth
from tests.test_bf16_paths_gpu import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("centred", [False, True], ids=["plain", "centred"])
@pytest.mark.parametrize("d", [64, 128])
def test_rounding_common_to_a_token_drops_out_of_dS(d, centred):
    """Every query has three features of 1/3 in each half of phi and next to nothing elsewhere, and fp16 holds 1/3 with a relative error of
    2^-12: against a normaliser from unrounded phi all of dS, and with it dW~_k, is 2^-12 = 2.4e-4 too small.  With the shared
    rounding only independent roundings are left, 2^-12 for each of the d channels of dS and of the 12 heads: 1e-5 in the
    mean.  Bar: half of 2^-12."""
    x = synth.generate("C5", n=2000, H=12, d=d, dtype="bf16")
    w = np.zeros((x.H, d, d // 2), np.float32)
    w[:, 0, :3], w[:, 0, 3:6] = 16.0, -16.0
    x.wq = synth._pack(w, x.dtype)
    q = O.to_f64(x.q).astype(np.float32)
    q[..., 0] = 1.0
    x.q = synth._pack(q, x.dtype)
    dwk = _run(x, False, True, centred)["dwk"]
    ref = O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)[4]
    # per head, so that no head's scale decides
    slope = np.mean([np.sum(a * r) / np.sum(r * r) for a, r in zip(dwk, ref)]) - 1.0
    assert abs(slope) <= 2.0 ** -13, slope


@pytest.mark.parametrize("centred", [False, True], ids=["plain", "centred"])
@pytest.mark.parametrize("d", [64, 128])
def test_token_whose_keyed_features_round_to_zero(d, centred):
    """The keys all sit on one feature of each half, one query on others: its phi at the keys' features is exp(-30), zero in fp16.  Its
    rounded normaliser is zero; the gradients that sum over the queries stay finite."""
    x = synth.generate("C5", n=300, H=2, d=d, dtype="bf16")
    w = np.zeros((x.H, d, d // 2), np.float32)
    w[:, 0, 0], w[:, 0, 1], w[:, 1, 2], w[:, 1, 3] = 30.0, -30.0, 30.0, -30.0
    x.wq = x.wk = synth._pack(w, x.dtype)
    for name in ("q", "k"):
        t = O.to_f64(getattr(x, name)).astype(np.float32)
        t[..., :2] = [1.0, 0.0]
        if name == "q":
            t[:, :, 7, :2] = [0.0, 1.0]
        setattr(x, name, synth._pack(t, x.dtype))
    got = _run(x, False, True, centred)
    for name in ("dk", "dv", "dwk"):
        assert np.isfinite(got[name]).all(), name
