"""bf16 backward: the sum dS = sum phi(q)^T dO / den takes phi rounded to fp16.  What the roundings of a token's features have in common does not
average out over tokens whose queries are alike; where it is large, the token's weight is formed with the normaliser of phi as it was rounded."""
import numpy as np
import pytest

from oracle import linattn_oracle as O
from paper_2510_08318_amd import synth
from tests.test_bf16_paths_gpu import _run

pytestmark = pytest.mark.gpu


def _slopes(d, centred, features):
    """dW~_k against 64 bits, head by head (so that no head's scale decides), with every query on the same `features` features of each half."""
    x = synth.generate("C5", n=2000, H=12, d=d, dtype="bf16")
    w = np.zeros((x.H, d, d // 2), np.float32)
    w[:, 0, :features], w[:, 0, features:2 * features] = 16.0, -16.0
    x.wq = synth._pack(w, x.dtype)
    q = O.to_f64(x.q).astype(np.float32)
    q[..., 0] = 1.0
    x.q = synth._pack(q, x.dtype)
    dwk = _run(x, False, True, centred)["dwk"]
    ref = O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)[4]
    return np.array([np.sum(a * r) / np.sum(r * r) - 1.0 for a, r in zip(dwk, ref)])


@pytest.mark.parametrize("centred", [False, True], ids=["plain", "centred"])
@pytest.mark.parametrize("d", [64, 128])
def test_rounding_common_to_a_token_drops_out_of_dS(d, centred):
    """Every query has three features of 1/3 in each half of phi and next to nothing elsewhere, which round alike, 2^-12 at most: all of dS, and
    with it dW~_k, would be off by as much.  Bar: half of 2^-12 for the mean over the heads (their independent roundings leave 2e-5)."""
    slopes = _slopes(d, centred, 3)
    assert abs(np.mean(slopes)) <= 2.0 ** -13, slopes


@pytest.mark.parametrize("centred", [False, True], ids=["plain", "centred"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("features", [1, 3])
def test_no_head_keeps_a_common_rounding(d, centred, features):
    """The same head by head (the errors of different heads differ in sign), with one feature of 1 as well: phi times the token's weight, whose digits
    are the head's, is what is rounded.  Up to 1.7e-4 of it may be left, in four ways of rounding that a head's tokens are dealt to: 5e-5 rms, beside
    the 5e-5 to 8e-5 of the independent roundings of the d channels of dS.  Bar: 2^-13 rms over the heads (with no normaliser from rounded phi
    1.5e-4 to 2.6e-4)."""
    slopes = _slopes(d, centred, features)
    assert np.sqrt(np.mean(slopes ** 2)) <= 2.0 ** -13, slopes


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
