"""The query-side backward's wavefronts of 16 tokens: lengths around a wavefront's, a tile's and a workgroup's share, and tokens whose upstream
gradient vanishes, is far below its neighbours' or is not finite, which the per-token weights of the sums dS and dz have to carry.

Bar: 1e-2 element by element, the bar of the bf16 mode."""
import numpy as np
import pytest

from oracle import linattn_oracle as O
from oracle import relu_oracle as R
from paper_2510_08318_amd import synth
from tests.test_bf16_paths_gpu import _check, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [15, 16, 17, 63, 113, 127, 129, 256 * 128 + 5])
def test_lengths(n, d):
    _check(synth.generate("C5", n=n, H=1, B=1, d=d, dtype="bf16"), centred=n == 113)


def _with_gradient(d, edit, n=333):
    x = synth.generate("C5", n=n, H=2, B=1, d=d, dtype="bf16")
    do = O.to_f64(x.dout).astype(np.float32)
    edit(do)
    x.dout = synth._pack(do, x.dtype)
    return x


@pytest.mark.parametrize("centred", [False, True], ids=["plain", "centred"])
@pytest.mark.parametrize("d", [64, 128])
def test_tokens_without_or_with_tiny_gradients(d, centred):
    def edit(do):
        do[:, :, ::3] = 0.0                    # in every wavefront
        do[:, :, 128:256] = 0.0                # a whole tile
        do[:, :, 1::5] *= 2.0 ** -8            # below the others of their wavefront, whose du share a scale: fp16 has 11 bits down to 2^-14
        do[:, :, 300:] *= 2.0 ** -110          # below what fp16 holds at any scale of a token
    x = _with_gradient(d, edit)
    ref = O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)
    got = _run(x, False, True, centred)
    for name, r in zip(("dk", "dv", "dwq", "dwk"), (ref[1], ref[2], ref[3], ref[4])):
        assert O.err_metric(got[name], r)[0] <= 1e-2, name
    # dq is proportional to a token's dO: each magnitude against its own floor
    for rows in (slice(0, 1), slice(2, 128, 15), slice(1, 128, 15)):
        r = ref[0][:, :, rows]
        if not r.any():
            assert not got["dq"][:, :, rows].any()
        else:
            assert O.err_metric(got["dq"][:, :, rows], r)[0] <= 1e-2, rows


@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_gradient_that_is_not_finite(value):
    """One entry of head 0: dk of that head sums it into every row, the other head has none of it."""
    def edit(do):
        do[0, 0, 40, 3] = value
    x = _with_gradient(128, edit)
    got = _run(x, False, True)
    ref = O.bwd_bh(x.q[:, 1:], x.k[:, 1:], x.v[:, 1:], x.wq[1:], x.wk[1:], x.dout[:, 1:])
    assert not np.isfinite(got["dk"][0, 0]).any() and not np.isfinite(got["dv"][0, 0, :, 3]).any()
    assert not np.isfinite(got["dq"][0, 0, 40]).any()
    finite = np.delete(np.arange(x.n), 40)
    assert np.isfinite(got["dq"][0, 0][finite]).all()
    for name, r in zip(("dq", "dk", "dv"), ref):
        assert O.err_metric(got[name][:, 1:], r)[0] <= 1e-2, name


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("relu", [False, True], ids=["hedgehog", "relu"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("token", [40, 300])
def test_gradient_that_is_not_finite_stays_in_its_channel_of_dv(token, d, relu, value):
    """dv_j = phi(k_j) dS takes channel c of dout into channel c alone; and dq of the other tokens does not take that token's dout."""
    def edit(do):
        do[0, 0, token, 3] = value
    x = _with_gradient(d, edit)
    got = _run(x, relu, False)
    def zeroed(do):
        do[0, 0, token, 3] = 0.0
    y = _with_gradient(d, zeroed)
    ref = R.relu_bwd_bh(y.q, y.k, y.v, y.dout) if relu else O.bwd_bh(y.q, y.k, y.v, y.wq, y.wk, y.dout)
    others, tokens = np.delete(np.arange(d), 3), np.delete(np.arange(x.n), token)
    # (ReLU: a key without a positive channel has dv = 0, or 0 times an infinity)
    dead = (O.to_f64(x.k)[0, 0] <= 0).all(-1) if relu else np.zeros(x.n, bool)
    assert not np.isfinite(got["dv"][0, 0, ~dead, 3]).any()
    assert O.err_metric(got["dv"][:, :1, :, others], ref[2][:, :1, :, others])[0] <= 1e-2
    assert O.err_metric(got["dq"][:, :1, tokens], ref[0][:, :1, tokens])[0] <= 1e-2


@pytest.mark.parametrize("relu", [False, True], ids=["hedgehog", "relu"])
@pytest.mark.parametrize("d", [64, 128])
def test_channels_of_the_gradient_far_below_the_others(d, relu):
    """A channel of dv comes from that channel of dout alone.  The largest operand of a workgroup's sum dS is scaled to 2^4, so one 2^-18 below it lies at
    2^-14, the smallest with 11 bits, and those of tokens with less weight have fewer: of the ReLU map, whose 1 / den spreads most, a few binades, 2^-9 of
    the sum; beside the bf16 store (2^-9), 2^-8 in 2-norm."""
    def edit(do):
        do[..., 5::16] *= 2.0 ** -18
    x = _with_gradient(d, edit)
    ref = R.relu_bwd_bh(x.q, x.k, x.v, x.dout)[2] if relu else O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)[2]
    dv = _run(x, relu, False)["dv"]
    a, r = dv[..., 5::16], ref[..., 5::16]
    assert np.linalg.norm(a - r) <= 2.0 ** -8 * np.linalg.norm(r)


# the key side deals 128 tokens to a workgroup: without dW~ blocks of 16 to 8 wavefronts, with it tiles to 8 beside 4 that contract them
@pytest.mark.parametrize("wgrads", [False, True], ids=["frozen", "wgrads"])
@pytest.mark.parametrize("n,H,d", [(1, 2, 128), (15, 2, 64), (17, 2, 128), (191, 2, 128), (193, 2, 128), (127, 2, 64), (129, 2, 64), (400, 255, 64),
                                   (193, 300, 128), (127, 2, 128), (128, 2, 128), (129, 2, 128), (128, 2, 64)])
def test_key_side_lengths(n, H, d, wgrads):
    x = synth.generate("C5", n=n, H=H, B=1, d=d, dtype="bf16")
    if n == 1:        # the output does not depend on k
        got = _run(x, False, wgrads)
        dv = O.bwd_bh(x.q, x.k, x.v, x.wq, x.wk, x.dout)[2]
        assert O.err_metric(got["dv"], dv)[0] <= 1e-2 and np.abs(got["dk"]).max() <= 1e-2 * np.abs(dv).max()
        return
    _check(x, wgrads=wgrads)


@pytest.mark.parametrize("scale", [1e36, 3e38])
def test_gradients_whose_quotient_by_the_normaliser_passes_fp32(scale):
    """One token: den = phi(q) . phi(k) is far below 1, |dO| / den above the largest fp32 for the larger of the two.  dv = dO there; what cannot
    be summed must not come out finite and wrong."""
    x = synth.generate("C5", n=1, H=4, B=1, d=128, dtype="bf16")
    do = np.sign(O.to_f64(x.dout).astype(np.float32)) * np.float32(scale)
    x.dout = synth._pack(do, x.dtype)
    dv = _run(x, False, False)["dv"]
    ref = O.to_f64(x.dout)
    for h in range(4):
        assert not np.isfinite(dv[0, h]).all() or O.err_metric(dv[:, h:h + 1], ref[:, h:h + 1])[0] <= 1e-2
    if scale == 1e36:
        assert O.err_metric(dv, ref)[0] <= 1e-2
