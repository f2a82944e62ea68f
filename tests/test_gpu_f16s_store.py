"""The FP16S store of the kernels: fp16_rn(fp32_rn(v / scale)) bit for bit, the
sign of a zero included.  (GPU)

With zero links (full storage takes any finite matrix) and 4 + m0 = 1 the
operator is the identity, so an application decodes and re-encodes each site:
the expected bytes follow from the input's bytes."""
import numpy as np
import pytest
import torch

from paper_2407_00041_amd import DiracOp

from util import need_gpu

pytestmark = pytest.mark.gpu


def identity(dims):
    return DiracOp(dims, np.zeros((int(np.prod(dims)), 4, 3, 3), dtype=complex), -3.0, 0.0, precisions=("f64", "f16s"))


def halves_and_scales(field, V):
    """[V, 24] fp16 components and [V] scales of one native FP16S field."""
    raw = field.cpu().numpy()
    h = raw[:48 * V].view(np.float16).reshape(3, V, 8).transpose(1, 0, 2).reshape(V, 24)
    return h, raw[48 * V:52 * V].view(np.float32)


# 2^14 sites of one right-hand side: the small-lattice kernel; two more right-hand sides: the site kernel in pairs and
# alone.  Scales from the subnormal range to 2^120, components from far below the scale's last fp16 bit up to it
@pytest.mark.parametrize("n", [1, 3])
def test_store_rounds_like_the_division(n):
    need_gpu()
    dims = (8, 8, 16, 16)
    V = int(np.prod(dims))
    rng = np.random.default_rng(7)
    mag = rng.uniform(1.0, 2.0, (n, V, 24)) * 2.0 ** -rng.integers(0, 28, (n, V, 24))
    exp = rng.integers(-140, 121, (n, V, 1))
    psi = mag * 2.0 ** exp.astype(float) * rng.choice([-1.0, 1.0], (n, V, 24))
    op = identity(dims)
    x = op.pack(torch.from_numpy(psi[..., 0::2] + 1j * psi[..., 1::2]).cuda(), "f16s")
    y = op.empty("f16s", n).zero_()
    op.apply_native(y, x, n, "f16s")
    rb = op.field_bytes("f16s", 1)
    for r in range(n):
        h, s = halves_and_scales(x[r * rb:(r + 1) * rb], V)
        got_h, got_s = halves_and_scales(y[r * rb:(r + 1) * rb], V)
        v = s[:, None] * h.astype(np.float32)
        m = np.abs(v).max(axis=1)
        want = (v / m[:, None]).astype(np.float16)
        assert np.array_equal(got_s.view(np.uint32), m.view(np.uint32))
        # values (a zero of either sign may follow from the sums; its sign is the next test)
        assert np.array_equal(got_h, want)


@pytest.mark.parametrize("n", [1, 3])
def test_store_keeps_the_sign_of_zero(n):
    need_gpu()
    dims = (8, 8, 16, 16)
    V = int(np.prod(dims))
    # component 0 has a negative zero as its real part; with real parts below and imaginary parts above zero in the
    # others every term that the operator adds to it is a negative zero too
    re, im = np.full((n, V, 12), -0.5), np.full((n, V, 12), 0.25)
    re[..., 0] = -0.0
    psi = torch.empty((n, V, 12), dtype=torch.complex128)
    torch.view_as_real(psi)[..., 0] = torch.from_numpy(re)
    torch.view_as_real(psi)[..., 1] = torch.from_numpy(im)
    op = identity(dims)
    x = op.pack(psi.cuda(), "f16s")
    y = op.empty("f16s", n).zero_()
    op.apply_native(y, x, n, "f16s")
    rb = op.field_bytes("f16s", 1)
    for r in range(n):
        h, _ = halves_and_scales(x[r * rb:(r + 1) * rb], V)
        assert np.all(h[:, 0].view(np.uint16) == 0x8000)  # as packed
        got, _ = halves_and_scales(y[r * rb:(r + 1) * rb], V)
        assert np.all(got[:, 0].view(np.uint16) == 0x8000)
        assert np.array_equal(got, h)
