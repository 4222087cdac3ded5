"""The short forms of the quantisers and of SiLU against their definitions: codes next to rounding boundaries (where the
two-neighbour test has to send the wave to the true division), values that are no numbers, and SiLU * up on every fp16
value of the gate."""
import numpy as np
import pytest

from oracle import oracle as O
from test_gpu_parity import dev, host

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_14597_amd as pkg
    pkg.load_library()
    return pkg


@pytest.mark.parametrize("K", [8, 520, 4096, 8192, 40960])
def test_codes_next_to_rounding_boundaries(P, K):
    rng = np.random.default_rng(K)
    M = 24
    amax = rng.uniform(0.01, 300.0, size=(M, 1)).astype(np.float16)
    s = amax.astype(np.float32) / np.float32(127.0)
    k = rng.integers(-127, 127, size=(M, K))
    x = ((k + 0.5) * s.astype(np.float64)).astype(np.float16)       # as close to (k + 1/2) s as fp16 allows,
    step = rng.integers(-1, 2, size=(M, K))                          # and its neighbours on both sides
    x = np.where(step > 0, np.nextafter(x, np.float16(np.inf)), np.where(step < 0, np.nextafter(x, np.float16(-np.inf)), x))
    x = np.clip(x, -amax, amax)
    x[:, K // 2:K // 2 + 1] = amax
    x[0] = 0                                                        # a row of zeros
    xq, sa = P.is_quantize_act_int8_token(dev(x))
    ref, ref_s = O.quantize_act_int8_token(x)
    assert np.array_equal(host(sa), ref_s) and np.array_equal(host(xq), ref)


def test_codes_of_values_that_are_no_numbers(P):
    """As the clamp of the quotient gives them: a NaN the lowest code, and in a row with an infinity (scale: infinity) the
    finite values 0."""
    x = np.ones((2, 64), np.float16)
    x[0, 5] = np.nan
    x[1, 7] = np.inf
    xq, sa = P.is_quantize_act_int8_token(dev(x))
    xq, sa = host(xq), host(sa)
    assert sa[0] == np.float32(1.0) / np.float32(127.0) and np.isinf(sa[1])
    assert xq[0, 5] == -128 and (np.delete(xq[0], 5) == 127).all()
    assert xq[1, 7] == -128 and (np.delete(xq[1], 7) == 0).all()


def test_silu_mul_on_every_gate_value(P):
    """One row of eight equal products per fp16 gate value: the token scale shows the product's magnitude exactly, the
    codes its sign."""
    g = np.arange(65536, dtype=np.uint16).view(np.float16)
    g = g[np.isfinite(g)]
    u = np.random.default_rng(3).uniform(0.25, 1.0, size=g.size).astype(np.float16)
    u[::7] *= -1
    gu = np.concatenate([np.repeat(g[:, None], 8, axis=1), np.repeat(u[:, None], 8, axis=1)], axis=1)
    xq, sa = P.is_silu_mul_quantize_act_int8_token(dev(gu))
    h = O.silu_mul_fp16(gu)
    ref, ref_s = O.quantize_act_int8_token(h)
    assert np.array_equal(host(sa), ref_s) and np.array_equal(host(xq), ref)
