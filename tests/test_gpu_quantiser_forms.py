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


@pytest.mark.parametrize("N,K,group", [(3, 128, 128), (130, 1024, 128), (5, 33792, 128), (9, 4096, 32), (70, 192, 64), (17, 2048, 256),
                                       (6, 3584, 512), (2, 131072, 64), (2, 1 << 18, 64), (11, 960, 24), (5, 1024, 1024),
                                       (100, 33792, 128), (96, 20480, 32), (5001, 128, 64), (2100, 384, 128)])
@pytest.mark.parametrize("bits", [4, 8])
def test_weight_codes_and_scales(P, N, K, group, bits):
    """One pass over whole rows (the last four: several rounds of loads a row, several rows a workgroup), and the shapes it leaves to
    the kernels in steps (few long rows, rows of more scales than LDS holds, groups that are no power of two, groups beyond 512)."""
    rng = np.random.default_rng(N + K + group)
    w = (rng.standard_normal((N, K)) * 0.02).astype(np.float16)
    w[0, :group] = 0                                                 # a group of zeros
    hi = 7 if bits == 4 else 127
    amax = np.abs(w[N - 1]).reshape(-1, group).max(axis=1).astype(np.float32)
    half = (rng.integers(-hi, hi, size=(K // group, group)) + 0.5) * (amax / np.float32(hi)).astype(np.float64)[:, None]
    half[:, 0] = amax
    w[N - 1] = np.clip(half.astype(np.float16), -amax[:, None].astype(np.float16), amax[:, None].astype(np.float16)).reshape(-1)
    quantise = P.is_quantize_weights_int4_group if bits == 4 else P.is_quantize_weights_int8_group
    oracle = O.quantize_weights_int4_group if bits == 4 else O.quantize_weights_int8_group
    for mode in (O.SCALE_RAW, O.SCALE_NORM):
        got, ref = quantise(dev(w), group, 10, mode), oracle(w, group, 10, mode)
        assert np.array_equal(host(got.scale_f32), ref.scale_f32) and np.array_equal(host(got.qweight), ref[0])
        assert np.array_equal(host(got.scale_i32), ref.scale_i32) and np.array_equal(host(got.chan_scale), ref.chan_scale)
        assert host(got.alpha_log2_dev)[0] == 10
