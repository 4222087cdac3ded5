"""Values that are no finite numbers (NaN of both kinds, infinities) in the quantisers' and SiLU * up's inputs: what the definitions
of Appendix A.1 and of SiLU give for the numbers beside them, on every kernel that quantises."""
import numpy as np
import pytest

from oracle import oracle as O
from test_gpu_parity import dev, host, rand_quantised

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

QUIET, SIGNALLING = 0x7E00, 0x7C01


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_14597_amd as pkg
    pkg.load_library()
    return pkg


def with_nan(x, where, pattern=QUIET):
    """The array with the NaN of this bit pattern in the places `where`."""
    bits = np.ascontiguousarray(x).view(np.uint16).copy()
    bits[where] = pattern
    return bits.view(np.float16)


# groups of 128 take the kernel of whole rows, groups of 1024 the kernels in steps; an amplifier that is searched for takes the
# latter for every group
@pytest.mark.parametrize("group,alpha", [(128, 10), (32, 10), (1024, 10), (128, -1)])
@pytest.mark.parametrize("bits", [4, 8])
def test_weight_groups_with_sixteen_bytes_of_nan(P, bits, group, alpha):
    """A NaN takes no part in its group's maximum: the scale and the other codes are those of the numbers, the NaN gets the lowest
    code."""
    rng = np.random.default_rng(bits + group)
    w = (rng.standard_normal((5, 2048)) * 0.02).astype(np.float16)
    hole = np.zeros(w.shape, bool)
    hole[1, 8:16] = hole[3, 1024:1040] = True
    oracle = O.quantize_weights_int4_group if bits == 4 else O.quantize_weights_int8_group
    ref = oracle(np.where(hole, np.float16(0), w), group, alpha, O.SCALE_NORM)
    quantise = P.is_quantize_weights_int4_group if bits == 4 else P.is_quantize_weights_int8_group
    got = quantise(dev(with_nan(w, hole)), group, alpha, P.IS_SCALE_NORM)
    assert np.array_equal(host(got.scale_f32), ref.scale_f32) and np.array_equal(host(got.scale_i32), ref.scale_i32)
    assert np.array_equal(host(got.chan_scale), ref.chan_scale)
    codes = O.unpack_int4(host(got.qweight)) if bits == 4 else host(got.qweight)
    codes_ref = O.unpack_int4(ref[0]) if bits == 4 else ref[0]
    assert np.array_equal(codes[~hole], codes_ref[~hole])
    assert (codes[hole] == (-8 if bits == 4 else -128)).all()


@pytest.mark.parametrize("K", [64, 4096, 40960])
def test_signalling_nan_beside_the_largest_value(P, K):
    """A signalling NaN takes no part in the row's maximum, and no neighbour with it: in every place of an 8-value chunk, next to
    the row's largest value in every other place."""
    rng = np.random.default_rng(K)
    places = [(i, j) for i in range(8) for j in range(8) if i != j]
    x = rng.uniform(-1.0, 1.0, size=(len(places), K)).astype(np.float16)
    hole = np.zeros(x.shape, bool)
    for m, (i, j) in enumerate(places):
        chunk = 8 * int(rng.integers(0, K // 8))
        x[m, chunk + i] = 100.0
        hole[m, chunk + j] = True
    xq_ref, sa_ref = O.quantize_act_int8_token(np.where(hole, np.float16(0), x))
    xq, sa = P.is_quantize_act_int8_token(dev(with_nan(x, hole, SIGNALLING)))
    assert np.array_equal(host(sa), sa_ref)
    assert np.array_equal(host(xq)[~hole], xq_ref[~hole]) and (host(xq)[hole] == -128).all()
    w = with_nan(x[:, :64], hole[:, :64], SIGNALLING)
    ref = O.quantize_weights_int4_group(np.where(hole[:, :64], np.float16(0), x[:, :64]), 32, 10, O.SCALE_NORM)
    got = P.is_quantize_weights_int4_group(dev(w), 32, 10, P.IS_SCALE_NORM)
    assert np.array_equal(host(got.scale_f32), ref.scale_f32)


@pytest.mark.parametrize("M", [5, 300])
@pytest.mark.parametrize("K", [64, 4096, 16384, 40960])
def test_rows_of_zeros_and_nan(P, M, K):
    """A row whose numbers are all zero has scale 0, and then every code is 0, a NaN's too (stand-alone quantiser and both
    producers, rows that stay in registers and longer ones)."""
    x = np.random.default_rng(K).standard_normal((M, K)).astype(np.float16)
    x[2] = 0
    hole = np.zeros(x.shape, bool)
    hole[2, [0, 9, K - 1]] = True
    x = with_nan(x, hole)
    xq, sa = P.is_quantize_act_int8_token(dev(x))
    assert host(sa)[2] == 0 and not host(xq)[2].any() and host(sa)[3] > 0 and host(xq)[3].any()
    gu = np.concatenate([np.where(hole, np.float16(0), x), np.ones_like(x)], axis=1)
    gu[:, K:][hole] = np.nan                                            # SiLU(0) * NaN beside SiLU(0) * 1
    xq, sa = P.is_silu_mul_quantize_act_int8_token(dev(gu))
    assert host(sa)[2] == 0 and not host(xq)[2].any() and host(xq)[3].any()
    xq, sa = P.is_rmsnorm_quantize_act_int8_token(dev(x), dev(np.ones(K, np.float16)), 1e-5)   # NaN in every place of the row
    assert host(sa)[2] == 0 and not host(xq)[2].any() and host(xq)[3].any()


@pytest.mark.parametrize("M", [1, 5, 70, 600])
@pytest.mark.parametrize("K", [1024, 4096])
def test_linear_calls_on_rows_of_zeros_and_nan(P, M, K):
    """The same inside the linear calls: the accumulators of such a row are 0."""
    N = 272
    _, qw, IS, _, _, c = rand_quantised(np.random.default_rng(M + K), 1, N, K)
    x = np.random.default_rng(M).standard_normal((M, K)).astype(np.float16)
    x[M // 2] = 0
    hole = np.zeros(x.shape, bool)
    hole[M // 2, [0, 77, K - 1]] = True
    x = dev(with_nan(x, hole))
    _, acc = P.is_linear_w4a8_intscale_prepacked(x, P.is_prepack_w4(dev(qw), dev(IS), 128), dev(c), 10, want_acc=True)
    assert not host(acc)[M // 2].any()
    _, acc = P.is_linear_w4a8_intscale(x, dev(qw), dev(IS), dev(c), 128, 10, want_acc=True)
    assert not host(acc)[M // 2].any()


@pytest.mark.parametrize("bits", [4, 8])
def test_weight_groups_of_zeros_and_nan(P, bits):
    w = np.random.default_rng(3).standard_normal((3, 1024)).astype(np.float16)
    w[1, 256:384] = 0
    hole = np.zeros(w.shape, bool)
    hole[1, [256, 300]] = True
    quantise = P.is_quantize_weights_int4_group if bits == 4 else P.is_quantize_weights_int8_group
    for alpha in (10, -1):
        got = quantise(dev(with_nan(w, hole)), 128, alpha, P.IS_SCALE_NORM)
        codes = O.unpack_int4(host(got.qweight)) if bits == 4 else host(got.qweight)
        assert host(got.scale_f32)[1, 2] == 0 and not codes[1, 256:384].any()


@pytest.mark.parametrize("up", [np.inf, -np.inf, 65504.0, -65504.0, 0.0, np.nan])
def test_silu_mul_on_every_gate_pattern(P, up):
    """All 65536 gates, infinities and NaN among them, against up values at the ends of the type: infinite products are infinite
    (also where SiLU is far below the smallest fp16 value), products that are no numbers leave a row of zeros."""
    g = np.arange(65536, dtype=np.uint16).view(np.float16)
    gu = np.concatenate([np.repeat(g[:, None], 8, axis=1), np.full((g.size, 8), up, np.float16)], axis=1)
    with np.errstate(invalid="ignore", over="ignore"):
        h = O.silu_mul_fp16(gu)[:, 0].astype(np.float32)
    amax = np.where(np.isnan(h), np.float32(0), np.abs(h))
    xq, sa = P.is_silu_mul_quantize_act_int8_token(dev(gu))
    assert np.array_equal(host(sa), amax / np.float32(127.0))
    code = np.where(amax == 0, 0, np.where(np.isinf(h), -128, np.sign(np.nan_to_num(h)) * 127)).astype(np.int8)
    assert np.array_equal(host(xq), np.repeat(code[:, None], 8, axis=1))
