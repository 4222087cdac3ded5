"""GPU parity of the kernel whose waves split K (prepacked calls of a moderate number of token rows) against the CPU oracle:
row tiles of 48 and 64 rows with remainders, fewer K steps than waves, workgroups of four and eight waves, ragged widths,
wide groups, wide scales, the float-scale twin, the SiLU * up epilogue, prepared activations and captured calls."""
import numpy as np
import pytest

from oracle import oracle as O
from test_gpu_parity import check_fs, check_out, dev, host, rand_quantised

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_14597_amd as pkg
    pkg.load_library()
    return pkg


# 65, 96 and 129 rows: tiles of 48; 128, 200, 250, 305: 64, most with a remainder; 5 K steps leave waves of eight without
# work; the widest calls run workgroups of four waves, the others of eight; widths that are no multiple of 8, 16 or 64
@pytest.mark.parametrize("M,N,K,group,shape", [(65, 300, 640, 128, "3, 8"), (96, 5003, 768, 128, "3, 8"), (129, 72, 640, 128, "3, 8"),
                                               (128, 264, 1024, 256, "4, 8"), (200, 1041, 2048, 1024, "3, 8"),
                                               (250, 64, 4096, 128, "4, 8"), (305, 4100, 1024, 128, "4, 4"),
                                               (65, 17001, 640, 128, "3, 4")])
def test_wavek_gemm(P, M, N, K, group, shape):
    names = P.is_describe_prepacked(M, N, K, group)
    assert names == ["prepare_activations_pk_kernel", f"gemm_wavek_kernel<true, false, {shape}, false>"]
    rng = np.random.default_rng(6000 + M + N + K)
    xq, qw, IS, s, sa, c = rand_quantised(rng, M, N, K)
    IS, s = np.ascontiguousarray(IS[:, :K // group]), np.ascontiguousarray(s[:, :K // group])
    xq[0], xq[M - 1] = -128, 127
    wide = rng.integers(-2 ** 31, 2 ** 31, size=IS.shape, dtype=np.int64).astype(np.int32)
    for scales, chan, a in ((IS, c, 10), (wide, None, 7)):
        ref = O.gemm_w4a8_intscale(xq, sa, qw, scales, chan, group, a)
        pk = P.is_prepack_w4(dev(qw), dev(scales), group)
        cd = None if chan is None else dev(chan)
        ws = torch.full((P.is_gemm_prepacked_workspace_bytes(M, N, K, group),), 0x5A, dtype=torch.uint8, device="cuda:0")
        out, acc = P.is_gemm_w4a8_intscale_prepacked(dev(xq), dev(sa), pk, cd, a, want_acc=True, workspace=ws)
        assert np.array_equal(host(acc), ref.acc), "int32 accumulators differ"
        check_out(host(out), ref.out, f"M{M} N{N} K{K}")
        P.is_prepare_activations_prepacked(dev(xq), ws)
        again, _ = P.is_gemm_w4a8_intscale_prepacked_prepared(dev(sa), pk, cd, a, workspace=ws)
        assert torch.equal(out, again)
    fs = O.gemm_w4a8_floatscale(xq, sa, qw, s, group)
    got = P.is_gemm_w4a8_floatscale_prepacked(dev(xq), dev(sa), P.is_prepack_w4(dev(qw), dev(s), group))
    check_fs(host(got), fs, f"M{M} N{N} K{K}")


def test_wavek_is_the_tiled_kernel_bit_for_bit(P):
    """Integer sums do not depend on their order: both kernels give the same fp16 outputs, from codes and from fp16 rows."""
    M, N, K = 93, 1003, 1152
    rng = np.random.default_rng(6500)
    xq, qw, IS, s, sa, c = rand_quantised(rng, M, N, K)
    x = torch.randn((M, K), device="cuda:0", dtype=torch.float16)
    pk = P.is_prepack_w4(dev(qw), dev(IS), 128)
    got = {}
    for route in ("auto", "tiled64"):
        before = P.is_set_kernel_route(route)
        out, _ = P.is_gemm_w4a8_intscale_prepacked(dev(xq), dev(sa), pk, dev(c), 10)
        got[route] = (out, P.is_linear_w4a8_intscale_prepacked(x, pk, dev(c), 10)[0])
        P.is_set_kernel_route(before)
    assert torch.equal(got["auto"][0], got["tiled64"][0]) and torch.equal(got["auto"][1], got["tiled64"][1])


# int8 weights: a matrix of few short rows (repeated rows behind the last one), 3 and 9 K steps (waves without work, quads of
# scales that end in mid-run), row tiles of 48 and 64 rows, workgroups of four and eight waves, wide groups
@pytest.mark.parametrize("M,N,K,group", [(70, 10, 128, 128), (97, 1, 384, 128), (130, 300, 1152, 128), (250, 4100, 1280, 256),
                                         (70, 9001, 640, 128)])
def test_wavek_w8(P, M, N, K, group):
    rng = np.random.default_rng(6800 + M + N + K)
    xq = rng.integers(-128, 128, size=(M, K)).astype(np.int8)
    q = rng.integers(-128, 128, size=(N, K)).astype(np.int8)
    xq[0], q[0], xq[M - 1] = -128, -128, 127
    sa = (rng.random(M) + 0.01).astype(np.float32)
    IS = rng.integers(-2 ** 22, 2 ** 22, size=(N, K // group)).astype(np.int32)
    wide = IS.copy()
    wide[N // 2, -1] = 2 ** 23  # one scale beyond 24 signed bits
    before = P.is_set_kernel_route("tiled")
    tiled_bytes = P.is_gemm_w8a8_workspace_bytes(M, N, K, group)
    P.is_set_kernel_route(before)
    assert P.is_gemm_w8a8_workspace_bytes(M, N, K, group) >= tiled_bytes
    for scales in (IS, wide):
        ref = O.gemm_w8a8_intscale(xq, sa, q, scales, None, group, 12)
        outs = []
        for nbytes in (tiled_bytes, max(tiled_bytes, P.is_gemm_w8a8_workspace_bytes(M, N, K, group))):  # tiled kernel, this one
            ws = torch.full((nbytes,), 0x5A, dtype=torch.uint8, device="cuda:0")
            out, acc = P.is_gemm_w8a8_intscale(dev(xq), dev(sa), dev(q), dev(scales), None, group, 12, want_acc=True, workspace=ws)
            assert np.array_equal(host(acc), ref.acc), "int32 accumulators differ"
            outs.append(out)
        assert torch.equal(outs[0], outs[1])
    s = (rng.random((N, K // group)) * 1e-4).astype(np.float32)
    fs = O.gemm_w8a8_floatscale(xq, sa, q, s, group)
    check_fs(host(P.is_gemm_w8a8_floatscale(dev(xq), dev(sa), dev(q), dev(s), group)), fs, f"M{M} N{N} K{K}")
