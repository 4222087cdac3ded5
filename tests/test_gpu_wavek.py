"""GPU parity of the kernel whose waves split K (prepacked and W8A8 calls of a moderate number of token rows) against the CPU
oracle: row tiles of 48 and 64 rows with remainders, fewer K steps than waves, workgroups of four and eight waves, ragged
widths, wide groups, wide scales, the float-scale twin, prepared activations and captured calls.  (Its SiLU * up epilogue is in
test_gpu_gate_up.py.)"""
import numpy as np
import pytest

from oracle import oracle as O
import test_gpu_few as few
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
    # (integer scales on codes go without a preparation from K = 2048 on; on prepared activations this kernel takes them as well)
    for int_scale in (K < 2048, False):
        names = P.is_describe_prepacked(M, N, K, group, int_scale)
        assert names == ["prepare_activations_pk_kernel", f"gemm_wavek_kernel<{str(int_scale).lower()}, false, {shape}, false>"]
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
        again, acc = P.is_gemm_w4a8_intscale_prepacked_prepared(dev(sa), pk, cd, a, workspace=ws, want_acc=True)
        assert torch.equal(out, again) and np.array_equal(host(acc), ref.acc)
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
    nbytes = P.is_gemm_w8a8_workspace_bytes(M, N, K, group)
    blocks = torch.zeros((max(nbytes, P.is_gemm_prepacked_workspace_bytes(M, N, K, group)),), dtype=torch.uint8, device="cuda:0")
    P.is_prepare_activations_prepacked(dev(xq), blocks)
    blocks = blocks[:(M + 15) // 16 * 16 * K]   # what only the kernel whose waves split K leaves in the workspace
    before = P.is_set_kernel_route("tiled")
    tiled_bytes = P.is_gemm_w8a8_workspace_bytes(M, N, K, group)
    P.is_set_kernel_route(before)
    assert nbytes >= tiled_bytes
    for scales in (IS, wide):
        ref = O.gemm_w8a8_intscale(xq, sa, q, scales, None, group, 12)
        outs = []
        for route, ws_bytes in (("auto", nbytes), ("tiled", tiled_bytes)):
            P.is_set_kernel_route(route)
            ws = torch.full((ws_bytes,), 0x5A, dtype=torch.uint8, device="cuda:0")
            out, acc = P.is_gemm_w8a8_intscale(dev(xq), dev(sa), dev(q), dev(scales), None, group, 12, want_acc=True, workspace=ws)
            P.is_set_kernel_route(before)
            assert (ws.numel() >= blocks.numel() and torch.equal(ws[:blocks.numel()], blocks)) == (route == "auto")
            assert np.array_equal(host(acc), ref.acc), "int32 accumulators differ"
            outs.append(out)
        assert torch.equal(outs[0], outs[1])
    s = (rng.random((N, K // group)) * 1e-4).astype(np.float32)
    fs = O.gemm_w8a8_floatscale(xq, sa, q, s, group)
    check_fs(host(P.is_gemm_w8a8_floatscale(dev(xq), dev(sa), dev(q), dev(s), group)), fs, f"M{M} N{N} K{K}")


# row tiles of 80 rows: workgroups of eight waves, whose partial sums meet in two passes, and of four; the last row tile part filled
EIGHTY = [(675, 1500, 2688, 384, "5, 8"), (530, 2048, 2688, 128, "5, 8"), (515, 4100, 2048, 256, "5, 4"), (645, 3008, 2048, 128, "5, 4")]


@pytest.mark.parametrize("M,N,K,group,shape", EIGHTY)
@pytest.mark.parametrize("wide", [False, True])
def test_wavek_tiles_of_80_rows(P, M, N, K, group, shape, wide):
    for int_scale in (True, False):
        name = P.is_describe_prepacked(M, N, K, group, int_scale)[-1]
        assert name == f"gemm_wavek_kernel<{str(int_scale).lower()}, false, {shape}, false>"
    few.check_call(P, M, N, K, group, wide, chan=not wide)


@pytest.mark.parametrize("M,inter,K,shape", [(530, 1024, 2688, "5, 8"), (645, 1504, 2048, "5, 4")])
def test_wavek_tiles_of_80_rows_fused_gate_up(P, M, inter, K, shape):
    for int_scale in (True, False):
        assert P.is_describe_prepacked(M, 2 * inter, K, 128, int_scale)[-1] == f"gemm_wavek_kernel<{str(int_scale).lower()}, false, {shape}, false>"
    few.test_fused_gate_up(P, M, inter, K)
    few.test_fused_gate_up_float_sums_in_one_order(P, M, inter, K)


@pytest.mark.parametrize("M,N,K,group", [(65, 8200, 2688, 384), (195, 4100, 2688, 128)])
@pytest.mark.parametrize("wide", [False, True])
def test_wavek_w8_tiles_of_80_rows(P, M, N, K, group, wide):
    xq, _, _, scale, sa, c = few.case(M, N, K, group, wide, seed=8)
    q = torch.randint(-128, 128, (N, K), generator=torch.Generator(device="cuda:0").manual_seed(N + K), device="cuda:0", dtype=torch.int8)
    acc = few.wrapped(few.reference(xq, q, scale, group))
    ws = torch.full((P.is_gemm_w8a8_workspace_bytes(M, N, K, group),), 0x5A, dtype=torch.uint8, device="cuda:0")
    out, got = P.is_gemm_w8a8_intscale(xq, sa * 2.0 ** -6, q, scale, c, group, 10, want_acc=True, workspace=ws)
    assert torch.equal(got, acc), "int32 accumulators"
    blocks = torch.zeros((P.is_gemm_prepacked_workspace_bytes(M, N, K, group),), dtype=torch.uint8, device="cuda:0")
    P.is_prepare_activations_prepacked(xq, blocks)
    blocks = blocks[:(M + 15) // 16 * 16 * K]
    assert torch.equal(ws[:blocks.numel()], blocks), "the kernel whose waves split K"
    before = P.is_set_kernel_route("tiled")
    try:
        tiled, tiled_acc = P.is_gemm_w8a8_intscale(xq, sa * 2.0 ** -6, q, scale, c, group, 10, want_acc=True)
    finally:
        P.is_set_kernel_route(before)
    assert torch.equal(tiled_acc, got) and torch.equal(tiled, out)
    s = scale.float() * (2.0 ** -32 if wide else 2.0 ** -23)
    fs = few.reference(xq, q, s, group) * sa.double()[:, None]
    size = few.reference(xq.abs().clamp(max=127), q.abs().clamp(max=127), s.abs(), group) * sa.double()[:, None]
    fout = P.is_gemm_w8a8_floatscale(xq, sa, q, s, group)
    # (as for the other recipe: the sum of K / group products in fp32; magnitudes clamped at 127 for 128, hence the hundredth)
    bound = 5e-4 * fs.abs() + 2.0 ** -25 + 1.02 * size * (K // group + 2) * 2.0 ** -24
    assert bool(((fout.double() - fs).abs() <= bound)[fs.abs() < 65000.0].all())


def test_w8_workspace_of_the_tiled_kernel_is_enough(P):
    """A workspace of the size that the tiled kernel alone needs keeps the call there, with the same integer results."""
    M, N, K, group = 97, 33, 1152, 128
    rng = np.random.default_rng(6900)
    xq = rng.integers(-128, 128, size=(M, K)).astype(np.int8)
    q = rng.integers(-128, 128, size=(N, K)).astype(np.int8)
    sa = (rng.random(M) + 0.01).astype(np.float32)
    IS = rng.integers(-2 ** 22, 2 ** 22, size=(N, K // group)).astype(np.int32)
    before = P.is_set_kernel_route("tiled")
    tiled_bytes = P.is_gemm_w8a8_workspace_bytes(M, N, K, group)
    P.is_set_kernel_route(before)
    assert P.is_gemm_w8a8_workspace_bytes(M, N, K, group) > tiled_bytes
    ws = torch.full((tiled_bytes,), 0x5A, dtype=torch.uint8, device="cuda:0")
    small, acc = P.is_gemm_w8a8_intscale(dev(xq), dev(sa), dev(q), dev(IS), None, group, 12, want_acc=True, workspace=ws)
    full, _ = P.is_gemm_w8a8_intscale(dev(xq), dev(sa), dev(q), dev(IS), None, group, 12)
    assert torch.equal(small, full)
    assert np.array_equal(host(acc), O.gemm_w8a8_intscale(xq, sa, q, IS, None, group, 12).acc)


def test_captured_calls(P):
    """A linear call on fp16 rows, a GEMM on codes and a W8A8 GEMM on this kernel in one graph, replayed with new inputs in the
    same buffers and with the program's own work between the replays: the results of the ordinary calls each time."""
    M, N, K = 130, 328, 1152
    assert P.is_describe_prepacked(M, N, K, 128)[-1].startswith("gemm_wavek_kernel<true, ")
    rng = np.random.default_rng(7100)
    _, qw, IS, _, sa, c = rand_quantised(rng, M, N, K)
    pk = P.is_prepack_w4(dev(qw), dev(IS), 128)
    q8, IS8 = dev(rng.integers(-128, 128, size=(N, K)).astype(np.int8)), dev(rng.integers(0, 1025, size=(N, K // 128)).astype(np.int32))
    c, sa = dev(c), dev(sa)
    x, xq = torch.zeros((M, K), dtype=torch.float16, device="cuda:0"), torch.zeros((M, K), dtype=torch.int8, device="cuda:0")
    outs = [torch.zeros((M, N), dtype=torch.float16, device="cuda:0") for _ in range(3)]
    ws = [torch.zeros((n,), dtype=torch.uint8, device="cuda:0") for n in (P.is_linear_prepacked_workspace_bytes(M, N, K, 128),
          P.is_gemm_prepacked_workspace_bytes(M, N, K, 128), P.is_gemm_w8a8_workspace_bytes(M, N, K, 128))]

    def calls(outs, ws):
        P.is_linear_w4a8_intscale_prepacked(x, pk, c, 10, out=outs[0], workspace=ws[0])
        P.is_gemm_w4a8_intscale_prepacked(xq, sa, pk, c, 10, out=outs[1], workspace=ws[1])
        P.is_gemm_w8a8_intscale(xq, sa, q8, IS8, c, 128, 10, out=outs[2], workspace=ws[2])

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        calls(outs, ws)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls(outs, ws)
    for i in range(4):
        x.copy_(torch.randn((M, K), device="cuda:0").half())
        xq.copy_(torch.randint(-128, 128, (M, K), dtype=torch.int8, device="cuda:0"))
        graph.replay()
        torch.cuda.synchronize()
        want = [torch.empty_like(o) for o in outs]
        calls(want, [torch.full_like(w, 0x5A) for w in ws])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, want)), f"replay {i}"
