"""The kernel for 2 to 64 token rows whose waves split K: one small call per instance that the library can pick, ragged rows and
columns, short and uneven runs of K steps, groups of several steps, scales beyond 24 bits, the fused SiLU * up epilogue.  The reference
is the same sums in plain PyTorch (exact in float64: a group's partial sum is below 2^22, its product with a scale below 2^53)."""
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu

G = 128


@pytest.fixture(scope="module")
def P():
    import paper_2405_14597_amd as P
    P.load_library()
    return P


def smallest_shape_per_instance():
    import paper_2405_14597_amd as P
    best = {}
    for M in (2, 16, 17, 32, 33, 48, 49, 64):
        for N in (20, 1000, 4100, 8184, 12280, 16376, 20472, 22000, 24568, 28664):
            for K in (128, 256, 640, 1024, 3072, 4224, 8192, 12288, 14336, 16384):
                name = P.is_describe_prepacked(M, N, K, G)[-1]
                if name.startswith("gemm_few_pk_kernel<") and N * K < best.get(name, (0, 1 << 60))[1]:
                    best[name] = ((M, N, K), N * K)
    return [(name, *shape) for name, (shape, _) in sorted(best.items())]


def reference(xq, q, scale, group):
    """Sum over the groups of (integer partial sum) * scale, in float64."""
    acc = torch.zeros((xq.shape[0], q.shape[0]), dtype=torch.float64, device=xq.device)
    for g in range(xq.shape[1] // group):
        cut = slice(g * group, (g + 1) * group)
        acc += (xq[:, cut].double() @ q[:, cut].double().t().contiguous()) * scale[:, g].double()
    return acc


def case(M, N, K, group=G, wide=False, seed=0):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(1000 * seed + M + N + K)
    xq = torch.randint(-128, 128, (M, K), generator=gen, device="cuda:0", dtype=torch.int8)
    q = torch.randint(-8, 8, (N, K), generator=gen, device="cuda:0", dtype=torch.int32)
    qw = ((q[:, 0::2] & 15) | ((q[:, 1::2] & 15) << 4)).to(torch.uint8).contiguous()
    scale = torch.randint(0, 1025, (N, K // group), generator=gen, device="cuda:0", dtype=torch.int32)
    if wide:
        scale[N // 2, -1] = 2 ** 25
        scale[0, 0] = -(2 ** 23) - 1
    sa = torch.rand((M,), generator=gen, device="cuda:0") + 0.1
    c = torch.rand((N,), generator=gen, device="cuda:0") + 0.5
    return xq, q, qw, scale, sa, c


def wrapped(acc):
    return ((acc.long() + 2 ** 31) % 2 ** 32 - 2 ** 31).to(torch.int32)


def check_call(P, M, N, K, group=G, wide=False, chan=True):
    xq, q, qw, scale, sa, c = case(M, N, K, group, wide)
    acc = wrapped(reference(xq, q, scale, group))
    cc = c if chan else None
    out, got = P.is_gemm_w4a8_intscale_prepacked(xq, sa, P.is_prepack_w4(qw, scale, group), cc, 10, want_acc=True)
    assert torch.equal(got, acc), "int32 accumulators"
    want = acc.double() * sa.double()[:, None] * (c.double()[None, :] if chan else 1.0) / 1024.0
    ok = want.abs() < 65000.0
    # two fp32 products and one rounding to fp16: 2^-11 of the value and a little more, and half a step of the smallest numbers
    assert bool(((out.double() - want).abs() <= 5e-4 * want.abs() + 2.0 ** -25)[ok].all())
    again, _ = P.is_gemm_w4a8_intscale_prepacked(xq, sa, P.is_prepack_w4(qw, scale, group), cc, 10)
    assert torch.equal(again, out)
    s32 = scale.float() * (2.0 ** -17 if not wide else 2.0 ** -32)
    fout = P.is_gemm_w4a8_floatscale_prepacked(xq, sa, P.is_prepack_w4(qw, s32, group))
    fs = reference(xq, q, s32, group) * sa.double()[:, None]
    size = reference(xq.abs().clamp(max=127), q.abs(), s32.abs(), group) * sa.double()[:, None]
    # (the sum of K / group products in fp32: their sizes times 2^-24 each and per addition)
    bound = 5e-4 * fs.abs() + 2.0 ** -25 + size * (K // group + 2) * 2.0 ** -24
    assert bool(((fout.double() - fs).abs() <= bound)[fs.abs() < 65000.0].all())


@pytest.mark.parametrize("name,M,N,K", smallest_shape_per_instance())
def test_every_instance(P, name, M, N, K):
    assert P.is_describe_prepacked(M, N, K, G)[-1] == name
    check_call(P, M, N, K)


@pytest.mark.parametrize("M,N,K,group", [(2, 16, 128, 128), (3, 17, 384, 384), (31, 300, 1536, 512), (64, 1003, 1152, 384), (50, 97, 1152, 1152),
                                         (16, 2050, 12288, 256), (33, 40, 14336, 256)])
@pytest.mark.parametrize("wide", [False, True])
def test_groups_ragged_sizes_and_wide_scales(P, M, N, K, group, wide):
    check_call(P, M, N, K, group, wide, chan=not wide)


# narrow matrices with a long K stay on the kernel that cuts K over workgroups
@pytest.mark.parametrize("M,N,K", [(2, 20, 65536), (8, 64, 32768), (16, 300, 65536), (17, 33, 65536), (32, 528, 65536), (33, 48, 28672), (64, 512, 28672)])
@pytest.mark.parametrize("wide", [False, True])
def test_narrow_matrices_with_a_long_k(P, M, N, K, wide):
    assert P.is_gemm_prepacked_workspace_bytes(M, N, K, G) > 0 and P.is_describe_prepacked(M, N, K, G)[-1].startswith("gemm_decode_pk_kernel<")
    check_call(P, M, N, K, wide=wide)


@pytest.mark.parametrize("M,inter,K", [(2, 16, 128), (16, 48, 1024), (17, 1200, 512), (40, 5504, 256), (64, 2064, 4096), (9, 14336, 256)])
def test_fused_gate_up(P, M, inter, K):
    """The epilogue gives the bits of the GEMM's fp16 outputs taken through SiLU * up (the quantiser of that product, on either)."""
    xq, q, qw, scale, sa, c = case(M, 2 * inter, K, seed=3)
    sa = sa * 1e-3
    gu, _ = P.is_gemm_w4a8_intscale_prepacked(xq, sa, P.is_prepack_w4(qw, scale, G), c, 10)
    codes, s = P.is_silu_mul_quantize_act_int8_token(gu)
    packed = P.is_prepack_w4_gate_up(qw, scale, c, G)
    fused = P.is_gemm_w4a8_intscale_gate_up_silu_prepacked(xq, sa, packed, 10)
    fused = fused[0] if isinstance(fused, tuple) else fused
    codes_f, s_f = P.is_quantize_act_int8_token(fused)
    assert torch.equal(codes, codes_f) and torch.equal(s, s_f)
    g, u = gu[:, :inter].double(), gu[:, inter:].double()
    want = g / (1.0 + torch.exp(-g)) * u
    assert bool(((fused.double() - want).abs() <= 1e-3 * want.abs() + 2.0 ** -24)[want.abs() < 65000.0].all())


def order_shows(xq, q, scale, size):
    """Float scales (powers of two times `scale`) whose sums show their order: the first and the last group are alike but for the sign of a
    large scale, so that what is added between the two loses bits that depend on what."""
    xq[:, -G:] = xq[:, :G]
    q[:, -G:] = q[:, :G]
    s = scale.float() * size
    s[:, 0] = size * 2.0 ** 24
    s[:, -1] = -size * 2.0 ** 24
    return ((q[:, 0::2] & 15) | ((q[:, 1::2] & 15) << 4)).to(torch.uint8).contiguous(), s.contiguous()


# one row: K whose fused quantiser needs more waves than the sums would, a narrow matrix with a long K (K cut over workgroups)
@pytest.mark.parametrize("N,K", [(4096, 4096), (300, 11008), (12288, 4096), (64, 28672), (64, 32768), (16, 20480)])
def test_one_float_row_sums_in_one_order(P, N, K):
    """Float sums depend on their order: the linear call on one fp16 row gives the bits of the quantiser and the GEMM on its codes."""
    codes, q, _, scale, _, _ = case(1, N, K, seed=5)
    qw, s = order_shows(codes, q, scale, 2.0 ** -17)
    pk = P.is_prepack_w4(qw, s, G)
    x = codes.half()
    xq, sa = P.is_quantize_act_int8_token(x)
    assert torch.equal(P.is_linear_w4a8_floatscale_prepacked(x, pk), P.is_gemm_w4a8_floatscale_prepacked(xq, sa, pk))


# widths whose plain call takes an odd number of weight tiles a workgroup, or other waves, than the paired one; long runs of K steps
@pytest.mark.parametrize("M,inter,K", [(1, 2048, 4096), (8, 6144, 4096), (32, 6144, 4096), (16, 2048, 4096), (32, 2048, 8192), (64, 6144, 4096),
                                       (48, 2064, 11008), (5, 14336, 4096), (16, 64, 65536), (17, 11008, 4096)])
def test_fused_gate_up_float_sums_in_one_order(P, M, inter, K):
    """The fused epilogue works on the bits of the float-scale GEMM's own outputs."""
    xq, q, _, scale, sa, _ = case(M, 2 * inter, K, seed=6)
    qw, s = order_shows(xq, q, scale, 2.0 ** -24)
    gu = P.is_prepack_w4_gate_up(qw, s, None, G)
    fused = P.is_gemm_w4a8_floatscale_gate_up_silu_prepacked(xq, sa, gu)
    plain = P.is_gemm_w4a8_floatscale_prepacked(xq, sa, gu.packed).view(M, inter // 16, 2, 16)
    gate, up = plain[:, :, 0].reshape(M, inter), plain[:, :, 1].reshape(M, inter)
    want = O.silu_mul_fp16(torch.cat([gate, up], dim=1).cpu().numpy())
    assert bool((fused.cpu().numpy().view("uint16") == want.view("uint16")).all())


# experts without rows, with one, with more than a workgroup takes at a time (32 or 64), ragged widths, groups of several steps
GROUPED = [(1, [5], 100, 256, 128), (4, [0, 3, 16, 17], 300, 640, 128), (8, [0, 0, 40, 1, 0, 33, 0, 0], 1000, 1536, 384),
           (4, [70, 1, 0, 25], 520, 1024, 128), (4, [40, 33, 64, 15], 264, 2048, 256), (16, [2] * 15 + [0], 4104, 384, 128),
           (3, [0, 31, 64], 84, 1152, 1152), (2, [12, 4], 28672, 256, 128),
           # many turns of one expert's rows, shared by more and by fewer workgroups; experts in several sets of 64
           (64, [1] * 20 + [301] + [0] * 30 + [65] + [2] * 12, 200, 640, 128), (130, [0] * 66 + [97, 33] + [1] * 60 + [0, 200], 68, 1024, 256),
           (4, [0, 0, 0, 155], 4112, 512, 128)]


@pytest.mark.parametrize("E,rows,N,K,group", GROUPED)
@pytest.mark.parametrize("wide", [False, True])
def test_grouped(P, E, rows, N, K, group, wide):
    M = sum(rows)
    assert P.is_describe_grouped_prepacked(E, M, N, K, group)[-1].startswith("gemm_few_grouped_pk_kernel<")
    offsets = torch.tensor([sum(rows[:e]) for e in range(E + 1)], dtype=torch.int32, device="cuda:0")
    sets = [case(max(r, 1), N, K, group, wide and e % 2 == 1, seed=e) for e, r in enumerate(rows)]
    xq = torch.cat([s[0][:r] for s, r in zip(sets, rows)])
    sa = torch.cat([s[4][:r] for s, r in zip(sets, rows)])
    chan = torch.stack([s[5] for s in sets])
    packed = P.is_prepack_w4_experts(torch.stack([s[2] for s in sets]), torch.stack([s[3] for s in sets]), group)
    acc = torch.cat([wrapped(reference(s[0][:r], s[1], s[3], group)) for s, r in zip(sets, rows)])
    out, got = P.is_gemm_w4a8_intscale_grouped_prepacked(xq, sa, packed, chan, offsets, 10, want_acc=True)
    assert torch.equal(got, acc), "int32 accumulators"
    # the tiled form computes the same bits
    before = P.is_set_kernel_route("tiled64")
    try:
        assert P.is_describe_grouped_prepacked(E, M, N, K, group)[-1] == "gemm_tile_grouped_pk_kernel<true>"
        tiled, tiled_acc = P.is_gemm_w4a8_intscale_grouped_prepacked(xq, sa, packed, chan, offsets, 10, want_acc=True)
    finally:
        P.is_set_kernel_route(before)
    assert torch.equal(tiled_acc, got) and torch.equal(tiled, out)
    floats = [s[3].float() * (2.0 ** -32 if wide else 2.0 ** -17) for s in sets]
    fpacked = P.is_prepack_w4_experts(torch.stack([s[2] for s in sets]), torch.stack(floats), group)
    fout = P.is_gemm_w4a8_floatscale_grouped_prepacked(xq, sa, fpacked, offsets)
    fs = torch.cat([reference(s[0][:r], s[1], f, group) for s, f, r in zip(sets, floats, rows)]) * sa.double()[:, None]
    size = torch.cat([reference(s[0][:r].abs().clamp(max=127), s[1].abs(), f.abs(), group) for s, f, r in zip(sets, floats, rows)]) * sa.double()[:, None]
    assert bool(((fout.double() - fs).abs() <= 5e-4 * fs.abs() + 2.0 ** -25 + size * (K // group + 2) * 2.0 ** -24)[fs.abs() < 65000.0].all())


@pytest.mark.parametrize("E,M,N,K", [(64, 1536, 2816, 2048), (8, 190, 4096, 4096)])
def test_grouped_with_all_rows_at_one_expert_takes_its_share_of_the_chip(P, E, M, N, K):
    """The plan does not know the router: an expert that all rows come to must not be left to a few workgroups, turn after turn (5.5 times the
    tiled kernel's time on the first of these once; half of it with the rows shared out).  Replayed graphs, the least of five."""
    gen = torch.Generator(device="cuda:0").manual_seed(E + M)
    q = torch.randint(0, 256, (E, N, K // 2), generator=gen, device="cuda:0", dtype=torch.uint8)
    packed = P.is_prepack_w4_experts(q, torch.randint(0, 1025, (E, N, K // G), generator=gen, device="cuda:0", dtype=torch.int32), G)
    xq = torch.randint(-128, 128, (M, K), generator=gen, device="cuda:0", dtype=torch.int8)
    sa = torch.rand((M,), generator=gen, device="cuda:0")
    offsets = torch.tensor([0] * (E // 2) + [M] * (E - E // 2 + 1), dtype=torch.int32, device="cuda:0")
    ws = torch.zeros((P.is_gemm_grouped_prepacked_workspace_bytes(E, M, N, K, G),), dtype=torch.uint8, device="cuda:0")
    us, outs = [], []
    for route in ("auto", "tiled64"):
        before = P.is_set_kernel_route(route)
        try:
            name = P.is_describe_grouped_prepacked(E, M, N, K, G)[-1]
            assert name.startswith("gemm_few_grouped_pk_kernel<") == (route == "auto"), name
            out = torch.empty((M, N), dtype=torch.float16, device="cuda:0")
            call = lambda: P.is_gemm_w4a8_intscale_grouped_prepacked(xq, sa, packed, None, offsets, 10, out=out, workspace=ws)
            call()
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                call()
        finally:
            P.is_set_kernel_route(before)
        graph.replay()
        least = 1e9
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(8):
                graph.replay()
            b.record()
            torch.cuda.synchronize()
            least = min(least, a.elapsed_time(b) * 125.0)
        us.append(least)
        outs.append(out.clone())
    assert torch.equal(*outs)
    assert us[0] < 1.5 * us[1], us


# the kernel's tiles of 48 and 64 rows for more than 64 rows: one and several row tiles with remainders, ragged widths, uneven runs of
# K steps, every instance
ROWS = [(65, 5121, 2176, 128), (100, 6144, 4096, 256), (72, 12288, 4096, 128), (128, 5120, 2048, 128),
        (300, 6144, 4096, 128), (130, 8200, 3072, 384), (512, 5128, 2048, 128), (200, 8192, 4096, 128), (256, 5200, 5120, 512), (400, 5120, 4096, 128),
        (65, 1, 2048, 128), (130, 20, 2176, 128), (300, 72, 4096, 256), (97, 49, 28672, 1024), (512, 1041, 2304, 384), (66, 4096, 4096, 128)]


@pytest.mark.parametrize("M,N,K,group", ROWS)
@pytest.mark.parametrize("wide", [False, True])
def test_more_than_64_rows(P, M, N, K, group, wide):
    names = P.is_describe_prepacked(M, N, K, group)
    assert len(names) == 1 and names[0].startswith("gemm_rows_pk_kernel<"), names
    check_call(P, M, N, K, group, wide, chan=not wide)


@pytest.mark.parametrize("M,inter,K", [(65, 2576, 2048), (100, 5504, 2176), (200, 4096, 2048), (256, 2560, 4096), (67, 16, 2048), (130, 48, 2176)])
def test_more_than_64_rows_fused_gate_up(P, M, inter, K):
    test_fused_gate_up(P, M, inter, K)
    # which kernel took the call: this one leaves the workspace alone, the others write the activations' blocks to it
    xq, _, qw, scale, sa, c = case(M, 2 * inter, K)
    ws = torch.full((P.is_gemm_gate_up_silu_prepacked_workspace_bytes(M, inter, K, G),), 0x5A, dtype=torch.uint8, device="cuda:0")
    P.is_gemm_w4a8_intscale_gate_up_silu_prepacked(xq, sa, P.is_prepack_w4_gate_up(qw, scale, c, G), 10, workspace=ws)
    assert bool((ws == 0x5A).all())


# int8 weights: 16-row token tiles of 1 to 4, one and two weight tiles a workgroup (more than 4096 columns), ragged rows and columns,
# uneven runs of K steps, groups of several steps
@pytest.mark.parametrize("M,N,K,group", [(1, 20, 1024, 128), (16, 4100, 1152, 128), (1, 4112, 3072, 256), (17, 300, 2176, 128), (32, 4097, 1536, 512),
                                         (33, 1003, 1152, 384), (48, 5120, 1024, 128), (49, 97, 1152, 1152), (64, 4104, 1664, 128),
                                         (64, 16, 14336, 256), (64, 40, 28672, 128), (5, 4136, 28672, 128)])
@pytest.mark.parametrize("wide", [False, True])
def test_int8_weights(P, M, N, K, group, wide):
    xq, _, _, scale, sa, c = case(M, N, K, group, wide, seed=7)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(N + K)
    q = torch.randint(-128, 128, (N, K), generator=gen, device="cuda:0", dtype=torch.int8)
    cc, sa = (None if wide else c), sa * 2.0 ** -6
    acc = wrapped(reference(xq, q, scale, group))
    out, got = P.is_gemm_w8a8_intscale(xq, sa, q, scale, cc, group, 10, want_acc=True)
    assert torch.equal(got, acc), "int32 accumulators"
    want = acc.double() * sa.double()[:, None] * (1.0 if wide else c.double()[None, :]) / 1024.0
    # two fp32 products and one rounding to fp16: 2^-11 of the value and a little more, and half a step of the smallest numbers
    assert bool(((out.double() - want).abs() <= 5e-4 * want.abs() + 2.0 ** -25)[want.abs() < 65000.0].all())


def test_captured_calls(P):
    """One graph of the calls whose kernels differ: few rows, K cut over workgroups (its counters; the call on the library's own scratch as well),
    row tiles without a preparation, a mixture whose offsets change, W8A8.  Replayed with new inputs in the same buffers, the program's own work
    in between, against the ordinary calls each time."""
    shapes = [(16, 1000, 1024), (1, 64, 28672), (16, 64, 65536), (130, 328, 2176)]
    data = [case(M, N, K, seed=11) for M, N, K in shapes]
    packs = [P.is_prepack_w4(d[2], d[3], G) for d in data]
    E, MG, NG, KG = 8, 72, 300, 1024
    sets = [case(MG, NG, KG, seed=20 + e) for e in range(E)]
    experts = P.is_prepack_w4_experts(torch.stack([d[2] for d in sets]), torch.stack([d[3] for d in sets]), G)
    assert P.is_describe_grouped_prepacked(E, MG, NG, KG, G)[-1].startswith("gemm_few_grouped_pk_kernel<")
    offsets = torch.tensor([0] + [MG] * E, dtype=torch.int32, device="cuda:0")
    q8 = torch.randint(-128, 128, (300, 2176), dtype=torch.int8, device="cuda:0")
    x8, s8 = torch.zeros((17, 2176), dtype=torch.int8, device="cuda:0"), torch.randint(0, 1025, (300, 17), dtype=torch.int32, device="cuda:0")
    sa8 = torch.rand((17,), device="cuda:0")
    sizes = [P.is_gemm_prepacked_workspace_bytes(*s, G) for s in shapes] + [P.is_gemm_grouped_prepacked_workspace_bytes(E, MG, NG, KG, G),
                                                                              P.is_gemm_w8a8_workspace_bytes(17, 300, 2176, G)]
    outs = [torch.empty((M, N), dtype=torch.float16, device="cuda:0") for M, N, _ in shapes + [(MG, NG, 0), (17, 300, 0), (16, 64, 0)]]

    def calls(outs, ws):
        for d, pk, out, w in zip(data, packs, outs, ws):
            P.is_gemm_w4a8_intscale_prepacked(d[0], d[4], pk, d[5], 10, out=out, workspace=w)
        P.is_gemm_w4a8_intscale_grouped_prepacked(sets[0][0], sets[0][4], experts, None, offsets, 10, out=outs[4], workspace=ws[4])
        P.is_gemm_w8a8_intscale(x8, sa8, q8, s8, None, G, 10, out=outs[5], workspace=ws[5])
        P.is_gemm_w4a8_intscale_prepacked_noalloc(data[2][0], data[2][4], packs[2], data[2][5], 10, outs[6])

    ws = [torch.zeros((max(n, 16),), dtype=torch.uint8, device="cuda:0") for n in sizes]
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
        for x in [d[0] for d in data] + [sets[0][0], x8]:
            x.copy_(torch.randint(-128, 128, tuple(x.shape), dtype=torch.int8, device="cuda:0"))
        ends = torch.randint(0, MG + 1, (E - 1,), device="cuda:0").sort().values.to(torch.int32)
        offsets[1:E].copy_(ends if i else torch.zeros_like(ends))
        graph.replay()
        torch.cuda.synchronize()
        want = [torch.empty_like(o) for o in outs]
        calls(want, [torch.zeros_like(w) for w in ws])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, want)), f"replay {i}"
    assert torch.equal(outs[2], outs[6])
