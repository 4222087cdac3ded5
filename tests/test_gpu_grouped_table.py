"""The mixture-of-experts form with more experts than a wave has lanes: the table of row tiles is built 64 experts at a time."""
import numpy as np
import pytest

from oracle import oracle as O
from test_gpu_parity import dev, host

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("experts", [63, 64, 65, 130])
def test_many_experts(experts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_14597_amd as P
    P.load_library()
    N, K, G = 48, 256, 128
    rng = np.random.default_rng(7000 + experts)
    counts = rng.choice([0, 0, 1, 16, 17, 33, 64, 65, 128, 129, 200], size=experts)
    counts[-1] = 40
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    M = int(offsets[-1])
    xq = rng.integers(-128, 128, size=(M, K)).astype(np.int8)
    qw = np.stack([O.pack_int4(rng.integers(-8, 8, size=(N, K)).astype(np.int8)) for _ in range(experts)])
    IS = rng.integers(0, 1025, size=(experts, N, K // G)).astype(np.int32)
    sa = (rng.random(M) + 0.1).astype(np.float32)
    c = (rng.random((experts, N)) * 0.05 + 1e-3).astype(np.float32)
    pk = P.is_prepack_w4_experts(dev(qw), dev(IS), G)
    out, acc = P.is_gemm_w4a8_intscale_grouped_prepacked(dev(xq), dev(sa), pk, dev(c), dev(offsets), 10, want_acc=True)
    for e in range(experts):
        lo, hi = offsets[e], offsets[e + 1]
        if hi > lo:
            ref = O.gemm_w4a8_intscale(xq[lo:hi], sa[lo:hi], qw[e], IS[e], c[e], G, 10)
            assert np.array_equal(host(acc)[lo:hi], ref.acc), f"expert {e}"
