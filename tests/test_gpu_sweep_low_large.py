"""GPU: dense two-qubit sweeps on qubit 0 use streaming accesses on states beyond the cache (256 MiB) and plain
ones below: the same amplitudes, bit for bit, on either side of the line."""
import numpy as np
import pytest

from workloads import U2, Gate

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a,b", [(0, 3), (6, 0), (0, 9), (15, 0)])
def test_streaming_and_plain_accesses_agree(a, b):
    n, few, many = 16, 2, 513          # 2^16 amplitudes of 8 bytes: 512 slots are 256 MiB
    m = np.linalg.qr(np.random.default_rng(1).standard_normal((4, 8)).view(np.complex128))[0]
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.view_as_complex(torch.randn((few, 1 << n, 2), generator=gen, device="cuda"))
    out = []
    for T in (few, many):
        sv = q.StateVector(n, q.C64, T)
        amps = sv.amplitudes()
        for t in range(0, T, few):
            amps[t:t + few].copy_(x[: min(few, T - t)])
        torch.cuda.synchronize()
        q.apply_gate(sv, Gate(U2, q0=a, q1=b, m=m))
        torch.cuda.synchronize()
        out.append(amps)
    assert torch.equal(out[0], out[1][:few])
    # every pair of slots of the large batch holds the same two states
    pairs = out[1][: many - 1].reshape(-1, few, 1 << n)
    assert bool((pairs == out[0]).all()) and torch.equal(out[1][many - 1], out[0][0])
