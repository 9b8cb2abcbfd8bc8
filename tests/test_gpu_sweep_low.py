"""GPU: dense two-qubit sweeps of complex<float> that touch qubit 0 (its two values share a vector), the
other qubit below, on and above the last lane bit, in both orders, for states smaller than, of and
larger than one workgroup's vectors, against numpy.

Tolerance: four products of single precision per amplitude of a unitary, 2e-6 of the state's norm."""
import numpy as np
import pytest

from workloads import U2, Gate

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,T", [(2, 1), (3, 3), (9, 2), (10, 3), (11, 1), (14, 3)])
def test_dense_sweeps_on_qubit_zero(n, T):
    rng = np.random.default_rng(n)
    sv = q.StateVector(n, q.C64, T)
    amps = sv.amplitudes()
    i = np.arange(1 << n)
    for hi in sorted({h for h in (1, 2, 5, 6, 7, n - 1) if h < n}):
        for a, b in ((0, hi), (hi, 0)):
            z = rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4))
            m = np.linalg.qr(z)[0]
            x = rng.standard_normal((T, 1 << n)) + 1j * rng.standard_normal((T, 1 << n))
            x = (x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.complex64)
            amps.copy_(torch.as_tensor(x).to(amps.device))
            torch.cuda.synchronize()
            q.apply_gate(sv, Gate(U2, q0=a, q1=b, m=m))
            torch.cuda.synchronize()
            loc, rest = ((i >> a) & 1) + 2 * ((i >> b) & 1), i & ~((1 << a) | (1 << b))
            want = sum(m[loc, k] * x.astype(np.complex128)[:, rest | ((k & 1) << a) | ((k >> 1) << b)] for k in range(4))
            assert np.linalg.norm(amps.cpu().numpy() - want) <= 2e-6 * np.sqrt(T), (a, b)
