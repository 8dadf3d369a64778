"""The executed flops that a plan reports for its adjoint passes: per amplitude and run two
unscaled rotations (4 each; 6 as shears with five register qubits) and the functionals that
are formed (4 each): three, or two where every run of an epoch is RY gates then RZ gates and
four qubits are in registers."""
import pytest

torch = pytest.importorskip("torch")

from paper_2603_02804_amd import qfuse  # noqa: E402
from paper_2603_02804_amd.workloads import hea_gates  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rots,R,flops", [
    (12, ("RY", "RZ"), 0, 16), (12, ("RX", "RY", "RZ"), 0, 20), (14, ("RY", "RZ"), 0, 16), (8, ("RY", "RZ"), 3, 20),
    (12, ("RY", "RZ"), 5, 24), (12, ("RX", "RY", "RZ"), 5, 24),
])
def test_executed_flops(n, rots, R, flops):
    torch.zeros(1, device="cuda")
    L = 3
    circ = qfuse.Circuit(n, hea_gates(n, L, rots, encoding=False), L * len(rots) * n, 0, [1])
    info = qfuse.Plan(circ, 2, qfuse.make_tuning(reg_qubits=R)).info
    assert info.n_runs == L * n
    assert info.exec_bwd_pass_flops_per_sample == flops * info.n_runs * 2.0 ** n
