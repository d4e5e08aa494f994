"""The recurrent core's gates by rows: 16-row blocks, 32-row blocks where those are one to a compute unit, 16-row blocks again."""
import pytest

from paper_1910_06591_amd import workloads as wl
from tests.test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,rows", [("C2", 128), ("C2", 129), ("C2", 239), ("C2", 256), ("C2", 257), ("C3", 257), ("C3", 500)])
def test_gates_by_rows(orc, name, rows):
    run_case(orc, wl.CONFIGS[name], rows, "bf16", intermediates=False)
