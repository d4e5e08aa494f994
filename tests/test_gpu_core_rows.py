"""The recurrent core's gates by rows: 16-row blocks, 32-row blocks where those are one to a compute unit and K is long enough
for their eight wavefronts, 16-row blocks again."""
import numpy as np
import pytest

from paper_1910_06591_amd import seedinf, workloads as wl
from tests.parity import to_device
from tests.test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,rows", [("C2", 128), ("C2", 129), ("C2", 239), ("C2", 256), ("C2", 257), ("C3", 257), ("C3", 500)])
def test_gates_by_rows(orc, name, rows):
    run_case(orc, wl.CONFIGS[name], rows, "bf16", intermediates=False)


def test_short_k_keeps_sixteen_row_blocks():
    """The DMLab agent's core has 16 chunks of K: its gates are summed over four wavefronts below and above 256 rows, so a
    row's state does not depend on which side its batch is."""
    cfg = wl.CONFIGS["C3"]
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=512), wl.make_weights(cfg))
    inputs = wl.make_batch(cfg, 512)

    def step(rows):
        out = net.step(**to_device({k: None if v is None else np.ascontiguousarray(v[:rows]) for k, v in inputs.items()}))
        return {k: out[k][:200].cpu().numpy() for k in ("h", "c", "logits")}

    small = step(200)
    for rows in (257, 400, 512):
        for k, v in step(rows).items():
            np.testing.assert_array_equal(v, small[k], err_msg=f"{k}, {rows} rows")
    net.close()
