"""Small batches of the wide models (d 1536 and 2048) over several key splits:
row counts on both sides of the one up to which the out-projection's workgroup
has a thread for every item that it merges (10 rows at d 1536, 8 at d 2048).
Selection exact at every step; logits of every sequence within 3e-2 of the
float64 oracle, as for the other bf16 models."""
import pytest

from gpu_common import log
from paper_2410_13839_amd.workloads import ModelShape, Workload
from test_gpu_parity import run_teacher_forced

pytestmark = pytest.mark.gpu

# d, heads K, batch: rows per step = K * batch
CASES = {"d1536, 10 rows": (1536, 2, 5), "d1536, 11 rows": (1536, 1, 11), "d1536, 16 rows": (1536, 4, 4),
         "d2048, 8 rows": (2048, 8, 1), "d2048, 9 rows": (2048, 3, 3), "d2048, 16 rows": (2048, 8, 2)}


@pytest.mark.parametrize("name", list(CASES))
def test_every_row_is_merged(name):
    d, K, B = CASES[name]
    log(f"{name}: start")
    shape = ModelShape(n_layers=2, d_model=d, n_heads=d // 64, d_ff=512, k_heads=K, dtype="bf16")
    wl = Workload("wide", shape, K=K, top_k=3, batch=B, phon_len=(3, 20), ac_len=(280, 420), max_new=4 * K, eos_min=4 * K)
    steps, _, chk = run_teacher_forced(wl, K, 3, steps_checked={1, 3}, tol=3e-2)
    assert steps == 4 and chk.checked == 2 * B
    log(f"{name}: max logit err {chk.max_err:.3g}")
