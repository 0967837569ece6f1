"""shadowkv_build_landmarks over chunk sizes at the edges of the eight rows a lane group takes at a time (-m gpu), both
storage types, every head width, against the oracle: outlier sets, landmarks and gathered rows bit for bit."""
import pytest

from workloads import Workload, generate, to_fp8_storage

import parity_util as PU

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kd", [0, 1])
@pytest.mark.parametrize("c,d", [(1, 64), (5, 96), (7, 128), (8, 96), (9, 128), (15, 64), (16, 128), (17, 96), (24, 64), (64, 128)])
def test_build_at_every_row_group(c, d, kd):
    wl = Workload("build-chunks", batch=2, n_q_heads=2, n_kv_heads=1, head_dim=d, ctx_len=c * 67, chunk_size=c, rank=16,
                  n_outlier_chunks=3, topk_chunks=4, local_len=2, seed=50 + c, n_queries=1)
    print(f"\n[case] kv_dtype {kd} {wl}", flush=True)
    t = generate(wl, device="cuda")
    if kd:
        t = to_fp8_storage(t)
    PU.run_build_parity(wl, t, kv_dtype=kd)
