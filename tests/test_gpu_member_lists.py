"""GPU: the formed list holds members only, and the next tile's list is built over what it leaves.

Workgroups take many tiles in a row: digis that are all members, none, and every second one, with
records and without. Against the oracle, bit-exact.
"""
import numpy as np
import pytest

import fedgen
import oracle
from helpers import NCH, NS, calib_arrays

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_common import bary_bit_exact, compare_clusters, make_ctx, run_fused  # noqa: E402

N_FED = 3


def _event(seed, occupancy, members, n_fed=N_FED):
    """Rows whose digis are large (members), or 1 (under every threshold)."""
    rng = np.random.default_rng(seed)
    dense = np.zeros((n_fed * NCH, NS), np.uint8)
    mask = rng.random(dense.shape) < occupancy
    big = rng.random(dense.shape) < members
    dense[mask] = np.where(big, rng.integers(60, 256, dense.shape), 1)[mask]
    return fedgen.encode_dense(dense, mask, max_run=255)


@pytest.mark.parametrize("modules", [False, True], ids=["plain", "rows"])
@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("waves,chunk", [(1, 1024), (2, 2880), (4, 3072)])
def test_lists_over_one_another(waves, chunk, order, modules):
    kinds = [_event(1, 0.05, 1.0), _event(2, 0.1, 0.0), _event(3, 0.04, 0.5), _event(4, 0.0, 0.0),
             _event(5, 0.002, 1.0), _event(6, 0.16, 0.7)]
    noise, gain, bad = calib_arrays(N_FED)
    noise[:] = np.random.default_rng(7).uniform(3.0, 6.0, noise.size)
    cm = np.arange(N_FED * NCH, dtype=np.uint32) // 2
    joins = np.zeros(cm.size, np.uint8)
    joins[1:] = cm[1:] == cm[:-1]
    refs = [oracle.process_event(z, f, noise, gain, bad, joins=joins if modules else None) for z, f in kinds]
    assert refs[0].adc.size > 2500 and refs[1].adc.size == 0 and refs[2].adc.size > 800
    which = np.random.default_rng(8).integers(0, len(kinds), 320)   # 960 tiles, 256 workgroups
    with make_ctx(noise, gain, bad) as ctx:
        if modules:
            ctx.set_modules(cm)
        ctx.tuning = {"use_graph": 0, "tile_waves": waves, "chunk_digis": chunk, "stage_bytes": 0,
                      "tiles_per_cu": 1, "fed_major": order}
        res, _, _, _ = run_fused(ctx, [kinds[k] for k in which])
        for k, r in zip(which, res):
            compare_clusters(r[0], r[1], refs[k], f"kind {k}")
            assert bary_bit_exact(r[0], refs[k])
