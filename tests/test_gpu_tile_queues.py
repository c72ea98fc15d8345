"""GPU: tile order 2 where workgroups run out of their own queue's tiles long before another queue does.

Queue 0 of the per-XCD order holds the first and the last FED, which are large; the other queues hold
small ones, whose offsets wait for the first FED of their event. Against the oracle, bit-exact.
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


@pytest.mark.parametrize("n_fed", [9, 17])
@pytest.mark.parametrize("waves,chunk", [(1, 1024), (2, 2880), (4, 6144)])
@pytest.mark.parametrize("tiles_per_cu", [1, 32])
def test_queues_of_unequal_work(tiles_per_cu, waves, chunk, n_fed):
    noise, gain, bad = calib_arrays(n_fed)
    kinds, refs = [], []
    for seed in range(3):
        rng = np.random.default_rng(seed)
        occ = np.full(n_fed, 0.002)
        occ[::8] = 0.1
        mask = rng.random((n_fed * NCH, NS)) < np.repeat(occ, NCH)[:, None]
        dense = np.where(mask, rng.integers(40, 256, mask.shape), 0).astype(np.uint8)
        kinds.append(fedgen.encode_dense(dense, mask, max_run=255))
        refs.append(oracle.process_event(*kinds[-1], noise, gain, bad))
        assert refs[-1].cl.size > 2000
    which = np.random.default_rng(8).integers(0, len(kinds), 320)
    with make_ctx(noise, gain, bad) as ctx:
        ctx.tuning = {"use_graph": 0, "tile_waves": waves, "chunk_digis": chunk,
                      "stage_bytes": 10240 if chunk == 6144 else 0, "tiles_per_cu": tiles_per_cu,
                      "fed_major": 2}
        res, _, _, _ = run_fused(ctx, [kinds[k] for k in which])
        for k, r in zip(which, res):
            compare_clusters(r[0], r[1], refs[k], f"kind {k}")
            assert bary_bit_exact(r[0], refs[k])


@pytest.mark.parametrize("waves,chunk,stage", [(1, 1024, 0), (1, 2048, 0), (2, 2048, 10240), (2, 2880, 0),
                                               (4, 2048, 0), (4, 6144, 10240)])
def test_many_tiles_of_every_queue(waves, chunk, stage):
    """Several tiles per workgroup of the largest grid, from every queue, each event's FEDs in a row."""
    n_fed = 440
    noise, gain, bad = calib_arrays(n_fed)
    rng = np.random.default_rng(2)
    mask = rng.random((n_fed * NCH, NS)) < 0.001
    dense = np.where(mask, rng.integers(40, 256, mask.shape), 0).astype(np.uint8)
    zs, fo = fedgen.encode_dense(dense, mask, max_run=255)
    ref = oracle.process_event(zs, fo, noise, gain, bad)
    assert ref.cl.size > 5000
    with make_ctx(noise, gain, bad) as ctx:
        ctx.tuning = {"use_graph": 0, "tile_waves": waves, "chunk_digis": chunk, "stage_bytes": stage,
                      "tiles_per_cu": 32, "fed_major": 2}
        res, _, _, _ = run_fused(ctx, [(zs, fo)] * 24)
        for r in res:
            compare_clusters(r[0], r[1], ref)
            assert bary_bit_exact(r[0], ref)
