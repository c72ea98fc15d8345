"""GPU: the dense front end's whole channel groups and its chunks, and unpacking from and past the
LDS stage, against the oracle. Digi counts at and next to what a wave's list holds. Bit-exact.
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

import paper_2101_11489_amd as sc  # noqa: E402
from gpu_common import bary_bit_exact, compare_clusters, make_ctx  # noqa: E402


@pytest.mark.parametrize("modules", [False, True], ids=["plain", "rows"])
@pytest.mark.parametrize("waves,chunk,stage", [(1, 1024, 0), (2, 2880, 0), (4, 3072, 0), (4, 6144, 10240)])
def test_groups_about_the_size_of_a_list(waves, chunk, stage, modules):
    cap, per = chunk // waves, NCH // waves
    rng = np.random.default_rng(11)
    counts = [0, 1, cap - 1, cap, cap + 1, min(2 * cap + 5, per * NS), per * NS]
    n_fed = -(-len(counts) // waves)
    noise, gain, bad = calib_arrays(n_fed)
    noise[:] = rng.uniform(2.0, 9.0, noise.size)
    gain[:] = rng.uniform(0.5, 2.0, gain.size)
    flat = np.zeros(n_fed * NCH * NS, np.uint8)
    for i, n in enumerate(counts):   # group i of the detector: waves groups per FED
        strips = i * per * NS + rng.choice(per * NS, n, replace=False)
        flat[strips] = rng.integers(1, 256, n)
    dense = flat.reshape(-1, NS)
    cm = np.arange(n_fed * NCH, dtype=np.uint32) // 3
    joins = np.zeros(cm.size, np.uint8)
    joins[1:] = cm[1:] == cm[:-1]
    zs, fo = fedgen.encode_dense(dense, dense > 0, max_run=255)
    ref = oracle.process_event(zs, fo, noise, gain, bad, joins=joins if modules else None)
    assert ref.cl.size > 0
    with make_ctx(noise, gain, bad) as ctx:
        if modules:
            ctx.set_modules(cm)
        ctx.tuning = {"use_graph": 0, "tile_waves": waves, "chunk_digis": chunk, "stage_bytes": stage}
        out = ctx.output(ref.cl.size, ref.adc.size)
        ctx.cluster(torch.from_numpy(dense).cuda(), out)
        compare_clusters(*out.to_numpy()[:2], ref, f"{waves}x{chunk}")
        assert bary_bit_exact(out.to_numpy()[0], ref)


@pytest.mark.parametrize("spoilt", [0, 8])
@pytest.mark.parametrize("max_run", [1, 5, 255])
@pytest.mark.parametrize("occupancy", [0.0, 0.02, 0.2, 1.0])
def test_unpack(occupancy, max_run, spoilt):
    """FEDs that fit the stage and larger ones, whole and with a few bytes changed."""
    rng = np.random.default_rng(5)
    n_fed = 6
    dense = rng.integers(1, 256, (n_fed * NCH, NS)).astype(np.uint8)
    dense[rng.random(dense.shape) >= occupancy] = 0
    dense[::7] = 0
    zs, fo = fedgen.encode_dense(dense, dense > 0, max_run=max_run)
    zs = zs.copy()
    zs[rng.integers(0, zs.size, spoilt)] ^= 3
    want, want_st, want_rc = oracle.unpack(zs, fo)
    assert spoilt or want_rc == 0
    noise, gain, bad = calib_arrays(n_fed)
    with make_ctx(noise, gain, bad) as ctx:
        st = torch.full((n_fed * NCH,), 99, dtype=torch.uint8, device="cuda")
        got, rc = ctx.unpack(sc.Event(zs, fo).to_device(), None, st)
        assert rc == want_rc
        assert np.array_equal(got.cpu().numpy().reshape(-1), want)
        assert np.array_equal(st.cpu().numpy(), want_st)
