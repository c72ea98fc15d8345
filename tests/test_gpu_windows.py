"""GPU: runs against the cuts of the 256-digi windows of forming and writing, against the oracle.

Chains of adjacent strips of 1 to 256 strips (768 in module rows), records that go on from one
another, lists just below, at and above whole windows, inactive strips inside records, in FEDs that
fit the LDS stage and in larger ones, and from dense rows. Everything bit-exact.
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
from gpu_common import bary_bit_exact, compare_clusters, make_ctx, run_fused  # noqa: E402


def _mask(kind, rng, n):
    """n strips in a row of channels: which ones carry a digi."""
    m = np.zeros(n, bool)
    if kind == "full":
        m[:] = True
    elif kind == "comb":
        m[::2] = True
    else:
        pos = 0
        while pos < n:
            w = int(rng.choice([1, 2, 3, 4, 5, 8, 9, 255, 256, 300] if kind == "long" else [1, 1, 1, 2, 3, 4, 5, 9]))
            m[pos:pos + w] = True
            pos += w + 1 + int(rng.integers(0, 40 if kind == "sparse" else 3))
    return m


def _event(kind, seed, channels, max_run):
    rng = np.random.default_rng(seed)
    noise, gain, bad = calib_arrays(2)
    noise[:] = rng.uniform(2.0, 9.0, noise.size)
    gain[:] = rng.uniform(0.5, 2.0, gain.size)
    bad[:] = rng.random(bad.size) < {"full": 0.0, "long": 0.001}.get(kind, 0.02)
    dense = np.zeros((2 * NCH, NS), np.uint8)
    for f in range(2):
        m = _mask(kind, rng, channels * NS).reshape(channels, NS)
        rows = dense[f * NCH:f * NCH + channels]
        rows[m] = rng.integers(30 if kind in ("full", "long") else 1, 256, int(m.sum()))
    mask = dense > 0
    mask[:, ::97] |= rng.random(mask[:, ::97].shape) < 0.1   # ADC 0 inside the data
    zs, fo = fedgen.encode_dense(dense, mask, max_run=max_run)
    return zs, fo, noise, gain, bad


CASES = [("full", 24, 255), ("full", 3, 7), ("comb", 40, 255), ("long", 30, 100), ("long", 24, 255),
         ("dense", 60, 3), ("sparse", 96, 255), ("sparse", 48, 2)]


@pytest.mark.parametrize("modules", [False, True], ids=["plain", "rows"])
@pytest.mark.parametrize("kind,channels,max_run", CASES)
def test_runs_across_window_cuts(kind, channels, max_run, modules):
    zs, fo, noise, gain, bad = _event(kind, 7, channels, max_run)
    cm = np.arange(2 * NCH, dtype=np.uint32) // 3
    joins = np.zeros(2 * NCH, np.uint8)
    joins[1:] = cm[1:] == cm[:-1]
    ref = oracle.process_event(zs, fo, noise, gain, bad, joins=joins if modules else None)
    assert ref.cl.size > 0
    with make_ctx(noise, gain, bad) as ctx:
        if modules:
            ctx.set_modules(cm)
        for waves, chunk, stage in ((2, 2880, 0), (1, 1024, 0), (4, 3072, 0), (4, 6144, 10240)):
            ctx.tuning = {"use_graph": 0, "tile_waves": waves, "chunk_digis": chunk, "stage_bytes": stage}
            (res,), rc, _, _ = run_fused(ctx, [(zs, fo)])
            compare_clusters(res[0], res[1], ref, f"{kind} {waves}x{chunk}")
            assert bary_bit_exact(res[0], ref)
        dense, _ = ctx.unpack(sc.Event(zs, fo).to_device())
        out = ctx.output(ref.cl.size, ref.adc.size)
        ctx.cluster(dense, out)
        compare_clusters(*out.to_numpy()[:2], ref, f"{kind} dense")


def test_gains_outside_the_reciprocal_range():
    """One tiny usable gain: the whole context divides; a zero and a NaN gain change nothing."""
    zs, fo, noise, gain, bad = _event("dense", 3, 30, 255)
    gain[4], gain[7], gain[9] = 1e-25, 0.0, np.nan
    ref = oracle.process_event(zs, fo, noise, gain, bad)
    assert (ref.adc == 65535).any()
    with make_ctx(noise, gain, bad) as ctx:
        (res,), _, _, _ = run_fused(ctx, [(zs, fo)])
        compare_clusters(res[0], res[1], ref)
        assert bary_bit_exact(res[0], ref)


@pytest.mark.parametrize("t_cluster", [0.0, 1e-14, 5.0, 1e14, 3e38])
def test_cluster_thresholds_outside_the_range_of_squares(t_cluster):
    zs, fo, noise, gain, bad = _event("sparse", 5, 40, 255)
    noise[:200] = 0.0
    noise[256:300] = 1e-30
    noise[512:600] = 1e25
    ref = oracle.process_event(zs, fo, noise, gain, bad, t_cluster=t_cluster)
    with make_ctx(noise, gain, bad, t_cluster=t_cluster) as ctx:
        (res,), _, _, _ = run_fused(ctx, [(zs, fo)])
        compare_clusters(res[0], res[1], ref)
