"""GPU: the default shape with its stage named (2 waves, 2880 digis, 6656 bytes) is used as it is, also
for launches that the library would give another. Sizes at which its lists of 1440 digis per wave and
its windows can go wrong, from ZS bytes and from dense rows, with and without module rows, against the
oracle, bit-exact; and what the tuning reads back as.
"""
import numpy as np
import pytest

import fedgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2101_11489_amd as sc  # noqa: E402
import test_gpu_batching as batching  # noqa: E402
import test_gpu_dense_groups as groups  # noqa: E402
import test_gpu_member_lists as lists  # noqa: E402
import test_gpu_tile_queues as queues  # noqa: E402
import test_gpu_windows as windows  # noqa: E402
from gpu_common import bary_bit_exact, compare_clusters, make_ctx, run_fused  # noqa: E402
from helpers import NCH, calib_arrays  # noqa: E402

SHAPE = {"chunk_digis": 2880, "tile_waves": 2, "stage_bytes": 6656, "use_graph": 0}
ROWS = pytest.mark.parametrize("modules", [False, True], ids=["plain", "rows"])


def _modules(n_fed, per):
    cm = np.arange(n_fed * NCH, dtype=np.uint32) // per
    joins = np.zeros(cm.size, np.uint8)
    joins[1:] = cm[1:] == cm[:-1]
    return cm, joins


@ROWS
@pytest.mark.parametrize("kind,channels,max_run", windows.CASES)
def test_windows(kind, channels, max_run, modules):
    zs, fo, noise, gain, bad = windows._event(kind, 7, channels, max_run)
    cm, joins = _modules(2, 3)
    ref = oracle.process_event(zs, fo, noise, gain, bad, joins=joins if modules else None)
    with make_ctx(noise, gain, bad) as ctx:
        if modules:
            ctx.set_modules(cm)
        ctx.tuning = SHAPE
        (res,), _, _, _ = run_fused(ctx, [(zs, fo)])
        dense, _ = ctx.unpack(sc.Event(zs, fo).to_device())
        out = ctx.output(ref.cl.size, ref.adc.size)
        ctx.cluster(dense, out)
        for got in (res, out.to_numpy()):
            compare_clusters(got[0], got[1], ref, kind)
            assert bary_bit_exact(got[0], ref)


@ROWS
def test_dense_groups(modules):
    groups.test_groups_about_the_size_of_a_list(2, 2880, 6656, modules)


@pytest.mark.parametrize("kind", ["all_empty", "zero_length_feds", "full_fed", "alternating_fed",
                                  "between_stages", "multichunk_fits_stage", "group_heads", "garbage"])
def test_edges(kind):
    batching.test_edge_cases(kind, (2880, 2, 6656))


def test_queues():
    queues.test_many_tiles_of_every_queue(2, 2880, 6656)


@ROWS
@pytest.mark.parametrize("order", [0, 1, 2])
def test_lists(order, modules):
    n_fed = lists.N_FED
    kinds = [lists._event(1, 0.05, 1.0), lists._event(2, 0.1, 0.0), lists._event(3, 0.04, 0.5),
             lists._event(6, 0.16, 0.7)]
    noise, gain, bad = calib_arrays(n_fed)
    noise[:] = np.random.default_rng(7).uniform(3.0, 6.0, noise.size)
    cm, joins = _modules(n_fed, 2)
    refs = [oracle.process_event(z, f, noise, gain, bad, joins=joins if modules else None) for z, f in kinds]
    which = np.random.default_rng(8).integers(0, len(kinds), 320)   # 960 tiles, 256 workgroups
    with make_ctx(noise, gain, bad) as ctx:
        if modules:
            ctx.set_modules(cm)
        ctx.tuning = dict(SHAPE, tiles_per_cu=1, fed_major=order)
        res, _, _, _ = run_fused(ctx, [kinds[k] for k in which])
        for k, r in zip(which, res):
            compare_clusters(r[0], r[1], refs[k], f"kind {k}")
            assert bary_bit_exact(r[0], refs[k])


def test_tuning_reads_back(tmp_path):
    noise, gain, bad = calib_arrays(1)
    cache = tmp_path / "tune.json"
    with make_ctx(noise, gain, bad, tune_cache=str(cache)) as ctx:
        first = ctx.tuning
        assert [first[k] for k in ("chunk_digis", "tile_waves", "stage_bytes")] == [2880, 2, 0]
        ctx.tuning = {"use_graph": 0, "fed_major": 1, "tiles_per_cu": 7}
        assert ctx.tuning["stage_bytes"] == 0                      # nothing said of the shape
        for named in ({"chunk_digis": 2880}, {"tile_waves": 2}, {"stage_bytes": 6656}):
            ctx.tuning = first
            ctx.tuning = named
            assert ctx.tuning == dict(first, stage_bytes=6656)
        ctx.tuning = {"chunk_digis": 1024, "tile_waves": 1, "stage_bytes": 0}
        assert ctx.tuning["stage_bytes"] == 6656
        ctx.tuning = {"chunk_digis": 6144, "tile_waves": 4, "stage_bytes": 10240}
        ctx.tuning = first
        assert ctx.tuning == first
        e = fedgen.make_event(fedgen.CONFIGS[0].with_(n_fed=1), fedgen.make_calibration(
            fedgen.CONFIGS[0].with_(n_fed=1)), 0)
        best = ctx.autotune([sc.Event(e.zs, e.fed_offset).to_device()])
        assert best["stage_bytes"] in (6656, 10240) and ctx.tuning == best
    # entries of the cache that are older than the stage size name the small one
    key, six = cache.read_text().split('"')[1], [2880, 2, 8, 2, 1, 6656]
    for entry in (six, six[:5], six[:5] + [0]):
        cache.write_text('{\n  "%s": %s\n}\n' % (key, str(entry).replace(" ", "")))
        with make_ctx(noise, gain, bad, tune_cache=str(cache)) as ctx:
            assert list(ctx.tuning.values()) == six
