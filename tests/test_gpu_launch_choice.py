"""GPU: the launches that the default tuning stands for, against the oracle: one tile per workgroup, the
large shape, and both shapes enqueued with the device choosing, for device and host events, ordinary
and large FEDs and a mix of both, through the batch, graph, allocation-free, pipelined and served calls.
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
from gpu_common import compare_clusters, make_ctx  # noqa: E402

N_FED = 41   # not a multiple of the eight queues


@pytest.fixture(scope="module")
def data():
    cfg = fedgen.CONFIGS[4].with_(n_fed=N_FED)
    cal = fedgen.make_calibration(cfg)
    evs = [fedgen.make_event(cfg.with_(occ=o), cal, i) for i, o in enumerate((0.06, 0.055, 0.005, 0.01))]
    refs = [oracle.process_event(e.zs, e.fed_offset, cal.noise, cal.gain, cal.bad) for e in evs]
    sizes = [np.diff(e.fed_offset.astype(np.int64)) for e in evs]
    assert sizes[0].min() > 6640 and sizes[2].max() < 5200
    return cal, evs, refs


def _caps(event, ref, room):
    return (ref.cl.size, ref.adc.size) if room == "exact" else sc.safe_caps(event)


# events (0, 1 large, 2, 3 ordinary) x copies: 41 FEDs each, so 24 events still have a workgroup per
# tile in the large shape and 40 do not
@pytest.mark.parametrize("pattern,n", [((0, 1), 1), ((2, 3), 24), ((0, 1), 25), ((0, 1), 40), ((2, 3), 40),
                                       ((0, 2, 3), 40), ((2, 3, 2, 3, 2, 3, 2, 0), 40)])
@pytest.mark.parametrize("where,room", [("dev", "safe"), ("dev", "exact"), ("host", "safe")])
def test_batches(data, pattern, n, where, room):
    cal, evs, refs = data
    idx = [pattern[i % len(pattern)] for i in range(n)]
    hosts = [sc.Event(e.zs, e.fed_offset) for e in evs]
    devs = [h.to_device() for h in hosts]
    with make_ctx(cal.noise, cal.gain, cal.bad) as ctx:
        src = devs if where == "dev" else hosts
        events = [src[i] for i in idx]
        outs = [ctx.output(*_caps(hosts[i], refs[i], room)) for i in idx]
        for graph in (1, 0, 1):
            ctx.tuning = {"use_graph": graph}
            rc, _ = ctx.process_events(events, outs)
            assert rc == sc.SC_OK
            for k, (i, o) in enumerate(zip(idx, outs)):
                compare_clusters(*o.to_numpy()[:2], refs[i], f"graph {graph} event {k}")
                o.cl.zero_()
                o.adc.zero_()


def test_other_calls(data):
    cal, evs, refs = data
    idx = [i % 4 for i in range(40)]
    hosts = [sc.Event(e.zs, e.fed_offset) for e in evs]
    devs = [h.to_device() for h in hosts]
    with make_ctx(cal.noise, cal.gain, cal.bad) as ctx:
        outs = [ctx.output(*sc.safe_caps(hosts[i])) for i in idx]
        b = ctx.batch([devs[i] for i in idx], outs)
        torch.cuda.synchronize()
        assert sc.lib().sc_process_events_static(ctx._h, b.c_ev, b.n, b.c_out, b.c_st) == sc.SC_OK
        for i, o in zip(idx, outs):
            compare_clusters(*o.to_numpy()[:2], refs[i], "static")
        outs = [ctx.output(*sc.safe_caps(hosts[i])) for i in idx]
        rc, _ = ctx.process_pipelined([hosts[i] if k % 3 else devs[i] for k, i in enumerate(idx)], outs, 30)
        assert rc == sc.SC_OK
        for i, o in zip(idx, outs):
            compare_clusters(*o.to_numpy()[:2], refs[i], "pipelined")
        outs = [ctx.output(*sc.safe_caps(hosts[i])) for i in idx]
        tickets = [ctx.submit(devs[i], o) for i, o in zip(idx, outs)]
        assert all(ctx.poll(t) == sc.SC_OK for t in tickets)
        for i, o in zip(idx, outs):
            compare_clusters(*o.to_numpy()[:2], refs[i], "served")
