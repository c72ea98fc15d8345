"""GPU: the default tuning at the sizes where its launches change, against the oracle. With 41 FEDs a
batch of n events has 48 n places (eight queues of 6 FEDs): up to 1024 of them every tile has a
workgroup of the large shape, up to 2048 one of the ordinary shape, and beyond that tiles go by ticket.
Outputs are of exactly the size needed, so that no capacity hints at the FEDs' sizes.
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

N_FED = 41


@pytest.fixture(scope="module")
def data():
    cfg = fedgen.CONFIGS[4].with_(n_fed=N_FED)
    cal = fedgen.make_calibration(cfg)
    evs = [fedgen.make_event(cfg.with_(occ=o), cal, i) for i, o in enumerate((0.06, 0.055, 0.005, 0.01))]
    refs = [oracle.process_event(e.zs, e.fed_offset, cal.noise, cal.gain, cal.bad) for e in evs]
    sizes = [np.diff(e.fed_offset.astype(np.int64)) for e in evs]
    assert sizes[0].min() > 6640 and sizes[2].max() < 5200
    return cal, evs, refs


# events 0, 1 have large FEDs, 2, 3 ordinary ones
@pytest.mark.parametrize("n", [1, 21, 22, 42, 43, 60])
@pytest.mark.parametrize("pattern", [(0, 1), (2, 3), (2, 3, 2, 3, 2, 3, 2, 0)])
@pytest.mark.parametrize("call", ["replay", "eager", "static", "host", "pipelined"])
def test_sizes(data, call, pattern, n):
    cal, evs, refs = data
    idx = [pattern[i % len(pattern)] for i in range(n)]
    src = [sc.Event(e.zs, e.fed_offset) for e in evs]
    if call != "host":
        src = [h.to_device() for h in src]
    with make_ctx(cal.noise, cal.gain, cal.bad) as ctx:
        if call == "eager":
            ctx.tuning = {"use_graph": 0}
        outs = [ctx.output(refs[i].cl.size, refs[i].adc.size) for i in idx]
        b = ctx.batch([src[i] for i in idx], outs)
        for rep in range(2):
            if call == "static":
                torch.cuda.synchronize()
                rc = sc.lib().sc_process_events_static(ctx._h, b.c_ev, b.n, b.c_out, b.c_st)
            elif call == "pipelined":
                rc, _ = ctx.process_pipelined(b.events, outs, n)
            else:
                rc, _ = ctx.process_batch(b)
            assert rc == sc.SC_OK
            for k, (i, o) in enumerate(zip(idx, outs)):
                compare_clusters(*o.to_numpy()[:2], refs[i], f"pass {rep} event {k}")
                o.cl.zero_()
                o.adc.zero_()


def test_events_that_change_between_calls(data):
    """One context and batch size, events of either kind in turn: each call's own events decide."""
    cal, evs, refs = data
    devs = [sc.Event(e.zs, e.fed_offset).to_device() for e in evs]
    with make_ctx(cal.noise, cal.gain, cal.bad) as ctx:
        for pattern in ((0, 1), (2, 3), (2, 3), (0, 1), (0, 1), (2, 3), 31 * (2,) + (0,), (3,)):
            idx = [pattern[i % len(pattern)] for i in range(50)]
            outs = [ctx.output(refs[i].cl.size, refs[i].adc.size) for i in idx]
            for call in ("replay", "static"):
                b = ctx.batch([devs[i] for i in idx], outs)
                torch.cuda.synchronize()
                if call == "static":
                    assert sc.lib().sc_process_events_static(ctx._h, b.c_ev, b.n, b.c_out, b.c_st) == sc.SC_OK
                else:
                    assert ctx.process_batch(b)[0] == sc.SC_OK
                for k, (i, o) in enumerate(zip(idx, outs)):
                    compare_clusters(*o.to_numpy()[:2], refs[i], f"{call} {pattern} event {k}")
                    o.cl.zero_()
                    o.adc.zero_()
