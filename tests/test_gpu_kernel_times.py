"""GPU: the kernel times in sc_stats are of eager launches. A graph replay records none, and must not
report an earlier launch's again.
"""
import pytest

import fedgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2101_11489_amd as sc  # noqa: E402
from gpu_common import make_ctx  # noqa: E402


def test_replays_report_no_kernel_time():
    cfg = fedgen.CONFIGS[0].with_(n_fed=8)
    cal = fedgen.make_calibration(cfg)
    e = fedgen.make_event(cfg, cal, 0)
    ev = sc.Event(e.zs, e.fed_offset).to_device()
    with make_ctx(cal.noise, cal.gain, cal.bad) as ctx:
        out = ctx.output(*sc.safe_caps(ev))
        dense = ctx.dense_buffer()

        def timed(call):
            before = ctx.stats()
            call()
            after = ctx.stats()
            return (after["kernels_timed"] - before["kernels_timed"],
                    after["kernel_ms_total"] - before["kernel_ms_total"], after["last_kernel_ms"])

        def batch():
            ctx.process_events([ev], [out])

        for earlier in (batch, lambda: ctx.unpack(ev, dense), lambda: ctx.cluster(dense, out)):
            ctx.tuning = {"use_graph": 0}
            n, ms, last = timed(earlier)
            assert n == 1 and last > 0.0 and ms == pytest.approx(last, rel=1e-6)
            ctx.tuning = {"use_graph": 1}
            for _ in range(2):
                assert timed(batch) == (0, 0.0, -1.0)
