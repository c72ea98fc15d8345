"""CPU: the launches that a batch gets (plan_launches in sc_runtime.cpp, compiled here with the kernel
side stubbed: 256 compute units, the residency that the shapes' LDS allows). The shape depends on the
FEDs' sizes where the host has them, is left to the device where it has not, and never depends on the
room in the outputs, which the plan is not told.
"""
import pytest

from runtime_probe import compile_probe

MAIN = r"""
// n_fed chunk waves tiles_per_cu stage | order n_ev host_bytes...: the FED bytes of each host event (all
// FEDs alike), 0 for a device event; chunk 0: the default tuning
int main(int argc, char** argv) {
    auto arg = [&](int i) { return (uint32_t)strtoul(argv[i], nullptr, 10); };
    sc_ctx c;
    c.n_cu = 256;
    c.n_fed = arg(1);
    c.tuning = kDefaultTuning;
    if (arg(2)) {
        const sc_tuning t{arg(2), arg(3), arg(4), 2, 1, arg(5)};
        if (sc_set_tuning(&c, &t) != SC_OK) return 1;
    }
    FedMix mix;
    const uint32_t n = arg(7);
    for (uint32_t i = 0; i < n; ++i) {
        const uint32_t bytes = arg(8 + (int)(i % (uint32_t)(argc - 8)));
        std::vector<uint64_t> fo(c.n_fed + 1);
        for (uint32_t f = 0; f <= c.n_fed; ++f) fo[f] = (uint64_t)f * bytes;
        add_event(mix, bytes ? fo.data() : nullptr, c.n_fed);
    }
    for (const Launch& l : plan_launches(&c, mix, n, arg(6)))
        std::printf("%u %u %u %u %u %u\n", l.shape.waves, l.shape.digis, l.shape.stage, l.grid,
                    l.one_each, l.pick);
}
"""
ORDINARY, LARGE = (2, 2880, 6656), (4, 6144, 10240)
DEVICE = 0


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    probe = compile_probe(tmp_path_factory.mktemp("launch_plan"), MAIN)

    def run(n_fed, n_ev, feds, order=2, tuning=(0, 0, 0, 0)):
        rows = [tuple(int(v) for v in line) for line in probe(n_fed, *tuning, order, n_ev, *feds)]
        return [(r[:3], r[5]) for r in rows], [r[3] for r in rows], [r[4] for r in rows]
    return run


@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("n_fed,n_ev", [(440, 20), (440, 64), (41, 27), (50, 32)])
def test_device_events_are_judged_by_the_device(plan, n_fed, n_ev, order):
    both = {(ORDINARY, 1), (LARGE, 2)}
    assert set(plan(n_fed, n_ev, [DEVICE], order)[0]) == both
    # also beside host events, whatever their sizes
    assert set(plan(n_fed, n_ev, [DEVICE, 1000], order)[0]) == both
    assert set(plan(n_fed, n_ev, [8000, 8000, 8000, DEVICE], order)[0]) == both


# FEDs past the small stage (6640 bytes) from one in 1024 on, long ones (6100 bytes) from one in eight
@pytest.mark.parametrize("n_ev,feds,shape", [
    (60, [6640] + 8 * [1], ORDINARY), (60, [6641], LARGE), (60, [6641] + 59 * [1], LARGE),
    (1024, [6641] + 1023 * [1], LARGE), (1025, [6641] + 1024 * [1], ORDINARY), (60, [6099], ORDINARY),
    (60, [6100], LARGE), (64, [6100] + 7 * [1], LARGE), (63, [6100] + 8 * [1], ORDINARY), (60, [1], ORDINARY)])
def test_host_events_are_judged_by_their_feds(plan, n_ev, feds, shape):
    assert plan(440, n_ev, feds)[0] == [(shape, 0)]


@pytest.mark.parametrize("feds", [[DEVICE], [1000], [8000]])
def test_small_launches_take_four_waves(plan, feds):
    launches, grid, one_each = plan(50, 1, feds)
    assert launches == [(LARGE, 0)] and grid == [56] and one_each == [1]
    assert plan(50, 1, feds, order=1)[1:] == ([50], [0])


def test_other_shapes_are_used_as_they_are(plan):
    for chunk, waves, stage in ((3072, 2, 6656), (6144, 4, 10240), (1024, 1, 6656), (2880, 2, 10240)):
        for n_ev, feds in ((1, [DEVICE]), (64, [DEVICE]), (64, [8000])):
            assert plan(440, n_ev, feds, tuning=(chunk, waves, 32, stage))[0] == [((waves, chunk, stage), 0)]


@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("n_fed,n_ev,feds", [(50, 1, [DEVICE]), (440, 2, [DEVICE]), (440, 64, [DEVICE]),
                                             (440, 64, [8000]), (440, 64, [8000, DEVICE]), (50, 1, [8000])])
def test_a_named_stage_pins_the_default_shape(plan, n_fed, n_ev, feds, order):
    pinned = plan(n_fed, n_ev, feds, order, tuning=(2880, 2, 32, 6656))
    assert pinned[0] == [(ORDINARY, 0)]
    assert plan(n_fed, n_ev, feds, order, tuning=(2880, 2, 32, 0)) == plan(n_fed, n_ev, feds, order)
