"""CPU: the cluster threshold on squares. Forming accepts a run where fl(q q) >= fl(S t2_hi) and rejects it
where fl(q q) < fl(S t2_lo), without the root of the definition, q >= fl(t fl(sqrt(S))); the runs that
neither test decides take the definition. Whatever is decided must agree with it: at the boundary, binary32
step by step, at the ends of the range of t, and for S that is 0, subnormal, huge or infinite. The factors
are the host runtime's own (device_calib, compiled here).
"""
import numpy as np
import pytest

from runtime_probe import compile_probe

MAIN = r"""
int main(int argc, char** argv) {
    sc_ctx c;
    for (int i = 1; i < argc; ++i) {
        c.t_cluster = strtof(argv[i], nullptr);
        const DeviceCalib d = device_calib(&c);
        std::printf("%a %a\n", d.t2_hi, d.t2_lo);
    }
}
"""
F = np.float32
INSIDE = [0.0, 2.0 ** -40, float(np.nextafter(F(2.0 ** -40), F(1))), 1e-9, 0.01, 0.3, 1.0, 3.0, 5.0, 7.3, 1e4,
          3.1e11, float(np.nextafter(F(2.0 ** 40), F(1))), 2.0 ** 40]
OUTSIDE = [1e-45, 1e-20, float(np.nextafter(F(2.0 ** -40), F(0))), float(np.nextafter(F(2.0 ** 40), F(2.0 ** 41))),
           1e25, 3e38]


@pytest.fixture(scope="module")
def factors(tmp_path_factory):
    rows = compile_probe(tmp_path_factory.mktemp("squares"), MAIN)(*(repr(t) for t in INSIDE + OUTSIDE))
    return {t: tuple(F(float.fromhex(v)) if v.lstrip("-") != "nan" else F(np.nan) for v in r)
            for t, r in zip(INSIDE + OUTSIDE, rows)}


def _charges():
    rng = np.random.default_rng(11489)
    top = 768 * 255   # the largest charge: a module row of full ADCs
    return np.unique(np.concatenate([np.arange(1, 300), rng.integers(1, top, 3000), 2 ** np.arange(17),
                                     top - np.arange(50)])).astype(F)


@pytest.mark.parametrize("t", INSIDE)
def test_squares_decide_as_the_definition(factors, t):
    hi, lo = factors[t]
    t, q = F(t), _charges()[:, None]
    # S beside (q / t)^2 by binary32 steps, then by parts in 2^24 to 2^16, and far from it
    with np.errstate(all="ignore"):
        S0 = ((q.astype(np.float64) / max(float(t), 1e-300)) ** 2).astype(F)
        near = [(S0.view(np.int32) + k).clip(0, 0x7f7fffff).astype(np.int32).view(F)
                for k in list(range(-40, 41)) + [s * 3 ** i for i in range(4, 10) for s in (-1, 1)]]
        far = [np.broadcast_to(F(v), q.shape) for v in (0.0, 1e-45, 3e-42, 1.1e-38, 1.2e-38, 1e-30, 1.0, 1e30, 3.4e38,
                                                          np.inf)]
        S = np.concatenate(near + far, axis=1)
        accepted = q >= t * np.sqrt(S)
        q2 = q * q
        s_hi, s_lo = S * hi, S * lo
    above, below = q2 >= s_hi, q2 < s_lo
    assert all(x.dtype == F for x in (S, q2, s_hi, s_lo))
    assert not (above & ~accepted).any() and not (below & accepted).any()
    if t > 0:   # what they leave open lies within a few parts in 2^19 of the boundary
        open_ = ~above & ~below & np.isfinite(S)
        ratio = S.astype(np.float64) * float(t) ** 2 / q.astype(np.float64) ** 2
        assert open_.any() and np.abs(ratio[open_] - 1.0).max() < 2.0 ** -18


@pytest.mark.parametrize("t", OUTSIDE)
def test_squares_decide_nothing_outside_their_range(factors, t):
    assert np.isnan(factors[t]).all()
