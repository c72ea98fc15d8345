"""CPU: the tiles by whose FED sizes a launch's workgroups choose their shape (sampled_tile in
sc_internal.h, compiled here). They must lie in the launch and meet every event (all of up to 512) and
every part of the detector, also where the numbers of events and of FEDs have factors in common with
theirs: else a few untypical events decide for a batch, or a busy one is overlooked.
"""
import os
import subprocess

import numpy as np
import pytest

from paper_2101_11489_amd import build

PROBE = r"""
#include <cstdio>
#include <cstdlib>
#include "sc_internal.h"
int main(int argc, char** argv) {
    for (int i = 1; i + 1 < argc; i += 2) {
        const uint32_t n_ev = strtoul(argv[i], nullptr, 10), n_fed = strtoul(argv[i + 1], nullptr, 10);
        const uint32_t shift = sc::sampled_shift(n_ev);
        for (uint32_t k = 0; k < 64u << shift; ++k) {
            const sc::SampledTile t = sc::sampled_tile(k, shift, n_ev, n_fed);
            std::printf("%u %u %u\n", i, t.e, t.f);
        }
    }
}
"""
SIZES = ([(e, f) for e in (1, 2, 3, 7, 8, 13, 16, 24, 32, 41, 63, 64, 65, 100, 256, 511, 512, 1000)
          for f in (1, 7, 8, 41, 50, 63, 64, 65, 96, 128, 256, 320, 384, 431, 440, 512, 20000)] +
         [(107374, 20000), (4880644, 440), (2147483647, 1)])


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    d = tmp_path_factory.mktemp("sampled_tiles")
    src, exe = d / "probe.cpp", d / "probe"
    src.write_text(PROBE)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(build.ROCM, "include"),
                    "-I", build.INCLUDE, "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe), *(str(v) for p in SIZES for v in p)], check=True, capture_output=True,
                         text=True).stdout
    rows = np.array(out.split(), dtype=np.int64).reshape(-1, 3)
    return {s: rows[rows[:, 0] == 2 * i + 1, 1:] for i, s in enumerate(SIZES)}


@pytest.mark.parametrize("n_ev,n_fed", SIZES)
def test_samples_meet_all_events_and_feds(tiles, n_ev, n_fed):
    e, f = tiles[n_ev, n_fed].T
    n = e.size
    assert n in (64, 128, 256, 512) and (n >= n_ev or n == 512) and (n < 2 * n_ev or n == 64)
    assert e.min() >= 0 and e.max() < n_ev and f.min() >= 0 and f.max() < n_fed
    assert f.max() + 4 <= max(n_fed, 4)                    # whole runs of four, where there are four
    assert np.unique(e).size == min(n, n_ev)
    feds = np.unique((f[:, None] + np.arange(4)).clip(0, n_fed - 1))
    assert feds.size >= min(n_fed, 256)
    # no event has more than its share, rounded up; nor has a FED (the last runs begin at one)
    assert np.unique(e, return_counts=True)[1].max() <= -(-n // n_ev)
    first, times = np.unique(f, return_counts=True)
    assert times[first < n_fed - 4].max(initial=0) <= -(-n // n_fed)
    # an event that has 8 or more of them has FEDs of every quarter of the detector
    if n_fed >= 16:
        for ev in np.unique(e):
            if (e == ev).sum() >= 8:
                assert np.unique(f[e == ev] * 4 // n_fed).size == 4
