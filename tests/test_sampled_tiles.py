"""CPU: the 64 tiles by whose FED sizes a launch's workgroups choose their shape (sampled_tile in
sc_internal.h, compiled here). They must lie in the launch and meet every event (64 of more) and every
part of the detector, also where the numbers of events and of FEDs have factors in common with 64:
else a few untypical events decide for a batch.
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
    for (int i = 1; i + 1 < argc; i += 2)
        for (uint32_t k = 0; k < 64; ++k) {
            const sc::SampledTile t = sc::sampled_tile(k, strtoul(argv[i], nullptr, 10),
                                                       strtoul(argv[i + 1], nullptr, 10));
            std::printf("%u %u\n", t.e, t.f);
        }
}
"""
SIZES = ([(e, f) for e in (1, 2, 3, 7, 8, 13, 16, 24, 32, 41, 63, 64, 65, 100, 256, 1000)
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
    return dict(zip(SIZES, np.array(out.split(), dtype=np.int64).reshape(len(SIZES), 64, 2)))


@pytest.mark.parametrize("n_ev,n_fed", SIZES)
def test_samples_meet_all_events_and_feds(tiles, n_ev, n_fed):
    e, f = tiles[n_ev, n_fed].T
    assert e.min() >= 0 and e.max() < n_ev and f.min() >= 0 and f.max() < n_fed
    assert np.unique(e).size == min(64, n_ev) and np.unique(f).size == min(64, n_fed)
    # no event or FED has more of the 64 than its share, rounded up
    assert np.unique(e, return_counts=True)[1].max() <= -(-64 // n_ev)
    assert np.unique(f, return_counts=True)[1].max() <= -(-64 // n_fed)
    # an event that has 8 or more of them (the choice is by 16) has FEDs of every quarter of the detector
    if n_fed >= 4:
        for ev in np.unique(e):
            if (e == ev).sum() >= 8:
                assert np.unique(f[e == ev] * 4 // n_fed).size == 4
