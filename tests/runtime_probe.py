"""Compiles the host runtime (sc_runtime.cpp) for the CPU into small programs that print what its internal
functions decide; the kernel side is stubbed (256 compute units' worth of the residency that the
shapes' LDS allows)."""
import os
import subprocess

from paper_2101_11489_amd import build

STUBS = r"""
#include "sc_runtime.cpp"
namespace sc {
hipError_t static_scratch_address(void**) { return hipErrorUnknown; }
hipError_t launch_derive_calib(const float*, const float*, const uint8_t*, uint32_t, float*, float*,
                               hipStream_t) { return hipErrorUnknown; }
hipError_t launch_reset(const FusedArgs&, uint32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_fused(const FusedArgs&, uint32_t, uint32_t, uint32_t, uint32_t, hipStream_t) {
    return hipErrorUnknown;
}
hipError_t add_fused(hipGraph_t, hipGraphNode_t*, const FusedArgs&, uint32_t, uint32_t, uint32_t,
                     uint32_t) { return hipErrorUnknown; }
hipError_t launch_cluster_dense(const uint8_t*, const FusedArgs&, uint32_t, uint32_t, uint32_t,
                                uint32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_unpack(const uint8_t*, const uint64_t*, uint32_t, uint8_t*, uint8_t*, EventResult*,
                         hipStream_t) { return hipErrorUnknown; }
hipError_t launch_hits(const HitDesc*, uint32_t, uint32_t, const uint32_t*, const float*, uint32_t,
                       hipStream_t) { return hipErrorUnknown; }
uint32_t stage_bytes_of(uint32_t stage) { return stage ? stage : 6656u; }
bool tile_shape_supported(uint32_t, uint32_t, uint32_t) { return true; }
bool tile_shape_supports_modules(uint32_t, uint32_t) { return true; }
int fused_blocks_per_cu(uint32_t w, uint32_t d, bool, bool, uint32_t stage) {
    return (int)(160 * 1024 / (4 * d + stage_bytes_of(stage) + 2400 + 16 * w));
}
}  // namespace sc
"""


def compile_probe(directory, main):
    """A function that runs the program `main` (its source) and returns what it prints, by words."""
    src, exe, lib = directory / "probe.cpp", directory / "probe", os.path.join(build.ROCM, "lib")
    src.write_text(STUBS + main)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(build.ROCM, "include"),
                    "-I", build.INCLUDE, "-I", build.CSRC, str(src), "-o", str(exe), "-L", lib,
                    "-lamdhip64", "-lpthread", "-Wl,-rpath," + lib], check=True)

    def run(*args):
        out = subprocess.run([str(exe), *(str(a) for a in args)], check=True, capture_output=True, text=True)
        return [line.split() for line in out.stdout.splitlines()]
    return run
