"""Rules on the kernel sources that no numerical test can see."""
import glob
import os

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_11430_amd", "csrc")


def test_wavefront_exchanges_are_fenced():
    """Lanes that exchange data through LDS without a workgroup barrier do so over wave_sync(), whose
    fences order the accesses; the bare scheduling barrier, which touches no memory, stands only there."""
    uses = {os.path.basename(p): open(p).read().count("__builtin_amdgcn_wave_barrier")
            for p in glob.glob(os.path.join(CSRC, "*.h*"))}
    assert {f: n for f, n in uses.items() if n} == {"wave_sync.h": 1}
