"""Rules of the kernel sources that no run shows reliably (CPU)."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KERNELS = os.path.join(ROOT, "paper_2108_07605_amd", "csrc", "kernels.hip")


def test_outer_columns_are_synchronised_within_the_wave():
    """layer_gradients passes the two outer columns from 54 lanes to two
    through LDS without a block barrier: between the write and the first read
    stands wave_sync, a release and acquire at wavefront scope with a wave
    barrier between."""
    text = re.sub(r"//[^\n]*", "", open(KERNELS).read())
    body = text[text.index("void layer_gradients("):]
    write, read = body.index("edges[lane] ="), body.index("&edges[")
    assert write < read
    assert "wave_sync();" in body[write:read]
    sync = re.search(r"void wave_sync\(\) \{(.*?)\n\}", text, re.S).group(1)
    order = ['__builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront")', "__builtin_amdgcn_wave_barrier()",
             '__builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront")']
    at = [sync.index(c) for c in order]
    assert at == sorted(at)
