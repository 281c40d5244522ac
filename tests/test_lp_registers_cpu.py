"""The 256x256 low-precision kernels, sixteen waves at 128 registers each, hold
their stage loops without scratch memory (gfx950 assembly of our own sources,
compiled on the CPU).  A value kept for a seldom taken branch is enough to push
one of them over."""
import re

from test_codegen_cpu import _device_asm

LAYOUTS = ((0, 0), (0, 1), (1, 0), (1, 1))


def test_no_scratch_in_the_largest_tiles(tmp_path):
    inst = "".join(f"template __global__ void gemm_lp_dma_kernel<{eb}, 256, 256, 8, {bk}, {ta}, {tb}>(GemmArgs);\n"
                   for eb, bk in ((2, 64), (1, 128)) for ta, tb in LAYOUTS)
    asm = _device_asm(tmp_path, "gemm_lp_dma.hpp", inst)
    sizes = dict(re.findall(r"\.amdhsa_kernel (\S+)\n\s+\.amdhsa_group_segment_fixed_size \d+\n"
                            r"\s+\.amdhsa_private_segment_fixed_size (\d+)", asm))
    assert len(sizes) == 8
    assert all(int(v) == 0 for v in sizes.values()), sizes
