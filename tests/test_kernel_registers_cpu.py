"""Waves per SIMD of the evaluation and finite-difference kernels.

A SIMD holds 512 vector registers per lane, handed out eight at a time, so a
kernel of r registers runs floor(512 / r) waves on it.  The grids of these two
are a single round of a few waves per SIMD for the walker counts they are called
with: one wave less is another round.  Spilling to get there would not help."""
import shutil

import pytest

from built_code import kernel_registers, llvm_tool

# kernel, compiled MO width, waves
WANTED = ([("k_evalILi{}EdLi0ELb0ELi0EE", n, w) for n, w in ((4, 4), (8, 4), (12, 4), (16, 3), (20, 3))] +
          [("k_eval_fdILi{}EE", n, w) for n, w in ((4, 3), (8, 3), (12, 3), (16, 2), (20, 2), (24, 2), (32, 2))])


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    from paper_2506_09743_amd import build
    return kernel_registers(build.LIB, tmp_path_factory.mktemp("co"))


@pytest.mark.skipif(not shutil.which(llvm_tool("llvm-readelf")), reason="needs llvm-readelf")
@pytest.mark.parametrize("kernel,n_mo,waves", WANTED)
def test_waves_per_simd(kernels, kernel, n_mo, waves):
    name = kernel.format(n_mo)
    (regs, spilled), = [v for k, v in kernels.items() if name in k]
    assert 512 // (-(-regs // 8) * 8) >= waves and spilled == 0
