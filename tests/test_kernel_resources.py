"""Workgroups per compute unit that the launch plans count on, from the
registers and LDS of the compiled kernels (no GPU needed): a compute unit has
four SIMDs with 512 registers a lane, given out by eight, and 160 KB of LDS."""

import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_2412_02962_amd import build

# kernel (a pattern of its mangled name), source, workgroups on a compute unit
KERNELS = [
    (r"gemm80_kernelILi2E", "gemm.hip", 3),
    (r"gemm80_kernelILi4E", "gemm.hip", 2),
    (r"gemm_dma_kernelILi0E", "gemm.hip", 3),
    (r"gemm_dma_kernelILi1E", "gemm.hip", 3),
    (r"gemm_dma_pair_kernelILi0E", "gemm.hip", 3),
    (r"gemm_wide_kernelILi64ELi128ELi2ELi2ELb0ELb1E", "gemm_wide.hip", 3),
    (r"gemm_wide_kernelILi64ELi128ELi2ELi3E", "gemm_wide.hip", 2),
    (r"gemm_wide_kernelILi256ELi160E", "gemm_wide.hip", 1),
    (r"attn_bf16_kernel", "attention_bf16.hip", 2),
    (r"attn_wide_kernel", "attention_wide.hip", 2),
]


def _metadata(src):
    """{kernel: (threads, registers, LDS bytes)} of one source, as it is built."""
    r = subprocess.run([build.hipcc()] + build.HIPCC_FLAGS + ["--cuda-device-only", "-S", "-o", "-",
                                                              os.path.join(build.CSRC, src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = {}
    for doc in re.split(r"\n  - \.agpr_count:", r.stdout)[1:]:
        field = lambda f: int(re.search(rf"\.{f}:\s+(\d+)", doc).group(1))
        out[re.search(r"\.name:\s+(_Z\S+)", doc).group(1)] = (field("max_flat_workgroup_size"), field("vgpr_count"),
                                                             field("group_segment_fixed_size"))
    return out


@pytest.fixture(scope="module")
def metadata():
    srcs = sorted({s for _, s, _ in KERNELS})
    with concurrent.futures.ThreadPoolExecutor(max_workers=4) as ex:
        return dict(zip(srcs, ex.map(_metadata, srcs)))


@pytest.mark.parametrize("pattern,src,per_cu", KERNELS, ids=lambda v: str(v))
def test_workgroups_per_compute_unit(metadata, pattern, src, per_cu):
    found = {k: v for k, v in metadata[src].items() if re.search(pattern, k)}
    assert found, f"no kernel {pattern} in {src}"
    for name, (threads, regs, lds) in found.items():
        waves = 4 * (512 // (-(-regs // 8) * 8))
        fit = min(waves * 64 // threads, (160 * 1024) // max(lds, 1))
        assert fit >= per_cu, (name, threads, regs, lds, fit)
