"""The benchmark's trace summaries: kernel-name patterns against the built library's kernels, and traces without a
dispatch of the asked family refused."""
import argparse
import re
import subprocess

import pytest

from paper_2505_20600_amd import build as B
from tests.test_bench_overlap import bench


@pytest.fixture(scope="module")
def kernels():
    """The library's kernels as a profiler names them."""
    import os
    if not os.path.exists(B.LIB):
        B.build()
    out = subprocess.run(["nm", "-C", B.LIB], capture_output=True, text=True, check=True).stdout
    return [l.split(maxsplit=2)[2].replace("__device_stub__", "") for l in out.splitlines() if "__device_stub__" in l]


def test_families_take_every_kernel_of_their_class(kernels):
    def of(family):
        return {k for k in kernels if re.search(bench.FAMILY[family][0], k)}

    for family in bench.FAMILY:
        assert of(family), family
    assert of("attention") == {k for k in kernels if "attention_dma_kernel" in k}
    gemms = [of(f) for f in ("gemm_up", "gemm_qkv", "gemm_out", "gemm_down")]
    assert sum(map(len, gemms)) == len(set().union(*gemms))        # told apart
    for n, g in enumerate(gemms):                                  # both main loops in each
        assert any("gemm_dl_kernel" in k for k in g) and any("gemm_pp_kernel" in k for k in g)
    rest = {k for k in kernels if re.search("gemm_(dl|pp)_kernel", k)} - set().union(*gemms)
    assert all(k.split("(ms::GemmDesc)")[0].endswith(", 0>") for k in rest)   # the plain bias epilogue: no class


def test_summary_without_a_dispatch_of_the_family_is_refused(tmp_path):
    trace = tmp_path / "t.csv"
    rows = ["Kernel_Name,Start_Timestamp,End_Timestamp", "spin_kernel,0,10", "other_kernel(int),20,30",
            "spin_kernel,40,50"]
    trace.write_text("\n".join(rows) + "\n")
    args = argparse.Namespace(summarize_trace=str(trace), family="attention", counters=[], pmc_fetch="", pmc_write="",
                              copy_fetch="", copy_write="")
    with pytest.raises(SystemExit, match="no dispatch of family attention"):
        bench.summarize_trace(args)
