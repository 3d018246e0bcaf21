"""bench.py's accounting of what each kernel does."""
import pytest

import bench


# A call's kernels together do the layer's work, on either path past 32 rows
@pytest.mark.parametrize("bwd", [False, True])
@pytest.mark.parametrize("path", [("rowprep", "adapter_gemm", "adapter_finish", "tile_%s"),
                                  ("rowprep", "mid_%s", "mid_finish_%s")])
@pytest.mark.parametrize("r", [0, 384])
def test_kernel_flops_add_up(path, bwd, r):
    names = [n % ("bwd" if bwd else "fwd") if "%" in n else n for n in path]
    assert sum(bench.kernel_flops(n, 333, 11008, 4096, r, bwd) for n in names) == bench.layer_flops(333, 11008, 4096, r)
