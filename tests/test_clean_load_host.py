"""Cleanup's loads at the end of a list, up to the longest one (2^32 - 1 elements),
on the CPU, under AddressSanitizer."""
from _kernel_source import run


def test_loads_end_with_the_list(tmp_path):
    r = run(tmp_path, "clean_load.cpp",
            [r"^constexpr int kCleanItems = ", r"^__device__ __forceinline__ void clean_load\("], "address")
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
