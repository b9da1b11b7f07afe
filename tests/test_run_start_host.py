"""The walk back to the start of a key's run on the CPU, under AddressSanitizer."""
from _kernel_source import run


def test_run_start(tmp_path):
    r = run(tmp_path, "run_start.cpp", [r"^__device__ __forceinline__ uint32_t run_start\("],
            "address,undefined")
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
