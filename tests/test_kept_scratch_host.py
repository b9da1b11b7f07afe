"""The scratch kept for bulk insertion and cleanup makes way: other handles and the
call's own levels get its memory when there is no other, and no more than 2 GiB
stay with a handle (the library's host code on the CPU, hipMalloc limited)."""
import os

from _kernel_source import HERE, run_host_code


def test_kept_scratch_makes_way(tmp_path):
    r = run_host_code(tmp_path, os.path.join(HERE, "kept_scratch.cpp"),
                      wrap=("_Z9hipMallocPPvm", "_Z7hipFreePv"))
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "kept scratch: ok" in r.stdout
