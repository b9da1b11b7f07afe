"""The merge of runs larger than LDS on the CPU, a thread per lane with the
work-group's barriers and the waves' ballots only, under ThreadSanitizer."""
from _kernel_source import run

PARTS = [
    r"^struct alignas\(16\) LocalLds \{", r"^__device__ void lds_merge_pair\(",
    r"^__device__ __forceinline__ uint32_t seg_bound\(", r"^__device__ uint32_t wave_upper\(",
    r"^__device__ __forceinline__ void merge_large\(",
]


def test_barriers_of_the_large_merge(tmp_path):
    r = run(tmp_path, "large_merge.cpp", PARTS, "thread")
    assert "ThreadSanitizer" not in r.stderr, r.stderr[:4000]
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "large merge: ok" in r.stdout
