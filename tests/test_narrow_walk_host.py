"""The lane walks of counts and emission on the CPU, over dictionaries that hold
the largest key, 2^31 - 1, whose key variable is all ones: counts and pairs
against a search of all levels, reads under AddressSanitizer."""
from _kernel_source import run

PARTS = [
    r"^struct QLevel \{", r"^struct QLevels \{", r"^constexpr uint32_t kNoKey = ",
    r"^constexpr uint32_t kMaxKey = ", r"^__device__ __forceinline__ uint32_t skip_run\(",
    r"^constexpr int kNarrowLevels = ", r"^constexpr uint32_t kNarrowSteps = ",
    r"^struct NarrowWalk \{", r"^__device__ __forceinline__ bool count_narrow\(",
    r"^__device__ __forceinline__ bool emit_narrow\(",
]


def test_narrow_walk_at_the_largest_key(tmp_path):
    r = run(tmp_path, "narrow.cpp", PARTS, "address,undefined")
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "narrow walk: ok" in r.stdout
