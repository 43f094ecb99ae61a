"""Compile-time checks of host and device arithmetic that no run of ordinary size
reaches (the kernels' headers, host pass only)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_10783_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def compiles(tmp_path, checks):
    src = tmp_path / "checks.hip"
    src.write_text('#include "ezo_kernels.hpp"\nusing namespace ezo;\n' + "\n".join(checks) + "\n")
    return subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only", "--offload-host-only",
                           "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src)], capture_output=True, text=True)


def test_candidate_lists_fit_their_counts(tmp_path):
    """Edges x candidates of a call may pass 2^31 (300 000 edges x 10 000 samples of
    a small arm fit the card's memory): the lists they are split into do not, hold
    every edge, and are one for calls of ordinary size."""
    r = compiles(tmp_path, [
        "constexpr bool fits(int64_t edges, int cap) {",
        "  const int g = list_group(cap), n = list_count((int)edges, g);",
        "  return g >= 1 && (g == 1 || (int64_t)g * cap <= kListMost) && (int64_t)n * g >= edges && (int64_t)(n - 1) * g < edges; }",
        "static_assert(kListMost < (1ll << 31) && fits(300000, 10000) && fits(65535, 57344) && fits(1, 2147483647));",
        "static_assert(fits(3, 1 << 28) && fits(3, (1 << 28) + 1) && fits(7, 1) && fits(5, 0) && fits(1 << 20, 16384));",
        "static_assert(list_count(96, list_group(10000)) == 1 && list_count(26843, list_group(10000)) == 1);",
        "static_assert(list_count(26844, list_group(10000)) == 2 && list_count(300000, list_group(10000)) == 12);",
    ])
    assert r.returncode == 0, r.stderr[-2000:]
