"""Host-side rules of the library that need no GPU, compiled with g++ and driven directly."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1912_08756_amd", "csrc")


def _run(tmp_path, driver, *sources):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(driver)
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, "-o", str(exe), str(src)]
                   + [a for s in sources for a in ("-x", "c++", os.path.join(CSRC, s))], check=True, timeout=120)
    return subprocess.run([str(exe)], check=True, timeout=60, stdout=subprocess.PIPE, text=True).stdout.split()


def test_dynamic_lds_is_allowed_again_when_a_call_needs_more(tmp_path):
    """The runtime's functions are replaced by ones that write down what they were asked for: a kernel's opt-in follows the most
    any call has needed, per device and kernel, and is not repeated for less."""
    out = _run(tmp_path, """
#include "icq_lds.h"
#include <stdio.h>
static int device = 0, fails = 0;
hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *) { *a = {}; a->sharedSizeBytes = 4; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int n) {
    printf("%d:%s:%d\\n", device, static_cast<const char *>(f), n);
    return fails ? hipErrorInvalidValue : hipSuccess;
}
int main() {
    const char *a = "a", *b = "b", *c = "c";
    for (int n : {100, 100, 300, 200, 300, 301}) if (icq_allow_lds(a, n) != hipSuccess) return 1;
    if (icq_allow_lds(b, 50) != hipSuccess) return 2;
    device = 1;
    if (icq_allow_lds(a, 70) != hipSuccess) return 3;
    fails = 1;
    if (icq_allow_lds(a, 80) == hipSuccess) return 4;
    fails = 0;
    if (icq_allow_lds(a, 75) != hipSuccess) return 5;
    return icq_allow_lds(c, 10, true) == hipErrorInvalidValue ? 0 : 6;
}
""", "icq_lds.hip")
    assert out == ["0:a:100", "0:a:300", "0:a:301", "0:b:50", "1:a:70", "1:a:80", "1:a:75"]


def test_scan_pieces_are_those_of_the_search_over_every_number(tmp_path):
    """The steps per block that follow from the rule are those that looking at every number of pieces gives (of equal costs the
    fewest rounds), for a handful of queries to thousands of groups; and it looks at few of them."""
    out = _run(tmp_path, """
#include "icq_pieces.h"
#include <chrono>
#include <initializer_list>
#include <stdio.h>
static int64_t every(int num_cu, int64_t groups, int64_t steps, int64_t fill) {
    int64_t best = 1, least = -1;
    const int64_t most = 2 * ((num_cu + groups - 1) / groups) + 2;
    for (int64_t c = 1; c <= most && c <= steps; ++c) {
        const int64_t cost = (groups * c + num_cu - 1) / num_cu * ((steps + c - 1) / c + fill);
        if (least < 0 || cost < least) { least = cost; best = c; }
    }
    return best;
}
int main() {
    long n = 0;
    for (int cu : {256, 304, 7}) for (int64_t g = 1; g < 2200; g = g < 600 ? g + 1 : g + 61)
        for (int64_t steps = 0; steps < 9000; steps = steps < 70 ? steps + 1 : steps * 9 / 8 + 1)
            for (int64_t fill : {1, 2, 8}) {
                const int64_t a = icq_scan_pieces(cu, g, steps, fill), b = every(cu, g, steps, fill);
                if (a < 1 || (steps > 0 && a > steps)) return 1;
                if ((steps + a - 1) / a != (steps + b - 1) / b) return 2;
                ++n;
            }
    volatile int64_t sink = 0;
    double t[2];
    for (int w = 0; w < 2; ++w) {
        const auto t0 = std::chrono::steady_clock::now();
        for (int i = 0; i < 3000; ++i) sink += w ? every(256, 1 + sink % 2, 6000 + i, 2) : icq_scan_pieces(256, 1 + sink % 2, 6000 + i, 2);
        t[w] = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    }
    printf("%ld %d\\n", n, t[0] * 10 < t[1]);
}
""")
    assert int(out[0]) > 100_000 and out[1] == "1"
