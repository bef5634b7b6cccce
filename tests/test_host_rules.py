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
