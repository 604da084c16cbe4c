"""Host code of the library that decides without a GPU, compiled by itself."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2503_17405_amd", "csrc")


def compiled(tmp_path, body):
    """The lines that `body` (the inside of main) prints."""
    src, exe = tmp_path / "unit.cpp", tmp_path / "unit"
    src.write_text('#include <cstdio>\n#include "fsmmc_host.h"\nusing namespace fsmmc;\nint main()\n{\n%s\n}\n' % body)
    r = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src),
                        "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return r.stdout.split()


def test_memory_that_kernels_reach(tmp_path):
    # of device memory only the job's own device's; managed and pinned memory of any;
    # nothing whose device address differs or that HIP does not know
    out = compiled(tmp_path, """
    char x[2];
    auto at = [&](hipMemoryType t, int dev, void* p) {
        hipPointerAttribute_t a{};
        a.type = t;
        a.device = dev;
        a.devicePointer = p;
        return (int)reaches(a, x, 1);
    };
    std::printf("%d %d ", at(hipMemoryTypeDevice, 1, x), at(hipMemoryTypeDevice, 0, x));
    std::printf("%d %d ", at(hipMemoryTypeManaged, 1, x), at(hipMemoryTypeManaged, 0, x));
    std::printf("%d %d ", at(hipMemoryTypeHost, 1, x), at(hipMemoryTypeHost, 0, x));
    std::printf("%d %d ", at(hipMemoryTypeHost, 1, x + 1), at(hipMemoryTypeUnregistered, 1, x));
    """)
    assert out == ["1", "0", "1", "1", "1", "1", "0", "0"]
