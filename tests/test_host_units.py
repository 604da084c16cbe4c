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


def test_idle_buffers(tmp_path):
    # kept up to the bound, the oldest given back for newer ones, handed out when
    # they fit within a quarter; all of them back at a release and when the last
    # context closes; none kept without one
    out = compiled(tmp_path, """
    static int freed;
    IdlePool q(100, [](void* p) { freed = 10 * freed + (int)(size_t)p; });
    auto say = [](int v) { std::printf("%d ", v); };  // a value each: arguments have no order
    auto give = [&](int i, size_t bytes) { say(q.give((void*)(size_t)i, bytes)); };
    auto take = [&](size_t bytes) {
        size_t got = 0;
        say((int)(size_t)q.take(bytes, &got));
        say((int)got);
    };
    give(9, 10);
    q.open();
    q.open();
    give(1, 40), give(2, 60), say(freed), give(8, 101), say(freed);
    give(3, 30), say(freed);
    take(45), take(61), take(50), take(30), take(30);
    give(4, 50), give(5, 50);
    q.release(), say(freed);
    give(6, 100);
    q.close(), say(freed);
    q.close(), say(freed);
    give(7, 1);
    """)
    assert " ".join(out) == ("0 "                       # no context
                             "1 1 0 0 0 "               # up to the bound, not past it
                             "1 1 "                     # the oldest goes
                             "0 0 0 0 2 60 3 30 0 0 "   # more than a quarter over, too small, taken
                             "1 1 145 "                 # released, oldest first
                             "1 145 1456 "              # the last context
                             "0")
