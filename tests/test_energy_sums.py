"""The energy arithmetic of the packed-row kernels on the CPU: their move
entries carry a flag in the top bit, so sums of accepted moves pass 2^31.  The
device header's own functions are compiled for the host with every signed
overflow a trap (it would be undefined, whatever today's code generation makes
of it) and compared with exact integers."""
import os
import subprocess

from paper_2509_17837_amd import build as B

PROGRAM = r"""
#include "xzzx_device.h"
#include <cstdio>
#include <cstdlib>
using namespace xzzx;
int main()
{
    const int32_t des[] = {0, -1, 1, -70000, 70000, -1200000000, 1200000000, -2147483647};
    const uint32_t thrs[] = {0u, 1u, 0x7FFFFFFFu, 0x80000000u, 0xFFFFFFFFu};
    unsigned seed = 1;
    for (int trial = 0; trial < 20000; ++trial) {
        // accepted moves one after another, the energy staying in [0, 2^31)
        uint32_t acc = 0;
        const int64_t start = (int64_t)(rand_r(&seed) % 0x7FFFFFFFu);
        int64_t want = start;
        for (int m = 0; m < 32; ++m) {
            const int32_t de = des[rand_r(&seed) % 8];
            const bool taken = rand_r(&seed) % 4 != 0 && want + de >= 0 && want + de < (1ll << 31);
            take_move(acc, move_entry(de, thrs[rand_r(&seed) % 5]), taken ? 0xFFFFFFFFu : 0u);
            if (taken) want += de;
        }
        const int32_t got = add_energy((int32_t)start, acc);
        if (got != want) { std::printf("trial %d: %d, not %lld\n", trial, got, (long long)want); return 1; }
    }
    return 0;
}
"""


def test_energy_sums_are_defined_and_exact(tmp_path):
    src, exe = tmp_path / "sums.hip", tmp_path / "sums"
    src.write_text(PROGRAM)
    check = "signed-integer-overflow"
    subprocess.check_call([B.hipcc(), "-O1", "-std=c++17", "--cuda-host-only", "-x", "hip", str(src), "-I", B.CSRC,
                           "-I", os.path.join(B.ROOT, "include"), "-Xarch_host", f"-fsanitize={check}",
                           "-Xarch_host", f"-fsanitize-trap={check}", "-w", "-o", str(exe)])
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, f"exit {run.returncode} {run.stdout}"
