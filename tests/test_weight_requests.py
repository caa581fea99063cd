"""Which bytes the gate/up product of up to 32 rows requests from its weights, computed on the host by the kernel's own code: the loads' range check
drops a lane's request if its offset is not below `bytes - base`, a difference of unsigned 32-bit numbers that wraps where the base is the larger one."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2412_07017_amd", "csrc")

PROGRAM = r'''
#include "weight_tile.h"
#include <cstdio>
#include <cstdlib>
#include <vector>

using namespace asynclm;

int main(int argc, char** argv) {
    const int waves = 4 * atoi(argv[1]);
    for (int a = 2; a + 1 < argc; a += 2) {
        const int F = atoi(argv[a]), K = atoi(argv[a + 1]), rp = gate_rows_per_wave(F, waves), tiles = (F + rp - 1) / rp;
        const long long row = 2LL * K;
        const bf16_t* W = (const bf16_t*)(uintptr_t)(1ULL << 40);
        long long outside = 0, wrong = 0, idle = 0;
        std::vector<long long> got(2 * (size_t)F);                    // bytes taken of every row
        for (int wave = 0; wave < (tiles + 3) / 4 * 4; ++wave) {
            const int n0 = wave * rp, nr = gate_rows(F, n0, rp);
            idle += nr == 0;
            for (int lane = 0; lane < 64; ++lane) {
                const WeightTile t = gate_up_tile(W, F, K, n0, nr, lane);
                for (int blk = 0; blk < K / 128 + 3; ++blk) {         // three blocks past the end of the run
                    const RunPart p = weight_part(t, blk < K / 128 ? blk : 0, blk < K / 128);
                    for (int q = 0; q < 8; ++q) {
                        if (!(t.off[q] < p.bytes - p.base)) continue;
                        const long long at = (long long)((uintptr_t)(q < 4 ? t.w0 : t.w1) - (uintptr_t)W) + t.off[q] + p.base;
                        if (at < 0 || at + 16 > 2LL * F * row) { ++outside; continue; }
                        if (blk >= K / 128) ++wrong;
                        got[at / row] += 16;
                    }
                }
            }
        }
        for (long long b : got) wrong += b != row;
        printf("%d %d %lld %lld %lld\n", F, K, idle, outside, wrong);
    }
}
'''


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    from paper_2412_07017_amd.build import hipcc_path
    try:
        hipcc = hipcc_path()
    except RuntimeError:
        pytest.skip("no hipcc")
    tmp = tmp_path_factory.mktemp("requests")
    src, exe = str(tmp / "requests.hip"), str(tmp / "requests")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-w", "-I", CSRC, "-I", os.path.join(os.path.dirname(HERE), "include"), src, "-o", exe],
                   check=True, capture_output=True, text=True)
    return exe


# 256 compute units: 1024 waves to spread the gate rows over.  F = 2176, 2432 and 11008 leave waves of the last workgroup without rows, 128 and 14336 do not.
def test_a_gate_up_product_requests_every_weight_once_and_nothing_else(program):
    shapes = [(128, 256), (640, 128), (2176, 256), (2432, 384), (11008, 512), (14336, 512)]
    out = subprocess.run([program, "256"] + [str(v) for s in shapes for v in s], check=True, capture_output=True, text=True, timeout=100).stdout
    got = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert [g[:2] for g in got] == shapes
    assert [g[2] > 0 for g in got] == [False, False, True, True, True, False]
    assert all(g[3:] == (0, 0) for g in got), got
