"""The offsets at which the fp16-pair kernel asks for its weights, replayed on the host with the kernel's own code (struct
PairWalk): every step of every wave finds its weights, and nothing lies outside the section."""
import os
import subprocess

import pytest

from paper_1802_10280_amd import build as esc_build

SOURCE = r"""
#include <cstdio>
#include "pair.h"
using namespace escoin;
int main() {
    const PairShape shapes[] = {{1, 1, 4}, {1, 1, 8}, {1, 2, 2}, {2, 1, 2}};
    const int channels[] = {16, 17, 33, 49, 64, 77, 100, 128, 143, 196, 250, 256, 384, 512}, taps[] = {1, 3, 4, 6, 9, 12, 15, 25},
              rows[] = {32, 64, 65, 90, 128, 136, 192, 250, 284, 384};
    long long asked = 0;
    for (const PairShape& s : shapes)
        for (int C : channels)
            for (int RS : taps)
                for (int M : rows) {
                    Dims d = {};
                    d.C = C, d.M = M, d.R = 1, d.S = RS;
                    const long long bytes = (long long)pair_weight_bytes(d);
                    const int chunks = (int)mfma_chunks(d), total = chunks * RS;
                    for (int mg = 0; mg < (M + 64 * s.MW - 1) / (64 * s.MW); ++mg)
                        for (int wm = 0; wm < s.MW; ++wm)
                            for (int kg = 0; kg < s.KW; ++kg) {
                                PairWalk w(s.KW, RS, chunks, PairWalk::row_block(mg, s.MW, wm, M), kg);
                                const bool rows_there = 64 * (mg * s.MW + wm) < M;
                                auto ask = [&](int step) {  // -1: one past the wave's last
                                    for (int p = 0; p < 2; ++p) {
                                        const long long at = w.at + (long long)p * w.block_bytes;
                                        if (at < 0 || at + kPairStepBytes > bytes) {
                                            printf("layout %d%d%d C %d RS %d M %d: offset %lld of %lld\n", s.MW, s.PW, s.KW, C, RS, M, at, bytes);
                                            return false;
                                        }
                                        const long long want = ((long long)(2 * (mg * s.MW + wm) + p) * total + step) * kPairStepBytes;
                                        if (rows_there && step >= 0 && at != want) {
                                            printf("layout %d%d%d C %d RS %d M %d step %d: offset %lld, not %lld\n", s.MW, s.PW, s.KW, C, RS, M, step, at, want);
                                            return false;
                                        }
                                    }
                                    ++asked;
                                    w.next();
                                    return true;
                                };
                                for (int round = 0; round < w.n_rounds; ++round)
                                    for (int i = w.first_step(round, kg); i < w.first_step(round, kg + 1); ++i)
                                        if (!ask(round * s.KW * RS + i)) return 1;
                                if (!ask(-1) || !ask(-1)) return 1;
                            }
                }
    printf("%lld\n", asked);
    return 0;
}
"""


def test_weight_offsets_stay_in_the_section(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc here")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(SOURCE)
    include = os.path.join(esc_build.ROOT, "include")
    subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-Wno-unused-function", "-I", include, "-I", esc_build.CSRC,
                    "-o", str(exe), str(src)], check=True, timeout=300)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout
    assert int(res.stdout) > 1_000_000
