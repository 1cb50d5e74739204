"""The price by which the splitting kernel picks its tile shape, against exact integers over the sizes that a layer may have
(T up to 2^24, d_model up to 2^16, d_ff up to 2^18).  (No GPU: the header is compiled for the host.)"""
import os
import subprocess

from paper_2308_15030_amd import build

MAIN = """
#include <cstdio>
#include "split_price.h"
int main() {
    float rounds, per;
    int w, h;
    while (std::scanf("%f %f %d %d", &rounds, &per, &w, &h) == 4) std::printf("%.9g\\n", smoe_split_price(rounds, per, w, h));
}
"""


def test_price(tmp_path):
    src, exe = tmp_path / "price.cpp", tmp_path / "price"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    asked, exact = [], []
    for d_model, d_ff, T, K in ((256, 768, 600, 5), (768, 3072, 4096, 16), (1024, 4096, 16000, 128), (65536, 262144, 1 << 24, 256),
                                (65536, 32, 1 << 24, 1), (32, 262144, 1 << 24, 256)):
        per = -(-(d_ff // 16) // 4)
        for w in range(1, 5):
            for h in range(1, 5):
                items = (T // 32 // h + K) * -(-(d_model // 32) // w)
                rounds = -(-items // 256)
                asked.append(f"{rounds} {per} {w} {h}")
                exact.append(rounds * (per * (15 * (w + h) + 4 * w * h) + 157 * w * h))
    assert max(exact) > 2 ** 33
    out = subprocess.run([str(exe)], input="\n".join(asked), capture_output=True, text=True, check=True).stdout.split()
    for got, want, what in zip(out, exact, asked):
        assert abs(float(got) - want) <= 4 * 2 ** -24 * want, what      # four roundings of 24 bits
    assert len(out) == len(exact)
