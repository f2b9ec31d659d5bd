"""CPU run of the kernel that ends a round of few labels (k_dadm_end),
compiled from its own text: one thread per lane, barriers that count the lanes
still running, and an LPDev whose stop flag is set by the first workgroup
while another one runs, so that the other's waves do not all see the same
value. The label weights have to come out as if nothing had happened: the
round that sets the flag moved nothing."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ADMIT = os.path.join(ROOT, "paper_1710_08231_amd", "csrc", "admit.hpp")

SHIM = r"""
#include <barrier>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <thread>
#include <vector>
using std::int32_t; using std::int64_t;
#define __global__
#define __device__
#define __forceinline__ inline
#define __launch_bounds__(x)
#define __shared__ static
struct Dim { int x; };
static thread_local Dim threadIdx, blockIdx;
static std::unique_ptr<std::barrier<>> wg, wave[4];
static void __syncthreads() { wg->arrive_and_wait(); }
constexpr int kWave = 64;
static int first_late = 0;  // waves of workgroup 1 from here on see the flag set
struct Flag {
    int32_t v = 0;
    operator int32_t() const { return blockIdx.x == 1 ? (int)threadIdx.x / kWave >= first_late : v; }
    Flag &operator=(int32_t x) { v = x; return *this; }
};
struct LPDev { int32_t round, rounds_run, prev_moves, round_moves; int64_t total_moves; Flag done; };
struct AdmitCtx {
    int32_t nlabels, ntiles, ncol;
    int64_t *W, *part;
    int32_t *tmoves;
    LPDev *dev;
};
template <int BLOCK, typename T>
T block_sum(T x, T *tmp) {  // the lanes' sum by wave, then the waves' sums, as on the GPU
    static T lanes[BLOCK];
    const int w = threadIdx.x / kWave;
    lanes[threadIdx.x] = x;
    wave[w]->arrive_and_wait();
    if (threadIdx.x % kWave == 0) {
        tmp[w] = 0;
        for (int i = 0; i < kWave; i++) tmp[w] += lanes[w * kWave + i];
    }
    __syncthreads();
    T r = 0;
    for (int i = 0; i < BLOCK / kWave; i++) r += tmp[i];
    __syncthreads();
    return r;
}
"""

MAIN = r"""
int main(int argc, char **argv) {
    first_late = std::atoi(argv[1]);
    const int tiles = 256, labels = 2;
    std::vector<int64_t> W{100, 200}, part(labels * tiles, 0);
    std::vector<int32_t> tmoves(labels + tiles, 0);
    LPDev dev{};
    dev.round = 1;
    AdmitCtx c{labels, tiles, labels + tiles, W.data(), part.data(), tmoves.data(), &dev};
    const auto run = [&](int b) {
        wg = std::make_unique<std::barrier<>>(256);
        for (auto &x : wave) x = std::make_unique<std::barrier<>>(kWave);
        std::vector<std::thread> t;
        for (int i = 0; i < 256; i++)
            t.emplace_back([&, b, i] {
                blockIdx.x = b;
                threadIdx.x = i;
                k_dadm_end(c);
                wg->arrive_and_drop();  // a barrier counts the waves that still run
            });
        for (auto &x : t) x.join();
    };
    // a round before it leaves its sums in the shared memory
    for (int i = 0; i < tiles; i++) part[tiles + i] = 7;
    const int late = first_late;
    first_late = 4;
    run(1);
    for (int i = 0; i < tiles; i++) part[tiles + i] = 0;
    first_late = late;
    const int64_t before = W[1];
    run(1);
    run(0);
    std::printf("%lld %lld %d %d %d\n", (long long)(before - 200), (long long)(W[1] - before), dev.done.v, dev.round, dev.rounds_run);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    text = open(ADMIT).read()
    body = text[text.index("// Round bookkeeping by one workgroup"):text.index("// ------", text.index("void k_dadm_end("))]
    d = tmp_path_factory.mktemp("admit_end")
    src, exe = d / "end.cpp", d / "end"
    src.write_text(SHIM + body + MAIN)
    subprocess.run(["g++", "-std=c++20", "-O1", "-pthread", "-o", str(exe), str(src)], check=True)
    return str(exe)


@pytest.mark.parametrize("first_late", [0, 1, 2, 3, 4])
def test_stop_flag_set_while_other_workgroups_run(program, first_late):
    out = subprocess.run([program, str(first_late)], check=True, capture_output=True, text=True, timeout=60).stdout
    applied, stray, done, rnd, run = map(int, out.split())
    assert applied == 7 * 256  # a round with moves: all tiles' changes, once
    assert stray == 0  # the round that sets the flag: none
    assert (done, rnd, run) == (1, 2, 2)
