"""grp_steps (lstm_rec.h) called twice in a row by a workgroup, as the one-layer time loops call it: first for the
group's timesteps, then for those with more pieces than the few-pieces form takes.  The function's own source is
compiled for the host, a thread per wave; a wave that is held up right before it reads the result has to get the same
count as the others.  CPU only."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WAVES = 8

HARNESS = r"""
#include <atomic>
#include <barrier>
#include <chrono>
#include <cstdio>
#include <thread>
#include <vector>
struct Dim { unsigned x; };
static thread_local Dim threadIdx;
static const Dim blockDim = {%(waves)d};
static std::barrier<> the_barrier(%(waves)d);
static void __syncthreads() { the_barrier.arrive_and_wait(); }
static int held_up;   // this wave reads shared memory late
struct Shared {
    std::atomic<int> v{0};
    operator int() {
        if ((int)threadIdx.x == held_up) std::this_thread::sleep_for(std::chrono::milliseconds(100));
        return v;
    }
    void operator=(int n) { v = n; }
};
static void atomicAdd(Shared* s, int n) { s->v += n; }
%(source)s
int main() {
    int batch_sizes[] = {40, 33, 33, 20, 20, 17, 16, 9, 9, 9, 9, 4, 4, 2, 1, 1, 1};
    const int T = sizeof(batch_sizes) / sizeof(int);
    for (held_up = 0; held_up < (int)blockDim.x; ++held_up) {
        std::vector<int> alive(blockDim.x), many(blockDim.x);
        std::vector<std::thread> waves;
        for (unsigned w = 0; w < blockDim.x; ++w)
            waves.emplace_back([&, w] {
                threadIdx.x = w;
                alive[w] = grp_steps(batch_sizes, T, 3);
                many[w] = grp_steps(batch_sizes, T, 16);
            });
        for (auto& t : waves) t.join();
        for (unsigned w = 0; w < blockDim.x; ++w)
            if (alive[w] != 13 || many[w] != 6) {
                printf("wave %%d held up: wave %%u counts %%d and %%d\n", held_up, w, alive[w], many[w]);
                return 1;
            }
    }
    return 0;
}
"""


def test_two_counts_in_a_row(tmp_path):
    text = open(os.path.join(ROOT, "paper_2210_05064_amd", "csrc", "lstm_rec.h")).read()
    body = re.search(r"__device__ __forceinline__ int grp_steps\(.*?\n}\n", text, re.S).group(0)
    body = body.replace("__device__ __forceinline__", "static").replace("int32_t", "int").replace("__shared__ int", "static Shared")
    src = tmp_path / "steps.cpp"
    src.write_text(HARNESS % dict(waves=WAVES, source=body))
    subprocess.check_call(["g++", "-std=c++20", "-O1", "-pthread", "-o", str(tmp_path / "steps"), str(src)])
    done = subprocess.run([str(tmp_path / "steps")], stdout=subprocess.PIPE, text=True, timeout=60)
    assert done.returncode == 0, done.stdout
