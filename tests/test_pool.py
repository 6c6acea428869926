"""The serving pool allocator (host-side first-fit over one device block),
compiled on the CPU with g++ and exercised by a randomised harness: blocks
never overlap, accounting is exact, freed neighbours coalesce, and a fully
freed pool is one block again."""
import os
import subprocess

HARNESS = r'''
#include "mc_pool.hpp"
#include <cstdio>
#include <random>
#include <vector>
#include <algorithm>
using mc::Pool;
int main() {
    std::mt19937_64 rng(7);
    for (int trial = 0; trial < 50; ++trial) {
        const int64_t size = (int64_t)(1 + rng() % 4096) * 256 + (int64_t)(rng() % 255);
        Pool p(size);
        if (p.size() % 256 != 0 || p.size() > size) { std::puts("FAIL size"); return 1; }
        std::vector<std::pair<int64_t,int64_t>> live;
        int64_t used = 0;
        for (int op = 0; op < 2000; ++op) {
            if (live.empty() || rng() % 3 != 0) {
                const int64_t want = 1 + (int64_t)(rng() % (size / 8 + 1));
                const int64_t off = p.alloc(want);
                if (off < 0) {
                    if (p.largest_free() >= Pool::round_up(want)) { std::puts("FAIL refused"); return 1; }
                    continue;
                }
                const int64_t len = Pool::round_up(want);
                if (off % 256 || off + len > p.size()) { std::puts("FAIL bounds"); return 1; }
                for (auto &b : live)
                    if (off < b.first + b.second && b.first < off + len) { std::puts("FAIL overlap"); return 1; }
                live.emplace_back(off, len);
                used += len;
            } else {
                const size_t k = rng() % live.size();
                if (!p.release(live[k].first)) { std::puts("FAIL release"); return 1; }
                used -= live[k].second;
                live.erase(live.begin() + k);
            }
            if (p.in_use() != used) { std::puts("FAIL accounting"); return 1; }
        }
        if (p.release(-256)) { std::puts("FAIL bogus release"); return 1; }
        for (auto &b : live) p.release(b.first);
        if (p.in_use() != 0 || p.n_free_blocks() != 1 || p.largest_free() != p.size()) {
            std::puts("FAIL coalesce"); return 1;
        }
    }
    std::puts("OK");
    return 0;
}
'''


def test_pool_allocator(tmp_path):
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_31258_amd", "csrc")
    src = tmp_path / "pool_test.cpp"
    src.write_text(HARNESS)
    exe = tmp_path / "pool_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Xlinker", "--no-as-needed", "-fsanitize=address,undefined",
                    "-I" + csrc, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.strip()
    assert out == "OK"


STAGE = r'''
#include "mc_pool.hpp"
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>
struct Heap {
    static std::atomic<int> made, live;
    static char *make() { ++made; ++live; return new char[16]; }
    static void free(char *p) { --live; delete[] p; }
};
std::atomic<int> Heap::made{0}, Heap::live{0};
#define CHECK(x) do { if (!(x)) { std::printf("%d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
    static mc::StagePool<Heap> pool;
    for (int k = 0; k < 10; ++k) {  // one context after the other
        pool.join();
        for (int call = 0; call < 3; ++call) pool.put(pool.take());
        pool.leave();
        CHECK(Heap::live == 1);
    }
    CHECK(Heap::made == 1);
    for (int k = 0; k < 3; ++k) pool.join();  // several at once, more calls than pieces kept
    std::vector<char *> out;
    for (int k = 0; k < 7; ++k) out.push_back(pool.take());
    for (char *p : out) pool.put(p);
    CHECK(Heap::live == mc::kStageKept);
    pool.leave();
    pool.leave();
    char *late = pool.take();
    pool.leave();
    CHECK(Heap::live <= 2);
    pool.put(late);
    CHECK(Heap::live == 1);
    std::vector<std::thread> threads;
    for (int t = 0; t < 4; ++t)
        threads.emplace_back([] {
            for (int k = 0; k < 2000; ++k) {
                pool.join();
                char *p = pool.take();
                p[k % 16] = (char)k;
                pool.put(p);
                pool.leave();
            }
        });
    for (std::thread &t : threads) t.join();
    CHECK(Heap::live == 1);
    std::puts("OK");
    Heap::free(pool.take());
    return 0;
}
'''


def test_staging_pieces_are_kept_and_given_back(tmp_path):
    """One piece serves contexts that follow one another, four at most wait beside live contexts, and what a call
    holds while the last context goes comes back too."""
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_31258_amd", "csrc")
    src = tmp_path / "stage_test.cpp"
    src.write_text(STAGE)
    exe = tmp_path / "stage_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-fsanitize=thread", "-I" + csrc, str(src), "-o", str(exe)],
                   check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0 and run.stdout.strip() == "OK", run.stdout + run.stderr
