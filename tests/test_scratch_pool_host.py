"""The pool of kept set-up memory (csrc/scratch_pool.h), compiled for the host on memory that only counts: what it may hand out
and keep, and what it gives back when."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_06941_amd", "csrc")

CODE = r'''
#include "scratch_pool.h"
#include <atomic>
#include <vector>
static std::atomic<uint64_t> g_now{0}, g_most{1000};
static std::vector<uint64_t> g_freed;          // in the order they were freed
struct Mem {
    static void free(void* p) { g_freed.push_back((uint64_t)(uintptr_t)p); }
    static uint64_t now_ns() { return g_now; }
    static uint64_t keep_at_most(int) { return g_most; }
    static bool wait(int device);
};
static std::vector<int> g_waited;              // devices that were waited for, and what was free to be taken on them then
static bool g_wait_fails = false;
static ScratchPool<Mem>* pool = new ScratchPool<Mem>();
bool Mem::wait(int device)
{
    uint64_t room = 0;
    if (void* p = pool->take(device, 1, ~0ull, &room)) { pool->give(device, p, room); g_waited.push_back(-1); }
    g_waited.push_back(device);
    return !g_wait_fails;
}
struct Block { void* ptr; uint64_t room; bool kept; };
extern "C" {
// a task that held block 1 (kept), 2 (scratch) and 3 (no block of the pool) ends; how many blocks are still its own
int end_of_task(int device, int fails)
{
    std::vector<Block> blocks = {{(void*)1, 100, true}, {(void*)2, 100, false}, {(void*)3, 0, true}};
    g_waited.clear();
    g_wait_fails = fails != 0;
    pool->take_back(device, blocks);
    int own = 0;
    for (const Block& b : blocks) own += b.ptr != nullptr;
    return own;
}
// tasks of five blocks each, of sizes more than a quarter apart, one after the other `rounds` times: blocks that had to be allocated
int allocated_by(uint64_t tasks, uint64_t rounds, uint64_t most)
{
    g_most = most;
    ScratchPool<Mem, kKeptBlocks> lasting;     // as the library has it
    int fresh = 0;
    for (uint64_t k = 0; k < rounds * tasks; ++k) {
        const uint64_t size = 100ull << k % tasks;
        void* held[5];
        uint64_t room[5];
        for (int i = 0; i < 5; ++i) {
            room[i] = size;
            held[i] = lasting.take(0, size, size + size / 4, &room[i]);
            if (!held[i]) { held[i] = (void*)(uintptr_t)(1000 + 10 * k + i); ++fresh; }
        }
        for (int i = 0; i < 5; ++i) lasting.give(0, held[i], room[i]);
    }
    return fresh;
}
int waited(uint64_t k) { return k < g_waited.size() ? g_waited[k] : -2; }
void reset(uint64_t most) { delete pool; pool = new ScratchPool<Mem>(); g_now = 0; g_most = most; g_freed.clear(); }
void set_now(uint64_t s) { g_now = s * 1000000000ull; }
uint64_t take(int device, uint64_t bytes, uint64_t most) { uint64_t room = 0; return pool->take(device, bytes, most, &room) ? room : 0; }
void give(int device, uint64_t id, uint64_t room) { pool->give(device, (void*)(uintptr_t)id, room); }
uint64_t trim(int all) { return pool->trim(all != 0); }
int begins(int device) { return pool->begins(device); }
uint64_t freed(uint64_t k) { return k < g_freed.size() ? g_freed[k] : 0; }
uint64_t most(uint64_t limit, uint64_t total, uint64_t bytes) { return most_room(limit, total, bytes); }
}
'''


def _build(tmp_path_factory, name, code, *flags):
    d = tmp_path_factory.mktemp(name)
    src, out = d / (name + ".cpp"), d / name
    src.write_text(code)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread", "-I", CSRC, *flags, str(src), "-o", str(out)], check=True)
    return str(out)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    L = ctypes.CDLL(_build(tmp_path_factory, "pool.so", CODE, "-shared", "-fPIC"))
    u64 = ctypes.c_uint64
    for name, args in (("reset", [u64]), ("set_now", [u64]), ("take", [ctypes.c_int, u64, u64]), ("give", [ctypes.c_int, u64, u64]),
                       ("freed", [u64]), ("trim", [ctypes.c_int]), ("most", [u64, u64, u64])):
        getattr(L, name).argtypes = args
        getattr(L, name).restype = u64
    return L


def _freed(L):
    out = []
    while L.freed(len(out)):
        out.append(L.freed(len(out)))
    return out


def test_a_task_with_a_limit_gets_blocks_of_the_size_that_is_booked(lib):
    total = 1 << 38
    assert lib.most(1 << 40, total, 1000) == 1250                 # no limit of its own: up to a quarter more
    assert lib.most(total - 1, total, 1000) == 1000 and lib.most(1 << 40, 0, 1000) == 1000
    lib.reset(10_000)
    lib.give(0, 1, 1200)
    assert lib.take(0, 1000, lib.most(total - 1, total, 1000)) == 0
    assert lib.take(0, 1000, lib.most(total, total, 1000)) == 1200
    lib.give(0, 1, 1000)
    assert lib.take(0, 1000, lib.most(1, total, 1000)) == 1000


def test_blocks_are_bounded_in_number_and_bytes_and_age(lib):
    lib.reset(1000)
    lib.give(0, 1, 1001)                                          # more than may be kept at all
    assert _freed(lib) == [1]
    lib.give(0, 2, 600); lib.give(0, 3, 300); lib.give(1, 4, 1000)
    lib.give(0, 5, 200)                                           # 1100: the oldest of that device goes
    assert _freed(lib) == [1, 2]
    for k in range(6):
        lib.give(0, 10 + k, 10)                                   # eight blocks of device 0
    assert _freed(lib) == [1, 2]
    lib.give(0, 20, 10)
    assert _freed(lib) == [1, 2, 3]
    assert lib.take(0, 150, 199) == 0 and lib.take(2, 10, 10) == 0 and lib.take(0, 150, 200) == 200
    assert lib.take(1, 900, 1000) == 1000
    lib.set_now(6)
    lib.trim(0)
    assert sorted(_freed(lib)[3:]) == [10, 11, 12, 13, 14, 15, 20]
    lib.give(0, 30, 10)
    lib.trim(0)
    assert len(_freed(lib)) == 10
    lib.trim(1)
    assert _freed(lib)[-1] == 30


def test_only_a_set_up_that_follows_another_takes_part(lib):
    lib.reset(1000)
    lib.set_now(100)
    assert not lib.begins(0)                                      # the first of the process
    lib.set_now(105)
    assert lib.begins(0) and not lib.begins(1)                    # within five seconds, on the same device
    lib.set_now(111)
    assert not lib.begins(0) and not lib.begins(-1) and not lib.begins(64)
    lib.give(0, 1, 300); lib.give(1, 2, 400)
    assert lib.trim(0) == 0 and lib.trim(1) == 700 and lib.trim(1) == 0


def test_what_a_task_held_is_kept_only_when_its_own_device_is_done_with_it(lib):
    lib.reset(1000)
    lib.waited.argtypes, lib.end_of_task.argtypes = [ctypes.c_uint64], [ctypes.c_int, ctypes.c_int]
    assert lib.end_of_task(3, 0) == 2                             # (whichever device is current: only device 3 is asked about)
    assert [lib.waited(k) for k in range(2)] == [3, -2]           # once, with nothing of the task's to be had before
    assert lib.take(0, 1, 1000) == 0 and lib.take(3, 1, 1000) == 100 and lib.take(3, 1, 1000) == 0
    assert lib.end_of_task(3, 1) == 3                             # a device in error: all blocks stay the task's, which frees them
    assert lib.trim(1) == 0


def test_tasks_of_several_sizes_in_turn_find_their_blocks_again(lib):
    lib.reset(1000)
    lib.allocated_by.argtypes = [ctypes.c_uint64] * 3
    assert lib.allocated_by(2, 10, 1 << 20) == 2 * 5 and lib.allocated_by(4, 10, 1 << 20) == 4 * 5 and lib.allocated_by(12, 10, 1 << 22) == 12 * 5
    assert lib.allocated_by(4, 10, 5 * 1500 - 1) > 4 * 5          # (bytes bound it)


def test_memory_is_freed_outside_the_pools_lock(tmp_path_factory):
    # giving memory back waits for the device: a thread that only wants a block must not wait for that
    exe = _build(tmp_path_factory, "pool_lock", r'''
#include "scratch_pool.h"
#include <cstdio>
static uint64_t g_now = 0;
static void on_free();
struct Mem {
    static void free(void*) { on_free(); }
    static uint64_t now_ns() { return g_now; }
    static uint64_t keep_at_most(int) { return 100; }
};
static ScratchPool<Mem> pool;
static int frees = 0;
static void on_free() { ++frees; uint64_t room = 0; (void)pool.take(9, 1, 1, &room); }       // hangs if the lock is held
int main()
{
    pool.give(0, (void*)1, 101);                                 // too large
    for (uintptr_t k = 2; k < 12; ++k) pool.give(0, (void*)k, 10);        // too many
    pool.give(0, (void*)20, 90);                                 // too much
    g_now = ScratchPool<Mem>::kKeepNs + 1;
    pool.trim(false);                                            // too old
    pool.give(0, (void*)21, 1);
    pool.trim(true);
    std::printf("%d\n", frees);
    return 0;
}
''')
    out = subprocess.run([exe], capture_output=True, text=True, timeout=20, check=True).stdout
    assert int(out) == 1 + 10 + 1 + 1


def test_threads_never_share_a_block(tmp_path_factory):
    exe = _build(tmp_path_factory, "pool_threads", r'''
#include "scratch_pool.h"
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>
static std::atomic<int> owners[4096];
static std::atomic<int> live{0}, bad{0};
struct Mem {
    static void free(void* p) { if (owners[(uintptr_t)p].fetch_add(1) != 0) ++bad; --live; }       // (a freed block is never used again)
    static uint64_t now_ns() { return 0; }
    static uint64_t keep_at_most(int) { return 6; }
};
static ScratchPool<Mem> pool;
int main()
{
    std::atomic<uintptr_t> next{1};
    std::vector<std::thread> t;
    for (int k = 0; k < 8; ++k)
        t.emplace_back([&, k] {
            for (int i = 0; i < 400; ++i) {
                uint64_t room = 1;
                void* p = pool.take(k % 3, 1, 1, &room);
                if (!p) { p = (void*)next.fetch_add(1); ++live; }
                if (owners[(uintptr_t)p].fetch_add(1) != 0) ++bad;
                owners[(uintptr_t)p].fetch_sub(1);
                pool.give(k % 3, p, room);
                if (i % 97 == 0) pool.trim(true);
            }
        });
    for (auto& x : t) x.join();
    pool.trim(true);
    std::printf("%d %d\n", bad.load(), live.load());
    return 0;
}
''')
    assert subprocess.run([exe], capture_output=True, text=True, timeout=60, check=True).stdout.split() == ["0", "0"]
