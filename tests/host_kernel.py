"""Runs pieces of the kernel sources on the CPU: constants, structs and whole
functions are taken out of a source by name, set into a small C++ program
between the few names that HIP gives them (thread and block indexes, LDS,
atomics, the workgroup barrier) and built with g++. A workgroup's threads are
threads of the program. Global arrays that a test wants watched are passed as
`Checked`, which ends the program at the first read outside them."""
from __future__ import annotations

import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2010_13100_amd", "csrc")

SHIM = r"""
#include <algorithm>
#include <barrier>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <thread>
#include <vector>
using std::min;
using std::max;
#define __device__
#define __global__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
struct dim3_ { int32_t x; };
static thread_local dim3_ threadIdx, blockIdx;
static dim3_ gridDim;
struct alignas(8) int2 { int32_t x, y; };
struct alignas(16) int4 { int32_t x, y, z, w; };
static inline int2 make_int2(int32_t x, int32_t y) { return {x, y}; }
static inline int4 make_int4(int32_t x, int32_t y, int32_t z, int32_t w) { return {x, y, z, w}; }
static inline int32_t atomicAdd(int32_t *p, int32_t v) {
    return __atomic_fetch_add(p, v, __ATOMIC_RELAXED);
}
static std::unique_ptr<std::barrier<>> group_barrier;
static inline void __syncthreads() { group_barrier->arrive_and_wait(); }
static inline int64_t min(int64_t a, int b) { return a < b ? a : b; }
struct Checked {
    const int32_t *p;
    int64_t n;
    int32_t operator[](int64_t i) const {
        if (i < 0 || i >= n) {
            std::printf("read of entry %lld of %lld\n", (long long)i, (long long)n);
            std::fflush(stdout);
            std::_Exit(3);
        }
        return p[i];
    }
};
// fn() as every thread of one workgroup after another
template <class F>
static void run_grid(int blocks, int threads, F fn) {
    gridDim.x = blocks;
    group_barrier = std::make_unique<std::barrier<>>(threads);
    std::vector<std::thread> ts;
    for (int t = 0; t < threads; ++t)
        ts.emplace_back([=] {
            for (int b = 0; b < blocks; ++b) {
                blockIdx.x = b, threadIdx.x = t;
                fn();
                __syncthreads();
            }
        });
    for (auto &t : ts) t.join();
}
"""


def source(name: str) -> str:
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def const(src: str, name: str) -> str:
    m = re.search(r"^constexpr [^=;]*\b" + name + r" = [^;]+;", src, re.M)
    assert m, name
    return m.group(0) + "\n"


def block(src: str, start: str) -> str:
    """The text from `start` (a struct or function head) to its closing brace,
    with a struct's semicolon."""
    at = src.index(start)
    depth, i = 0, src.index("{", at)
    while True:
        depth += {"{": 1, "}": -1}.get(src[i], 0)
        i += 1
        if depth == 0:
            break
    return src[at:i] + (";\n" if src[i] == ";" else "\n")


def program(tmp_path, parts, main: str) -> str:
    """Builds the program and returns its path."""
    cpp, exe = os.path.join(tmp_path, "k.cpp"), os.path.join(tmp_path, "k")
    with open(cpp, "w") as f:
        f.write(SHIM + "\n".join(parts) + main)
    subprocess.run(["g++", "-std=c++20", "-O1", "-pthread", "-w", "-fwrapv", cpp, "-o", exe],
                   check=True)
    return exe


def run(exe: str, *args) -> str:
    r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, (args, r.returncode, r.stdout[-200:])
    return r.stdout
