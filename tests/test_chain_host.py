"""The backward's chains (a wavefront's, a workgroup's, and the one with 64-bit
addresses) on the CPU, with the kernels' own text: the sums bit for bit as the
sequential definition at the lengths where their code changes, every id read
inside its segment, every row load inside the buffer or, where the loads are
range-checked, past it at an offset that is still positive, and no row load
that is not range-checked outside it. Rows lie up to the end of the largest
window (2 GiB less a page), addressed from the start of the array and from the
segment's first row."""
import pytest

from tests import host_kernel as hk

SHIM = r"""
#include <sys/mman.h>
#include <bit>
#include <cstring>
#include <type_traits>
constexpr int kWave = 64, kBlock = 256;
static std::unique_ptr<std::barrier<>> wave_barrier[4];
static int32_t exchange[4][kWave];
static int32_t emu_readlane(int32_t v, int k) {
    const int w = threadIdx.x / kWave;
    exchange[w][threadIdx.x % kWave] = v;
    wave_barrier[w]->arrive_and_wait();
    const int32_t r = exchange[w][k];
    wave_barrier[w]->arrive_and_wait();
    return r;
}
static inline void lds_barrier() { __syncthreads(); }
struct Buffer { const char *p; int64_t size; bool checked; };
using __amdgpu_buffer_rsrc_t = Buffer;
static bool range_checked;  // whether the chain under test relies on it
[[noreturn]] static void bad(const char *what, int64_t i) {
    std::printf("%s %lld\n", what, (long long)i);
    std::fflush(stdout);
    std::_Exit(3);
}
static Buffer make_rsrc(const float *p, int, int32_t size, int) {
    return {reinterpret_cast<const char *>(p), size, range_checked};
}
static int32_t load_b32(const Buffer &b, int32_t voff, int32_t soff, int) {
    const int64_t at = int64_t(voff) + soff;
    if (voff < 0 || soff < 0) bad("negative offset", at);
    if (at + 4 > b.size) {
        // only the vector offset is checked by the hardware
        if (!b.checked || soff != 0) bad("row load past the buffer at", at);
        return 0;
    }
    int32_t v;
    std::memcpy(&v, b.p + at, 4);
    return v;
}
#define __builtin_amdgcn_readlane emu_readlane
#define __builtin_amdgcn_readfirstlane(v) (v)
#define __builtin_amdgcn_make_buffer_rsrc make_rsrc
#define __builtin_amdgcn_raw_buffer_load_b32 load_b32
#define __builtin_amdgcn_sched_barrier(x) (void)0
template <int K> using Int = std::integral_constant<int, K>;
struct Ids {  // of one segment, at `beg` of the array
    const int32_t *p;
    int64_t len;
    int32_t operator[](int64_t i) const {
        if (i < 0 || i >= len) bad("read of id", i);
        return p[i];
    }
};
"""

MAIN = r"""
// kind 0: a wavefront, 1: a workgroup, 2: 64-bit addresses
int main(int argc, char **argv) {
    const int kind = atoi(argv[1]), dim = atoi(argv[2]), whole = atoi(argv[3]);
    const int64_t rows = int64_t(kOutOfRange) / (dim * 4);  // the most that a window holds
    const int64_t first = whole ? 0 : 7;  // grad from its first row, or a window that starts later
    const int64_t floats = (rows + first) * dim;
    float *grad = static_cast<float *>(mmap(nullptr, floats * 4, PROT_READ | PROT_WRITE,
                                            MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
    if (grad == MAP_FAILED) return 9;
    range_checked = kind == 1;
    const int threads = kind == 1 ? 256 : 64;
    for (int w = 0; w < 4; ++w) wave_barrier[w] = std::make_unique<std::barrier<>>(kWave);
    for (int a = 4; a < argc; ++a) {
        const int32_t len = atoi(argv[a]);
        std::vector<int32_t> ids(len);
        uint32_t s = 99u + uint32_t(len);
        auto next = [&] { return s = s * 1664525u + 1013904223u, s >> 8; };
        for (int32_t k = 0; k < len; ++k)
            ids[k] = int32_t(first + (k < 2 ? 0 : k > len - 3 ? rows - 1 : int64_t(k) * (rows - 1) / len));
        for (int32_t k = 0; k < len; ++k)
            for (int c = 0; c < dim; ++c)
                grad[int64_t(ids[k]) * dim + c] = float(int(next() % 20011) - 10005) * 0.37f;
        const int parts = (dim + kPartCols - 1) / kPartCols;
        for (int part : {0, parts - 1}) {
            static float sum[kBlock], hand[kWave];
            run_grid(1, threads, [&] {
                const int w = threadIdx.x / kWave, col = part * kPartCols + int(threadIdx.x % kWave);
                const Ids sid{ids.data(), len};
                const int32_t bytes = whole ? int32_t(rows * dim * 4) : 0;
                sum[threadIdx.x] =
                    kind == 0   ? wave_chain(grad, dim, sid, 0, len, part, bytes, [] {})
                    : kind == 1 ? block_chain(hand, grad, dim, sid, 0, len, w, part, bytes)
                                : far_chain(grad, dim, sid, len, col);
            });
            for (int lane = 0; lane < kWave && part * kPartCols + lane < dim; ++lane) {
                float acc = 0.f;
                for (int32_t k = 0; k < len; ++k)
                    acc = acc + grad[int64_t(ids[k]) * dim + part * kPartCols + lane];
                const float got = sum[(kind == 1 ? kBlock - kWave : 0) + lane];
                if (std::memcmp(&got, &acc, 4)) bad("sum of column", part * kPartCols + lane);
            }
        }
        std::printf("%d rows\n", len);
    }
    munmap(grad, floats * 4);
    return 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    src = hk.source("tc_backward.hip")
    parts = [SHIM, "constexpr int kPartCols = 64;\n"]
    parts += [hk.const(src, c) for c in ("kBufferWord3", "kOutOfRange", "kFarRows", "kDepth",
                                         "kGroupRows", "kWgWaves")]
    for head in ("__device__ __forceinline__ float far_chain(",
                 "template <class Last>\n__device__ __forceinline__ float wave_chain(",
                 "__device__ __forceinline__ float block_chain("):
        fn = hk.block(src, head)
        fn = fn.replace("const int32_t *__restrict__ ids", "Ids ids")
        fn = fn.replace("const int32_t *__restrict__ sid", "Ids sid")
        fn = fn.replace("const int32_t *sid = ids + beg;", "const Ids sid = ids;")
        fn = fn.replace("const_cast<float *>(", "(")
        fn = fn.replace('asm volatile("" : "+v"(next_id));', "")
        assert "asm" not in fn and "int32_t *" not in fn
        parts.append(fn)
    return hk.program(tmp_path_factory.mktemp("chain"), parts, MAIN)


@pytest.mark.parametrize("kind,dim,whole,lens", [
    (0, 100, 1, [48, 80, 81, 121]), (0, 100, 0, [49, 79, 120, 511]), (0, 1024, 0, [119]),
    (0, 4, 1, [160]), (1, 100, 1, [512, 640]), (1, 100, 0, [513, 641]), (1, 1024, 1, [639]),
    (2, 100, 0, [48, 63, 64, 65]), (2, 1024, 0, [96])])
def test_chains(exe, kind, dim, whole, lens):
    hk.run(exe, kind, dim, whole, *lens)


def test_lengths_beyond_the_buffer_path():
    src = hk.source("tc_backward.hip")
    # an id's byte offset and the rounds' positions fit 32 bits below the
    # length from which the 64-bit addresses are taken
    assert src.count("span > uint64_t(kOutOfRange) || len >= (1 << 28)") == 3
    ahead = 3 * 4 * 40 + 63  # positions past the end that are named
    assert ((1 << 28) + ahead) * 4 < 2 ** 31
