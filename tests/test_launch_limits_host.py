"""Launch grids of the largest batches, without a device: a launch takes fewer
than 2^32 threads along x.  A small program that defines the runtime's launch
calls itself (so that the library's go there) records the grids that the
launchers ask for; nothing runs, and no pointer is followed.

* copies of states: 64 GiB and more go in pieces that cover every byte once;
* adjoint passes: 65535 chains of 32768 nodes;
* graph terms: 2^24 + 8 graphs of two nodes;
* steps held on chip: a long run in launches of bounded length;
* which calls run on chip: not those of batches whose realisations are mostly much
  smaller than the largest, nor short calls on states beyond the caches."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1612_00746_amd")

PROGRAM = r"""
#include "ctqw_internal.hpp"
#include "adjoint_pipe.hpp"
#include "graph.hpp"
#include "resident.hpp"
#include "ctqw.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

namespace { dim3 g_grid, g_block; size_t g_lds; hipStream_t g_stream; bool g_copy; const void* g_only; }

extern "C" {
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    g_grid = grid; g_block = block; g_lds = lds; g_stream = stream;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
    *grid = g_grid; *block = g_block; *lds = g_lds; *stream = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
    if (g_only) {   // on-chip steps: steps, and where they start and end
        const auto* a = (const ctqw::ResidentArgs*)args[0];
        if (fn == g_only)
            std::printf("launch %lld %llu %llu %lld\n", (long long)a->steps, (unsigned long long)a->psi_in,
                        (unsigned long long)a->psi_out, (long long)a->out_stride);
        return hipSuccess;
    }
    std::printf("launch %u %u %u %u", grid.x, grid.y, grid.z, block.x);
    if (g_copy)   // source, destination, 16-byte elements, words after them
        std::printf(" %llu %llu %lld %d", (unsigned long long)*(void**)args[0], (unsigned long long)*(void**)args[1],
                    (long long)*(int64_t*)args[2], *(int*)args[3]);
    std::printf("\n");
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) { *a = {}; a->maxThreadsPerBlock = 256; return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void*, size_t n, hipMemcpyKind kind, hipStream_t) {
    if (kind == hipMemcpyDeviceToHost) std::memset(dst, 0, n);
    return hipSuccess;
}
}

int main(int argc, char** argv) {
    using namespace ctqw;
    hipError_t e = hipErrorInvalidValue;
    if (!std::strcmp(argv[1], "copy")) {
        g_copy = true;
        e = launch_copy((void*)(1ull << 40), (const void*)(1ull << 44), std::atoll(argv[2]), nullptr);
    } else if (!std::strcmp(argv[1], "adjoint")) {
        AdjPipeArgs a{};
        double x = 0;
        a.x = &x;
        a.sign = 1;
        a.y[0] = &x;
        a.R = std::atoll(argv[2]);
        a.max_n = std::atoi(argv[3]);
        a.nb = (a.max_n + pipe_band_width(1) - 1) / pipe_band_width(1);
        a.levels = 1;
        e = launch_adj_pipe(a, nullptr);
        std::printf("bands %d\n", a.nb);
    } else if (!std::strcmp(argv[1], "graph")) {
        GraphTermArgs a{};
        a.n = std::atoi(argv[2]);
        a.R = std::atoi(argv[3]);
        a.width = 1;
        e = launch_graph_term(a, 1, nullptr);
    }
    else if (!std::strcmp(argv[1], "steps")) {
        const int N = 20, R = 3;
        ResidentShape s;
        if (!resident_shape(kResTri, 1, 0, N, 6, R, &s)) return 1;
        g_only = (const void*)resident_tri(s).kernel;
        ctqw_problem pr{};
        pr.m = 2;
        pr.statistics = CTQW_BOSON;
        pr.dtype = CTQW_C128;
        pr.R = R;
        pr.n_sites = N;
        pr.dt = 0.05;
        pr.taylor_order = 6;
        ctqw_plan* p = nullptr;
        std::vector<double> J(R * (N - 1), 1.0), eps(R * N, 0.0), U(R, 0.0), w(N, 1.0), g(2 * N);
        double loss;
        char* const base = (char*)(1ull << 40);
        int32_t sites[2] = {1, 2};
        int64_t state, work, grad;
        const int64_t n = std::atoll(argv[2]), every = std::atoll(argv[3]);
        int st = ctqw_plan_create(&pr, &p);
        if (!st) st = ctqw_set_params(p, J.data(), eps.data(), U.data());
        if (!st) st = ctqw_sizes(p, &state, &work);
        if (!st) st = ctqw_bind(p, base, base + (1 << 28), state, base + (1 << 29), work, nullptr);
        if (!st) st = ctqw_init_product_state(p, sites, 0);
        if (!st && !every) st = ctqw_propagate(p, n, 0, 0, nullptr);
        if (!st && every) st = ctqw_gradient_workspace(p, n, every, &grad);
        if (!st && every)
            st = ctqw_gradient(p, n, every, CTQW_LOSS_PRODUCT, w.data(), base + (1ull << 32), grad, &loss, g.data(),
                               g.data() + N);
        e = (hipError_t)st;
        std::printf("state %lld\n", (long long)state);
        ctqw_plan_destroy(p);
    } else if (!std::strcmp(argv[1], "route")) {
        // statistics, boundary, dtype, largest lattice, how many, the others' size, how many, order, steps
        const int N = std::atoi(argv[5]), n1 = std::atoi(argv[6]), small = std::atoi(argv[7]), n2 = std::atoi(argv[8]);
        ctqw_problem pr{};
        pr.m = 2;
        pr.statistics = std::atoi(argv[2]);
        pr.boundary = std::atoi(argv[3]);
        pr.dtype = std::atoi(argv[4]);
        pr.R = n1 + n2;
        std::vector<int32_t> Ns(n1, N);
        Ns.resize(pr.R, small);
        pr.n_sites_per_real = Ns.data();
        pr.dt = 0.05;
        pr.taylor_order = std::atoi(argv[9]);
        int64_t sites = 0, state, work;
        for (int x : Ns) sites += x;
        std::vector<double> J(sites, 1.0), eps(sites, 0.0), U(pr.R, 0.0);
        ctqw_plan* p = nullptr;
        char* const base = (char*)(1ull << 40);
        int32_t at[2] = {1, 2};
        const int layout = pr.statistics ? kResTri : (pr.boundary ? kResRing : kResFull);
        ResidentShape s;
        if (!resident_shape(layout, pr.dtype, pr.dtype ? 0 : 1, N, pr.taylor_order, pr.R, &s)) return 1;
        g_only = (const void*)(layout == kResTri ? resident_tri(s) : layout == kResRing ? resident_ring(s)
                                                                                         : resident_full(s)).kernel;
        int st = ctqw_plan_create(&pr, &p);
        if (!st) st = ctqw_set_params(p, J.data(), eps.data(), U.data());
        if (!st) st = ctqw_sizes(p, &state, &work);
        if (!st) st = ctqw_bind(p, base, base + (1ull << 36), state, base + (1ull << 37), work, nullptr);
        if (!st) st = ctqw_init_product_state(p, at, 0);
        if (!st) st = ctqw_propagate(p, std::atoll(argv[10]), 0, 0, nullptr);
        e = (hipError_t)st;
        ctqw_plan_destroy(p);
    }
    std::printf("status %d\n", (int)e);
    return 0;
}
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    cc = next((c for c in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc")
               if c and os.path.exists(c)), None)
    if cc is None or not os.path.exists(os.path.join(PKG, "libctqw.so")):
        pytest.skip("needs hipcc and the built library")
    d = tmp_path_factory.mktemp("launches")
    src, exe = str(d / "launches.hip"), str(d / "launches")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run([cc, "--offload-host-only", "-std=c++17", "-w", "-I" + os.path.join(PKG, "csrc"),
                    "-I" + os.path.join(ROOT, "include"), src, "-o", exe, "-rdynamic", "-L" + PKG, "-l:libctqw.so",
                    "-Wl,-rpath," + PKG], check=True)

    def run(*args):
        out = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True, timeout=60).stdout
        lines = [l.split() for l in out.splitlines()]
        grids = [tuple(map(int, l[1:])) for l in lines if l[0] == "launch"]
        rest = {l[0]: int(l[1]) for l in lines if l[0] != "launch"}
        return grids, rest
    return run


def assert_launchable(g):
    assert g[0] * g[3] < 2 ** 32 and 1 <= g[1] <= 65535 and 1 <= g[2] <= 65535, g


@pytest.mark.parametrize("size", [4, 12, 16, 4096, 2 ** 34 - 8, 2 ** 34, 2 ** 34 + 24, 2 ** 36 - 16, 2 ** 36, 2 ** 37 + 8])
def test_copies_are_launchable_and_cover_every_byte(recorder, size):
    grids, rest = recorder("copy", size)
    assert rest["status"] == 0 and grids
    at = 0
    for k, g in enumerate(grids):
        assert_launchable(g)
        dst_src, elements, words = (g[5], g[4]), g[6], g[7]
        assert dst_src == (2 ** 40 + at, 2 ** 44 + at)
        assert g[0] * g[3] > elements      # a thread for each, and one for the words after them
        assert words == 0 or k == len(grids) - 1
        at += 16 * elements + 4 * words
    assert at == size


def test_adjoint_passes_of_the_largest_batches(recorder):
    for R, n in ((65535, 32768), (65535, 15000), (9, 100)):
        grids, rest = recorder("adjoint", R, n)
        assert rest["status"] == 0 and len(grids) == 1
        assert_launchable(grids[0])
        # whole groups of eight realisations, every band of each
        assert grids[0][0] * grids[0][1] == (R + 7) // 8 * 8 * rest["bands"]
        assert grids[0][3] == 64   # one particle's row is one wave's work


def test_graph_terms_of_many_small_graphs(recorder):
    for n, R in ((2, 2 ** 24 + 8), (300, 2 ** 23), (2, 64)):
        grids, rest = recorder("graph", n, R)
        assert rest["status"] == 0 and len(grids) == 1
        assert_launchable(grids[0])


@pytest.mark.parametrize("n", [1, 256, 257, 100000])
def test_long_runs_on_chip_are_cut(recorder, n):
    """propagate: every launch at most 256 steps, in place."""
    grids, rest = recorder("steps", n, 0)
    assert rest["status"] == 0
    assert sum(g[0] for g in grids) == n and all(1 <= g[0] <= 256 for g in grids)
    assert all(g[1] == g[2] and g[3] == 0 for g in grids)


@pytest.mark.parametrize("n,every", [(700, 700), (40, 40), (1024, 512)])
def test_recomputed_segments_on_chip_are_cut(recorder, n, every):
    """gradient: a segment's states are stored one after the other, a launch
    starting from the state that the one before it stored last."""
    grids, rest = recorder("steps", n, every)
    assert rest["status"] == 0 and all(1 <= g[0] <= 256 for g in grids)
    stored = [g for g in grids if g[3]]
    assert sum(g[0] for g in grids if not g[3]) == n and sum(g[0] for g in stored) == n // every * (every - 1)
    at = 0
    for a, b in zip(stored, stored[1:]):
        at += a[0]
        if at % (every - 1):   # inside a segment
            assert b[2] == a[2] + a[0] * a[3] and b[1] == b[2] - b[3]


GRID, BOSON = 0, 1
OPEN, RING = 0, 1
C64, C128 = 0, 1


@pytest.mark.parametrize("batch,steps,on_chip", [
    # one large lattice among small ones
    ((GRID, OPEN, C64, 128, 1, 16, 4095, 7), 20, False),
    ((GRID, OPEN, C128, 96, 1, 16, 4095, 10), 20, False),
    ((BOSON, OPEN, C64, 128, 1, 16, 4095, 7), 20, False),
    ((GRID, OPEN, C128, 96, 1, 32, 1000, 10), 20, False),
    ((GRID, OPEN, C64, 128, 1, 16, 255, 7), 20, True),
    ((BOSON, OPEN, C128, 128, 500, 60, 500, 10), 20, True),
    # large states: short calls, and lattices that leave waves idle
    ((GRID, OPEN, C64, 96, 8000, 0, 0, 7), 1, False),
    ((GRID, OPEN, C64, 80, 8000, 0, 0, 7), 16, False),
    ((GRID, OPEN, C64, 64, 16000, 0, 0, 7), 1, False),
    ((GRID, OPEN, C64, 64, 16000, 0, 0, 7), 16, True),
    ((GRID, RING, C64, 48, 16000, 0, 0, 7), 16, False),
    ((BOSON, OPEN, C64, 128, 16000, 0, 0, 7), 1, False),
    ((BOSON, OPEN, C64, 128, 16000, 0, 0, 7), 16, True),
    # few realisations of the widest shapes
    ((GRID, OPEN, C64, 128, 1, 0, 0, 7), 4, True),
    ((GRID, OPEN, C64, 128, 1, 0, 0, 7), 1, False),
    ((GRID, RING, C128, 96, 1, 0, 0, 10), 30, False),
    # what the on-chip steps are for
    ((BOSON, OPEN, C128, 128, 1000, 0, 0, 12), 1, True),
    ((GRID, OPEN, C128, 16, 8, 0, 0, 9), 1, True),
    ((GRID, OPEN, C64, 64, 1000, 0, 0, 7), 4, True),
])
def test_calls_go_on_chip_where_that_is_faster(recorder, batch, steps, on_chip):
    grids, rest = recorder("route", *batch, steps)
    assert rest["status"] == 0 and sum(g[0] for g in grids) == (steps if on_chip else 0)
