"""The library's host code from inside, without a GPU: a driver includes
fk_host.cpp, is linked with the kernel objects of the last build, and runs one
check per process.  Contexts have no device (device -1); where a check needs a
HIP call, the driver's own stands in for the runtime's."""
import glob
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2407_21445_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

DRIVER = r'''
extern "C" {
int test_purify_steps(const double *, double *const *, int, int, int, int, const double *, double *, int *, void *);
int test_reduce(const double *, const double *, int, int, double *, double *, int, void *);
int test_lincomb(double *, const double *, const double *, const double *, int, double, double, double, double, void *);
}
#include <hip/hip_runtime.h>
#include "fk_internal.h"
#define fk_scf_purify_steps test_purify_steps
#define fk_scf_reduce test_reduce
#define fk_scf_lincomb test_lincomb
#include "fk_host.cpp"

#include <random>

#define CHECK(x)                                                          \
    do {                                                                  \
        if (!(x)) { std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x); return 1; } \
    } while (0)

// order_descending against a stable comparison sort
static int check_order()
{
    std::mt19937_64 rng(5);
    const uint64_t tops[] = {0, 1, 255, 256, 65535, 1 << 20, ~0ull};
    for (size_t n : {0, 1, 2, 3, 64, 1000, 4097})
        for (uint64_t top : tops)
            for (uint64_t base : {(uint64_t)0, (uint64_t)77 << 32}) {
                std::vector<uint64_t> key(n);
                for (auto &k : key) k = base + (top == ~0ull ? rng() : rng() % (top + 1));
                std::vector<int> got, want(n);
                order_descending(key, got);
                std::iota(want.begin(), want.end(), 0);
                std::stable_sort(want.begin(), want.end(), [&](int x, int y) { return key[x] > key[y]; });
                CHECK(got == want);
            }
    return 0;
}

// s, p and d shells on eight atoms, mixed contraction; two molecules
static int small_system(fk_ctx **ctx)
{
    CHECK(fk_create(ctx, -1) == FK_OK);
    const int na = 8;
    std::vector<int> Z(na, 6), atom, l, np;
    std::vector<double> xyz, ex, co;
    for (int a = 0; a < na; ++a) {
        xyz.insert(xyz.end(), {2.5 * (a % 4) + (a / 4) * 60.0, 0.3 * a, 0.7 * (a % 2)});
        for (int s = 0; s < 3; ++s) {
            atom.push_back(a); l.push_back(s); np.push_back(3 - s);
            for (int k = 0; k < 3 - s; ++k) { ex.push_back(8.0 / (1 + 3 * k + s)); co.push_back(0.3 + 0.2 * k); }
        }
    }
    CHECK(fk_set_geometry(*ctx, na, Z.data(), xyz.data(), 0) == FK_OK);
    CHECK(fk_set_basis(*ctx, (int)l.size(), atom.data(), l.data(), np.data(), ex.data(), co.data()) == FK_OK);
    const int mol[na] = {0, 0, 0, 0, 1, 1, 1, 1};
    CHECK(fk_set_molecules(*ctx, 2, mol) == FK_OK);
    CHECK(fk_build_quartets(*ctx, nullptr) == FK_OK);
    return 0;
}

// every kind of inconsistency is found
static int check_validation()
{
    fk_ctx *c = nullptr;
    if (small_system(&c)) return 1;
    CHECK(validate_lists(c) == FK_OK);
    const QuartetClass *task = nullptr;
    for (const auto &q : c->qclasses)
        if (q.ntask > 1 && !task) task = &q;
    CHECK(task);
    int bad = 0;
#define BREAK(lvalue, value)                                              \
    do {                                                                  \
        const auto keep = lvalue;                                         \
        lvalue = value;                                                   \
        if (validate_lists(c) == FK_OK) { std::printf("not found: %s = %s\n", #lvalue, #value); ++bad; } \
        lvalue = keep;                                                    \
    } while (0)
    for (size_t t : {(size_t)0, c->tiles.size() / 2, c->tiles.size() - 1}) {
        FkTile &T = c->tiles[t];
        const int gid = T.grp & ~FK_TILE_SAME;
        BREAK(T.blk, -1);
        BREAK(T.blk, (int)c->blocks.size());
        BREAK(T.grp, (int)c->groups.size());
        BREAK(T.grp, gid == 0 ? (int)c->groups.size() - 1 : 0);  // a group of another class, or of other kets
        BREAK(T.ket_count, 0);
        BREAK(T.ket_count, 65);
        BREAK(T.p0, T.p1);
        BREAK(T.p1, (unsigned char)(c->groups[gid].npp + 1));
        BREAK(T.ket_begin, c->groups[gid].begin - 1);
        BREAK(T.ket_begin, c->groups[gid].begin + c->groups[gid].len);
    }
    const size_t b = c->blocks.size() / 2;
    BREAK(c->blocks[b].first, -1);
    BREAK(c->blocks[b].count, FK_MAX_BRA_BLOCK + 1);
    BREAK(c->blk_bra[c->blocks[b].first], -1);
    BREAK(c->blk_pos[c->blocks[b].first], c->blk_pos[c->blocks[b].first] + 1);
    FkGroup &G = c->groups[c->groups.size() / 2];
    BREAK(G.npp, G.npp_min - 1);
    BREAK(G.base, (long long)c->ppT.size());
    BREAK(G.mol, 1 - G.mol);
    BREAK(c->lst_npp[G.begin], c->lst_npp[G.begin] + 1);
    BREAK(c->lst_sa[G.begin], c->lst_sa[G.begin] == 0 ? 1 : 0);
    const int p = c->ket_list_all[G.begin];
    BREAK(c->ket_list_all[G.begin], (int)c->pr_sa.size());
    BREAK(c->pr_npp[p], FK_MAX_K * FK_MAX_K + 1);
    BREAK(c->pr_sb[p], c->nshell);
    BREAK(c->pr_G[p], std::nan(""));
    BREAK(c->pr_ppoff[p], -1);
    QuartetClass &q = const_cast<QuartetClass &>(*task);
    BREAK(q.krow_ncol, 1);
    BREAK(q.krow_nbk, 0);
    BREAK(c->tasks[q.task_off].y, c->tasks[q.task_off].y + 1);
    BREAK(c->tasks[q.task_off + 1].x, 0);
    BREAK(c->krow_col[c->lst_sa[c->ket_off[q.Q]]], 1 << 20);
    CHECK(bad == 0);
    CHECK(validate_lists(c) == FK_OK);
    fk_destroy(c);
    return 0;
}

// The runtime's part in a launch: the LDS limit each kernel was last given, per
// device, and whether a launch kept to it.
static int g_dev = 0, g_refused = 0, g_launched = 0;
static std::map<std::pair<int, const void *>, int> g_limit;
extern "C" hipError_t hipGetDevice(int *d) { *d = g_dev; return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void *k, hipFuncAttribute, int v)
{
    g_limit[{g_dev, k}] = v;
    return hipSuccess;
}
extern "C" hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 1;
    return hipSuccess;
}
static size_t g_lds;
extern "C" hipError_t __hipPushCallConfiguration(dim3, dim3, size_t lds, hipStream_t)
{
    g_lds = lds;
    return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st)
{
    *grid = *block = dim3(1);
    *lds = g_lds;
    *st = nullptr;
    return hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void *k, dim3, dim3, void **, size_t lds, hipStream_t)
{
    ++g_launched;
    if (lds > 65536 && (int)lds > g_limit[{g_dev, k}]) ++g_refused;
    return hipSuccess;
}

// two contexts that use one kernel with rows of different lengths, on two devices
static int check_lds()
{
    const int P = pair_class(1, 1);
    auto probe = [&](int ncol) {
        int nb = 0;
        const int lds = fk_kernels_jk_lds_bytes(P, P, ncol, 1, 8, 4);
        if (lds <= 65536 || lds > 160 * 1024) std::printf("%d columns take %d bytes\n", ncol, lds);
        return fk_kernels_max_blocks(P, P, lds, 0, 1, 4, &nb) == 0 && nb == 1 && lds > 65536 && lds <= 160 * 1024;
    };
    auto launch = [&](int ncol) {
        FkJKArgs a;
        std::memset((void *)&a, 0, sizeof a);
        a.kind = 1; a.nw = 4; a.ntask = 1; a.krow_ncol = ncol; a.krow_nbk = 8;
        return fk_kernels_launch_jk(P, P, &a, 1, nullptr) == 0;
    };
    FkClassInfo info;
    CHECK(fk_kernels_class_info(P, P, &info) == 0 && info.wave_per_quartet == 1);
    for (g_dev = 0; g_dev < 2; ++g_dev) {
        CHECK(probe(440) && launch(440));
        CHECK(probe(300) && launch(300));
        CHECK(launch(440));
        CHECK(probe(480) && launch(440) && launch(480));
    }
    std::printf("%d launches, %d beyond their limit\n", g_launched, g_refused);
    CHECK(g_launched == 10 && g_refused == 0);
    return 0;
}

// Purification buffers: the second allocation fails once; the next purification
// must not run without it.
static int g_mallocs = 0, g_fail_at = 0, g_null_trace = 0, g_purified = 0;
extern "C" hipError_t hipMalloc(void **p, size_t n)
{
    *p = nullptr;
    if (++g_mallocs == g_fail_at) return hipErrorOutOfMemory;
    *p = std::calloc(1, n);
    return hipSuccess;
}
extern "C" hipError_t hipFree(void *p)
{
    std::free(p);
    return hipSuccess;
}
extern "C" hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
extern "C" hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
// stands in for the step kernels: done at once, one step
int test_purify_steps(const double *, double *const *, int, int, int, int last, const double *, double *trace, int *state,
                      void *)
{
    ++g_purified;
    if (!trace || !state) ++g_null_trace;
    if (state) { state[3 * (last - 1) + 1] = 1; state[3 * (last - 1) + 2] = 0; }
    return 0;
}
int test_reduce(const double *, const double *, int, int, double *, double *, int, void *) { return 0; }
int test_lincomb(double *, const double *, const double *, const double *, int, double, double, double, double, void *)
{
    return 0;
}

static int check_purify()
{
    for (int fail_at = 1; fail_at <= 2; ++fail_at) {
        fk_ctx c;
        ScfWork w;
        w.c = &c;
        w.n = 4;
        g_mallocs = 0;
        g_fail_at = fail_at;
        g_purified = 0;
        CHECK(scf_purify(w, 1, nullptr) == FK_ERR_OOM && g_purified == 0);
        g_fail_at = 0;
        CHECK(scf_purify(w, 1, nullptr) == FK_OK && g_purified == 1 && g_null_trace == 0);
    }
    return 0;
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    const int rc = what == "order" ? check_order() : what == "validation" ? check_validation() :
                   what == "lds" ? check_lds() : what == "purify" ? check_purify() : 2;
    std::printf("%s %s\n", what.c_str(), rc == 0 ? "passed" : "failed");
    return rc;
}
'''


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    objs = [o for o in sorted(glob.glob(os.path.join(PKG, "_build", "*.o"))) if os.path.basename(o) != "fk_host.o"]
    if not os.path.exists(HIPCC) or len(objs) < 14:
        pytest.skip("needs hipcc and the kernel objects of a build")
    d = tmp_path_factory.mktemp("driver")
    src, obj, exe = (str(d / x) for x in ("driver.cpp", "driver.o", "driver"))
    with open(src, "w") as f:
        f.write(DRIVER)
    for cmd in ([HIPCC, "-x", "hip", "-O1", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
                 "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-DFK_BUILD_MAXL=3", "-Wno-unused-function", "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG, "csrc"),
                 "-c", src, "-o", obj],
                [HIPCC, "--offload-arch=gfx950", "-o", exe, obj] + objs +
                ["-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib", "-lrocsolver", "-lrocblas"]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("what", ["order", "validation", "lds", "purify"])
def test_host_code(driver, what):
    """order: the radix order of tiles and chunks equals a stable sort by
    descending key.  validation: each inconsistency planted in the lists (tiles,
    blocks, groups, list positions, pairs, block tasks and their columns) is
    found before anything is uploaded.  lds: a context that asks for less dynamic
    LDS of a kernel does not take it from one that launches with more.  purify:
    after a failed allocation the next purification allocates what is missing."""
    r = subprocess.run([driver, what], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and f"{what} passed" in r.stdout, (r.stdout + r.stderr)[-4000:]
