"""Where the library's device memory comes from: the context's pool, which gives kept memory back before an allocation fails."""
import glob
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_09424_amd", "csrc")


def test_every_allocation_goes_through_the_pool():
    """hipMalloc is called in DevPool::alloc and nowhere else."""
    calls = []
    for path in sorted(glob.glob(os.path.join(CSRC, "**", "*.h*"), recursive=True)):
        where = None
        for line in open(path):
            m = re.match(r"\s*(?:inline )?hipError_t (?:DevPool::)?(\w+)\(", line)
            if m:
                where = m.group(1)
            if re.search(r"\bhipMalloc\(", line.split("//")[0]):
                calls.append((os.path.basename(path), where))
    assert calls and all(where == "alloc" for _, where in calls), calls


# DevPool on a simulated card: the runtime's calls it makes are defined here, so no GPU and no HIP library are needed.
CARD = r"""
#include <cstdio>
#include <cstdlib>
#include "devpool.h"
static bool host_full = false;
void *operator new(size_t bytes) {
    void *p = host_full ? nullptr : malloc(bytes);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
static size_t card_free = (size_t)4096 << 20, n_freed;
static hipError_t last = hipSuccess, sync_result = hipSuccess;
static std::map<void *, size_t> live;
extern "C" {
hipError_t hipMalloc(void **p, size_t bytes) {
    if (bytes > card_free) return last = hipErrorOutOfMemory;
    card_free -= bytes;
    live[*p = malloc(1)] = bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    card_free += live.at(p);
    live.erase(p);
    free(p);
    n_freed++;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return sync_result == hipSuccess ? hipSuccess : last = sync_result; }
hipError_t hipGetLastError() { hipError_t e = last; last = hipSuccess; return e; }
}
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
static const size_t MB = 1 << 20;
int main() {
    @BODY@
    return 0;
}
"""


def run_on_simulated_card(tmp_path, body):
    src, exe = tmp_path / "card.cpp", tmp_path / "card"
    src.write_text(CARD.replace("@BODY@", body))
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, str(src), "-o", str(exe), "-pthread"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_pool_gives_back_before_an_allocation_fails(tmp_path):
    run_on_simulated_card(tmp_path, """
        DevPool pool; void *a, *b, *c; size_t got;
        CHECK(pool.take(&a, 200 * MB, &got) == hipSuccess && got == 200 * MB);
        pool.give(a, got);
        CHECK(n_freed == 0 && pool.held == 200 * MB);
        CHECK(pool.take(&b, 190 * MB, &got) == hipSuccess && b == a && got == 200 * MB && pool.held == 0);  // the kept block serves it
        pool.give(b, got);
        CHECK(pool.take(&c, 4000 * MB, &got) == hipSuccess && n_freed == 1 && pool.held == 0);  // only fits once the kept block is back
        CHECK(last == hipSuccess);
    """)


def test_failed_allocation_leaves_no_error_behind(tmp_path):
    """The caller is told; the launch check of the next call must not find the same error again."""
    run_on_simulated_card(tmp_path, """
        DevPool pool; void *a; size_t got;
        CHECK(pool.take(&a, 5000 * MB, &got) == hipErrorOutOfMemory && a == nullptr);
        CHECK(hipGetLastError() == hipSuccess);
    """)


def test_pool_where_the_device_cannot_be_waited_for(tmp_path):
    """A kept block may still be in use, so it is not handed out then: it stays in the pool, and a new one serves the call."""
    run_on_simulated_card(tmp_path, """
        DevPool pool; void *a, *b; size_t got;
        CHECK(pool.take(&a, 200 * MB, &got) == hipSuccess);
        pool.give(a, got);
        sync_result = hipErrorStreamCaptureUnsupported;
        CHECK(pool.take(&b, 190 * MB, &got) == hipSuccess && b != a && got == 190 * MB && pool.held == 200 * MB);
        CHECK(hipGetLastError() == hipSuccess);
        sync_result = hipSuccess;
        CHECK(pool.take(&b, 200 * MB, &got) == hipSuccess && b == a && pool.held == 0);
    """)


def test_freeing_a_handle_does_not_throw(tmp_path):
    """Without host memory to note a block down, it goes back to the card."""
    run_on_simulated_card(tmp_path, """
        DevPool pool; void *a; size_t got;
        CHECK(pool.take(&a, 200 * MB, &got) == hipSuccess);
        host_full = true;
        pool.give(a, got);
        host_full = false;
        CHECK(n_freed == 1 && pool.held == 0 && card_free == 4096 * MB);
    """)
