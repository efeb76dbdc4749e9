"""The library's device memory pool (mgrw_pool.h), compiled here for the CPU
against a stand-in for the few HIP calls it makes, with two devices and a
memory of bounded size; and on the GPU, that the memory comes back."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2312_07440_amd", "csrc")

STAND_IN = r"""
#pragma once
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <map>
#include <vector>
typedef int hipError_t;
typedef int hipDevice_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2 };
struct fake_stream { int dev; };
typedef fake_stream* hipStream_t;
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
enum { hipMemAllocationTypePinned = 1, hipMemHandleTypeNone = 0, hipMemLocationTypeDevice = 1,
       hipMemPoolAttrReleaseThreshold = 4 };
struct hipMemPoolProps { int allocType, handleTypes; struct { int type, id; } location; };
// held: bytes freed by the program but kept by the pool; pending: freed, the work before it not yet done
struct fake_pool { int dev; uint64_t keep; size_t held, pending; };
typedef fake_pool* hipMemPool_t;
struct fake_block { fake_pool* pool; size_t bytes; };
static int cur_dev = 0;
static size_t room = 1000;                       // bytes of each device
static size_t used[2] = {};                      // bytes out of the system's hands
static std::vector<fake_pool*> all_pools;
static fake_pool default_pool[2] = {{0, 0, 0, 0}, {1, 0, 0, 0}};
static std::map<void*, fake_block> blocks;
inline hipError_t hipGetDevice(int* d) { *d = cur_dev; return hipSuccess; }
inline hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { *d = s->dev; return hipSuccess; }
inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
    *c = hipStreamCaptureStatusNone;
    return hipSuccess;
}
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipMemPoolCreate(hipMemPool_t* p, const hipMemPoolProps* q) {
    all_pools.push_back(*p = new fake_pool{q->location.id, 0, 0, 0});
    return hipSuccess;
}
inline hipError_t hipMemPoolSetAttribute(hipMemPool_t p, int, void* v) {
    p->keep = *static_cast<uint64_t*>(v);
    return hipSuccess;
}
inline hipError_t hipMemPoolTrimTo(hipMemPool_t p, size_t keep) {
    if (p->held > keep) { used[p->dev] -= p->held - keep; p->held = keep; }
    return hipSuccess;
}
inline hipError_t hipMallocFromPoolAsync(void** ptr, size_t bytes, hipMemPool_t p, hipStream_t) {
    const size_t reuse = bytes <= p->held ? bytes : 0;   // a larger one is a new block
    if (used[p->dev] - reuse + bytes > room) return hipErrorOutOfMemory;
    used[p->dev] += bytes - reuse;
    p->held -= reuse;
    *ptr = std::malloc(1);
    blocks[*ptr] = {p, bytes};
    return hipSuccess;
}
inline hipError_t hipMallocAsync(void** ptr, size_t bytes, hipStream_t s) {
    return hipMallocFromPoolAsync(ptr, bytes, &default_pool[s ? s->dev : cur_dev], s);
}
inline hipError_t hipFreeAsync(void* ptr, hipStream_t) {
    blocks[ptr].pool->pending += blocks[ptr].bytes;
    return hipSuccess;
}
// a synchronisation: pending frees complete, what exceeds the threshold goes back
inline void synchronize() {
    std::vector<fake_pool*> ps = all_pools;
    ps.push_back(&default_pool[0]);
    ps.push_back(&default_pool[1]);
    for (fake_pool* p : ps) {
        p->held += p->pending;
        p->pending = 0;
        hipMemPoolTrimTo(p, p->keep);
    }
}
"""

PROGRAM = r"""
#include <cstdio>
#include "mgrw_pool.h"
using namespace mgrw;
#define NEED(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
    fake_stream s0{0}, s1{1};
    void* a = nullptr;
    CASE
    return 0;
}
"""

CASES = {
    # kept over a synchronisation while a handle is there
    "kept": """
    pools().handle_created();
    NEED(work_alloc(&a, 600, &s0) == hipSuccess && hipFreeAsync(a, &s0) == hipSuccess);
    synchronize();
    NEED(used[0] == 600);
    pools().handle_destroyed();
    NEED(used[0] == 0);
    """,
    # the last handle goes while its work is still queued
    "closed before the work is done": """
    pools().handle_created();
    NEED(work_alloc(&a, 600, &s0) == hipSuccess && hipFreeAsync(a, &s0) == hipSuccess);
    pools().handle_destroyed();
    synchronize();
    NEED(used[0] == 0);
    pools().handle_created();
    NEED(work_alloc(&a, 500, &s0) == hipSuccess && hipFreeAsync(a, &s0) == hipSuccess);
    synchronize();
    NEED(used[0] == 500);
    """,
    # what the pool keeps is in the way of a larger buffer
    "kept memory makes room": """
    pools().handle_created();
    NEED(work_alloc(&a, 600, &s0) == hipSuccess && hipFreeAsync(a, &s0) == hipSuccess);
    synchronize();
    NEED(work_alloc(&a, 700, &s0) == hipSuccess && used[0] == 700);
    """,
    # a stream of another device than the current one
    "device of the stream": """
    pools().handle_created();
    NEED(work_alloc(&a, 600, &s1) == hipSuccess);
    NEED(used[0] == 0 && used[1] == 600);
    void* b = nullptr;
    NEED(work_alloc(&b, 500, nullptr) == hipSuccess);
    NEED(used[0] == 500 && used[1] == 600);
    """,
}


def run_case(case, tmp_path):
    os.makedirs(tmp_path / "hip", exist_ok=True)
    (tmp_path / "hip" / "hip_runtime.h").write_text(STAND_IN)
    (tmp_path / "t.cpp").write_text(PROGRAM.replace("CASE", case))
    exe = str(tmp_path / "t")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wno-unused-variable", "-I", str(tmp_path), "-I", CSRC, "-o", exe,
                    str(tmp_path / "t.cpp")], check=True, capture_output=True, text=True)
    return subprocess.run([exe], capture_output=True, text=True)


@pytest.mark.parametrize("name", sorted(CASES))
def test_pool(name, tmp_path):
    r = run_case(CASES[name], tmp_path)
    assert r.returncode == 0, r.stdout


ON_GPU = """
import time, torch
import paper_2312_07440_amd as mg
from synth import generate_events
mom = torch.from_numpy(generate_events("gg_ttggg", 2000, first_event=5)).cuda()
out = torch.empty((16, 2000), dtype=torch.float64, device="cuda")
def call():
    p = mg.Process("gg_ttggg", "mixed")
    p.set_params([{"kappa_ttg": 0.9 + 0.01 * k} for k in range(16)])
    p.reweight(mom, out=out)
    return p
def free():
    torch.cuda.synchronize()
    time.sleep(0.5)              # released memory is counted as free with some delay
    return torch.cuda.mem_get_info()[0]
call().close()
a = free()                       # code objects and streams are there from now on
p = call()
b = free()
p.close()
c = free()
call().close()                   # closed while the kernels run
d = free()
print("held with a handle:", a - b, "after it:", a - c, "closed before the work was done:", a - d, flush=True)
assert a - b > 1 << 30 and abs(a - c) < 1 << 28 and abs(a - d) < 1 << 28
"""


@pytest.mark.gpu
def test_memory_comes_back():
    """A process of its own: no other handle is open there."""
    r = subprocess.run([sys.executable, "-c", ON_GPU], cwd=ROOT, capture_output=True, text=True, timeout=110)
    print(r.stdout, r.stderr[-2000:], flush=True)
    assert r.returncode == 0


HELD = """
import sys, torch
import paper_2312_07440_amd as mg
from synth import generate_events
n = 1 << 20
mom = torch.from_numpy(generate_events("gg_ttgg", 4096)).cuda().repeat(1, 1, n // 4096).contiguous()
out = torch.empty((1, n), dtype=torch.float64, device="cuda")
def call(p, k):
    p.set_params([{"kappa_ttg": 1.1}])
    getattr(p, sys.argv[1])(mom[:, :, :k].contiguous(), out=out[:, :k])
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
with torch.no_grad():
    call(mg.Process("gg_ttgg", "mixed"), 64)     # code objects
    a = torch.cuda.mem_get_info()[0]
    p = mg.Process("gg_ttgg", "mixed")
    call(p, n)
    print((a - torch.cuda.mem_get_info()[0]) / n)
"""


@pytest.mark.gpu
@pytest.mark.parametrize("call,need", [("reweight", 1984 + 352 + 8), ("reweight_kpoly", 1984 + 160 + 4)])
def test_bytes_per_event(call, need):
    """What a g g -> t tbar g g call holds per event: the record's kinematics
    and the wavefunctions' table or bases, whichever the call reads, a list
    entry, the base |M|^2, and up to 64 MiB that allocations are rounded up by."""
    r = subprocess.run([sys.executable, "-c", HELD, call], cwd=ROOT, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stderr[-2000:]
    held = float(r.stdout.split()[-1])
    print(call, held, "bytes per event", flush=True)
    assert need <= held <= need + 16 + 64
