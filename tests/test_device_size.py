"""A device of another number of compute units than the usual: what a plan, its workspace and its first call are laid out by
is the same number. The runtime and the launches are stand-ins, so this runs on the host."""
import os
import subprocess

import pytest

from paper_2510_18546_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# reads compute units, KV heads, tokens, splits; prints the scratch's bytes before and after the first attention call, the waves
# (`sub`) and tiles (`once_tiles`) that the launch was given and the partial results that the merge was
DRIVER = '''
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "en_internal.h"
static int units, sub, tiles, partial = 1;
extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = units; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) { memset(p, 0, sizeof *p); p->multiProcessorCount = units; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = malloc(n); return hipSuccess; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorNotFound; }
}
int en_launch_attention(const en_pool *, const EnAttnArgs &a, void *) { sub = a.sub; tiles = a.once_tiles; return 0; }
int en_launch_combine(const en_pool *, const EnAttnArgs &a, const EnMassArgs &, void *) { partial = a.n_splits; return 0; }
int main() {
    int kv, tokens, splits;
    if (scanf("%d %d %d %d", &units, &kv, &tokens, &splits) != 4) return 1;
    en_pool_desc d = {};
    d.n_kv_heads = kv; d.n_q_heads = 4 * kv; d.n_groups = 1; d.capacity = tokens; d.max_ctx = tokens + 1;
    d.head_dim = 128; d.dtype = EN_BF16; d.rope_base = 1e4;
    const int32_t len = tokens, sel = 0, ptr[2] = {0, 1};
    en_pool *pool = nullptr; en_plan *plan = nullptr;
    if (kv_pool_create(&d, (void *)256, (void *)256, &len, &pool) != EN_OK) return 2;
    if (segment_select(pool, 1, &sel, ptr, 1, &plan) != EN_OK) return 3;
    if (splits && en_plan_set_splits(plan, splits) != EN_OK) return 4;
    const size_t before = en_workspace_bytes(pool, plan);
    void *at = (void *)4096;
    if (segmented_prefill_attention(pool, plan, at, at, at, at, at, before, nullptr) != EN_OK) return 5;
    printf("%zu %zu %d %d %d\\n", before, en_workspace_bytes(pool, plan), sub, tiles, partial);
    en_plan_destroy(plan); kv_pool_destroy(pool);
    return 0;
}
'''


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    at = tmp_path_factory.mktemp("device")
    src, exe = at / "device.cpp", at / "device"
    src.write_text(DRIVER)
    csrc, inc = os.path.join(ROOT, "paper_2510_18546_amd", "csrc"), os.path.join(ROOT, "include")
    B.load()
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", inc, "-I", csrc,
                           str(src), "-o", str(exe), "-rdynamic", B._build.LIB_PATH,
                           "-Wl,-rpath," + os.path.dirname(B._build.LIB_PATH)])
    return str(exe)


@pytest.mark.parametrize("units", [32, 64, 128, 256, 304, 512])
@pytest.mark.parametrize("kv,tokens,splits", [(8, 11000, 35), (8, 11000, 0), (2, 500, 0), (64, 1200, 0), (64, 1200, 5), (16, 4000, 17), (300, 200, 1)])
def test_first_call_agrees_with_its_workspace(driver, kv, tokens, splits, units):
    run = subprocess.run([driver], input=f"{units} {kv} {tokens} {splits}", capture_output=True, text=True, check=True)
    before, after, sub, tiles, partial = map(int, run.stdout.split())
    assert before == after
    assert tiles == 0 or sub == 1                # the one-pass kernel leaves one result a split
    if splits:
        assert partial == splits * sub
