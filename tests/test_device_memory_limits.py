"""Uploads near the end of device memory: the host side of the library
(lf_api.cpp as it stands) built with g++ over a model of the device runtime
whose memory has a limit.  Nothing here touches a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
API = os.path.join(ROOT, "paper_2402_14670_amd", "csrc", "lf_api.cpp")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

DRIVER = r'''
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>
#include "lf_internal.h"
#include "lf.h"

static size_t g_limit = ~size_t(0) / 2, g_held = 0;
static std::map<void *, size_t> g_blocks;
extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    if (g_held + n > g_limit) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    g_blocks[*p] = n;
    g_held += n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    if (!g_blocks.count(p)) { std::printf("free of unknown memory\n"); std::exit(3); }
    g_held -= g_blocks[p];
    g_blocks.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)1; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *, unsigned) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
}
namespace lfk {
hipError_t fixed_scratch(void **p) { static char mem[16]; *p = mem; return hipSuccess; }
hipError_t launch_find(const DevBatch &, const KParams *, int, int, int, const ExecCfg &, const uint32_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_event_index(const DevBatch &, const KParams *, uint8_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_count(const DevBatch &, const KParams *, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_poison(const DevBatch &, hipStream_t) { return hipSuccess; }
hipError_t launch_zero_words(uint32_t *, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_fit_table(const KParams *, FitRow *, hipStream_t) { return hipSuccess; }
int persistent_blocks_per_cu(int, int, const ExecCfg &) { return 1; }
void plane_constants(KParams &) {}
}

struct Events {   // n events without hits, all tracks in the last one
    std::vector<uint32_t> ho, to;
    std::vector<float> v;
    lf_batch b{};
    Events(uint32_t n, uint32_t tracks) : ho(24 * n + 1, 0), to(n + 1, 0), v(tracks, 0.5f) {
        to[n] = tracks;
        b.n_events = n;
        b.hit_off = ho.data();
        b.trk_off = to.data();
        b.trk_x = b.trk_y = b.trk_tx = b.trk_ty = b.trk_qop = v.data();
    }
};
#define CHECK(c) if (!(c)) { std::printf("line %%d: " #c " (held %%zu)\n", __LINE__, g_held); return 1; }
int main() {
    lf_geometry g{};
    for (int l = 0; l < 12; ++l) g.z[l] = 7800.0f + 100 * l;
    g.kick = 1.0f;
    g.polarity = 1;
    lf_params p;
    lf_default_params(&p);
    lf_ctx *c = nullptr;
    CHECK(lf_create(&g, &p, 0, &c) == LF_OK);
    const size_t base = g_held;
    Events many(1000, 10), tracks(1, 20000);
    uint64_t id = 0;
    CHECK(lf_upload_events(c, &many.b, nullptr, &id) == LF_OK);
    const size_t with_index = g_held;
    CHECK(with_index > base + 3840 * 1000);          // the search indexes beside the block
    CHECK(lf_release_batch(c, id) == LF_OK);
    CHECK(g_held == with_index);                     // both kept
    // room for the next batch's block only where the kept indexes are
    size_t block = 0;
    {
        lf_ctx *probe = nullptr;
        CHECK(lf_create(&g, &p, size_t(1) << 30, &probe) == LF_OK);
        uint64_t pid = 0;
        CHECK(lf_upload_events(probe, &tracks.b, nullptr, &pid) == LF_OK);
        CHECK(lf_batch_info(probe, pid, nullptr, nullptr, nullptr, &block) == LF_OK);
        lf_destroy(probe);
    }
    CHECK(g_held == with_index);
    CHECK(block < 3840 * 1000);
    g_limit = base + block + 3840;
    CHECK(lf_upload_events(c, &tracks.b, nullptr, &id) == LF_OK);
    CHECK(lf_release_batch(c, id) == LF_OK);
    // memory for the block alone: the batch goes without indexes
    g_limit = base + block;
    CHECK(lf_upload_events(c, &tracks.b, nullptr, &id) == LF_OK);
    CHECK(lf_release_batch(c, id) == LF_OK);
    g_limit = base + block - 1;
    Events more(1, 20300);
    CHECK(lf_upload_events(c, &more.b, nullptr, &id) == LF_ERR_NOMEM);
    lf_destroy(c);
    CHECK(g_held == 0);
    std::printf("ok\n");
    return 0;
}
'''


def test_kept_indexes_are_given_back_before_an_upload_fails(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("no g++ or no HIP headers on this host")
    prog = tmp_path / "limits.cpp"
    prog.write_text(DRIVER.replace("%%", "%"))
    exe = tmp_path / "limits"
    build = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-w", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                            "-I", os.path.dirname(API), "-I", os.path.join(ROOT, "include"), str(prog), API, "-o", str(exe)],
                           capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-3000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "ok" in run.stdout, (run.returncode, run.stdout, run.stderr[-2000:])
