"""CPU check of what a decode call sets up (nx_capi.cpp, built here for the host
with stand-ins for the kernels and the HIP calls): the LDS limit of the decoder
that the call launches is raised before, and of no other. The set-up is on the
host path of every call.
"""
import os
import subprocess

import numpy as np
import pytest

from paper_2201_05213_amd import blob as nxblob

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2201_05213_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>
#include "nellox.h"
#include "nx_kernels.hpp"
using namespace nx;
static std::string log_;
static int teams_;
#define OK return hipSuccess
namespace nx {
bool supported(int, int) { return true; }
int decode_teams(const TeamQuery& q) { return q.order == 0 ? 0 : teams_; }
hipError_t prepare_team(int, int, int K) { log_ += " set:team" + std::to_string(K); OK; }
hipError_t prepare_rows(int, int) { log_ += " set:rows"; OK; }
hipError_t prepare_decode(int, int, int K) { log_ += " set:wave" + std::to_string(K); OK; }
hipError_t launch_decode_team(int, int, const DecArgs& a, int, hipStream_t) { log_ += " run:team" + std::to_string(a.K); OK; }
hipError_t launch_decode_rows(int, int, const DecArgs&, int, hipStream_t) { log_ += " run:rows"; OK; }
hipError_t launch_decode(int, int, const DecArgs& a, int, int, size_t, hipStream_t) { log_ += " run:wave" + std::to_string(a.K); OK; }
hipError_t launch_sample(int, int, const DecArgs& a, int, int, size_t, hipStream_t) { log_ += " run:wave" + std::to_string(a.K); OK; }
hipError_t launch_decode_prep(int32_t*, int, int32_t*, hipStream_t, int32_t*, int64_t) { OK; }
hipError_t launch_pass(int, int, const PassArgs&, int, hipStream_t) { OK; }
hipError_t launch_pack(const PackArgs&, hipStream_t) { OK; }
hipError_t launch_rans_encode(const RansEncArgs&, hipStream_t) { OK; }
hipError_t launch_reduce_bits(const ImgDesc*, int, const float*, double*, double*, hipStream_t) { OK; }
hipError_t launch_check_monotone(unsigned long long*, hipStream_t) { OK; }
hipError_t launch_wgrad(int, int, const WgradArgs&, int, hipStream_t) { OK; }
hipError_t launch_swizzle(const float*, int, int, int, int, float*, int64_t, float*, int64_t, hipStream_t) { OK; }
hipError_t launch_bits_img(const float*, int, int64_t, double*, hipStream_t) { OK; }
hipError_t launch_train_fwd(int, int, const TrainArgs&, int, hipStream_t) { OK; }
hipError_t launch_train_bwd(int, int, const TrainArgs&, int, hipStream_t) { OK; }
hipError_t launch_grad_reduce(const GradReduceArgs&, hipStream_t) { OK; }
int wgrad_blocks_per_cu(int, int) { return 1; }
hipError_t static_scratch(void** p) { static void* s = malloc(STATIC_SCRATCH_BYTES); *p = s; OK; }
}
extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; OK; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  p->sharedMemPerBlock = 160 << 10;
  OK;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; OK; }
hipError_t hipMalloc(void** p, size_t n) { *p = malloc(n); OK; }
hipError_t hipFree(void* p) { free(p); OK; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = malloc(n); OK; }
hipError_t hipHostFree(void* p) { free(p); OK; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); OK; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); OK; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; OK; }
hipError_t hipEventDestroy(hipEvent_t) { OK; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { OK; }
hipError_t hipEventSynchronize(hipEvent_t) { OK; }
const char* hipGetErrorString(hipError_t) { return ""; }
}
int main(int, char** argv) {
  FILE* f = fopen(argv[1], "rb");
  std::vector<uint8_t> blob(1 << 20);
  blob.resize(fread(blob.data(), 1, blob.size(), f));
  nellox_model* m = nullptr;
  if (nellox_model_create(blob.data(), blob.size(), &m)) { printf("model: %s\n", nellox_last_error()); return 1; }
  std::vector<uint8_t> px(64 * 64 * 3), in(64), ws(64 << 20);
  uint64_t offs[2] = {0, 64}, seed = 1;
  int32_t status;
  nellox_image im{};
  im.px = px.data(); im.H = 64; im.W = 64;
  for (teams_ = 0; teams_ <= 2; ++teams_)
    for (int order = 0; order <= 2; ++order)
      for (int K : {1, 2, 4, 8, 16, -1, 0}) {
        if ((order == 0 && K != 1 && K != 0) || (order == 2 && K == -1)) continue;
        nellox_opts o{};
        o.order = order; o.interleave = K;
        log_.clear();
        nellox_status st;
        if (K == 0) {
          o.interleave = 1;
          st = nellox_sample(m, 1, &seed, &o, &im, ws.data(), ws.size(), nullptr);
        } else {
          st = nellox_decode(m, 1, in.data(), offs, &o, &im, &status, ws.data(), ws.size(), nullptr);
        }
        printf("%d %d %d %d%s\n", (int)st, teams_, order, K, log_.c_str());
      }
}
"""


def test_a_decode_sets_up_the_decoder_it_launches(tmp_path):
    src, exe, model = tmp_path / "setup.cpp", tmp_path / "setup", tmp_path / "model.nlxw"
    src.write_text(DRIVER)
    dims = (3, 16, 1, 10)
    model.write_bytes(nxblob.blob_from_params(dims, np.zeros(nxblob.param_count(*dims[:3]), "<f4")))
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I",
                        os.path.join(ROOT, "include"), "-I", "/opt/rocm/include", str(src),
                        os.path.join(CSRC, "nx_capi.cpp"), "-o", str(exe)], capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail("host build of nx_capi.cpp failed:\n" + r.stderr[-3000:])
    out = subprocess.run([str(exe), str(model)], capture_output=True, text=True, timeout=60, check=True).stdout
    rows = [line.split() for line in out.splitlines()]
    assert len(rows) == 3 * (2 + 7 + 6)
    for status, teams, order, K, *calls in rows:
        case = (teams, order, K, calls)
        assert status == "0", case
        assert len(calls) == 2, case
        (done, what), (run, ran) = (c.split(":") for c in calls)
        assert (done, run) == ("set", "run") and what == ran, case
        kind = "rows" if K == "-1" else "wave" if teams == "0" or order == "0" else "team"
        assert ran.startswith(kind), case
