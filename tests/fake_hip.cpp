// Host-only stand-ins for the HIP runtime calls and kernel launches that the library's host files
// make, so that their bookkeeping runs without a GPU: "device" memory is host memory of exactly the
// size asked for, and a launch checks that the arrays which its kernel writes by tile hold as many
// entries as it would write.  Compiled together with pic_capi.cpp and pic_batch.cpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

#include "pic_internal.h"

static std::map<const char *, size_t> g_live;
static int g_short = 0;  // launches with an array shorter than they write

extern "C" int fake_short_arrays() { return g_short; }

static void need(const void *p, size_t bytes, const char *what) {
  const char *q = static_cast<const char *>(p);
  auto it = g_live.upper_bound(q);
  size_t have = 0;
  if (it != g_live.begin()) {
    --it;
    if (q < it->first + it->second) have = (size_t)(it->first + it->second - q);
  }
  if (have >= bytes) return;
  ++g_short;
  std::printf("%s: %zu bytes needed, %zu there\n", what, bytes, have);
}

extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 160 * 1024; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *, int) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMalloc(void **p, size_t n) {
  *p = std::malloc(n);
  g_live[static_cast<char *>(*p)] = n;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  g_live.erase(static_cast<char *>(p));
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 0; return hipSuccess; }
}

namespace pic {

// Rough sizes of the kernels' LDS, in the right order of each other: accumulators and fields per
// cell of the tile and its ring, and the staging per wavefront.
size_t particle_lds_bytes(const GridArgs &g, const TileArgs &t, bool mixed, int waves) {
  const size_t cells = (size_t)(t.tx + 2) * (t.tz + 2);
  return cells * ((size_t)g.n_planes * 8 + (mixed ? 36 : 72) + 100) + (size_t)waves * 5472;
}
size_t runs_lds_bytes(const GridArgs &g, const TileArgs &t, bool pw) {
  return particle_lds_bytes(g, t, true, 0) + (pw ? 11264 : 10240);
}
size_t rank_lds_bytes(const TileArgs &t) { return (size_t)(t.tx + 4) * (t.tz + 4) * 88; }

static void tiles_need(const StepArgs &a, const char *what) {
  need(a.tile_active_next, (size_t)a.t.ntiles, what);
  need(a.tile_list_next, ((size_t)a.t.ntiles + 1) * sizeof(int32_t), what);
}
hipError_t launch_tile_list(const StepArgs &a, bool, hipStream_t) { tiles_need(a, "tile list"); return hipSuccess; }
hipError_t launch_particles(const StepArgs &a, bool push, hipStream_t) {
  if (push) tiles_need(a, "particles");
  return hipSuccess;
}
hipError_t launch_particles_alt(const StepArgs &a, bool push, int, bool, int32_t, hipStream_t) {
  if (push) tiles_need(a, "particles");
  return hipSuccess;
}
hipError_t launch_sort(const StepArgs &a, hipStream_t) { tiles_need(a, "sort"); return hipSuccess; }
hipError_t launch_batch_cycle(const BatchArgs &b, const BatchLaunch &l, hipStream_t) {
  for (int r = 0; r < 2 * b.nruns; ++r) {
    tiles_need(b.step[r], "batch cycle");
    for (int s = 0; s < b.step[r].nsp; ++s)
      if (b.step[r].sp[s].active) need(b.step[r].sp[s].cs, (size_t)(b.step[r].g.ncells + 1) * sizeof(int32_t), "cell starts");
  }
  return l.lds_particles <= 160 * 1024 ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_field_solve(const FieldArgs &, hipStream_t) { return hipSuccess; }
hipError_t launch_iota(int32_t *p, int64_t n, hipStream_t) {
  for (int64_t i = 0; i < n; ++i) p[i] = (int32_t)i;
  return hipSuccess;
}
hipError_t launch_energy(const StepArgs &, const double *, const double *, double *, hipStream_t) { return hipSuccess; }
hipError_t launch_energy_scratch(const StepArgs &, const double *, const double *, double *, hipStream_t) { return hipSuccess; }
hipError_t energy_scratch(int32_t, double **) { return hipErrorInvalidDevice; }

}  // namespace pic
