// TEST INFRASTRUCTURE: which launches advance which channels, without a GPU.
//
// Stands in for the HIP runtime and for the sweep launchers of the runtime
// (lb_runtime.hip, linked with this file instead of lb_kernels.hip): copies
// between the workspace and the host are plain copies, captured launches are
// kept and replayed, and every launcher books on each channel of its list what
// the kernel would do. A booking fails unless the list covers every node of the
// channel once, reads the buffer the channel's last launch wrote, starts at the
// channel's own step, and (pressure drive) the boundary of the step before was
// applied, once.
//
// host_routing <fp32|fp64> <K> <viscoelastic> <stress_force> <steps_per_sweep>
//              <steps[,steps...]> <nx,ny,pressure,wall,zou_he> ...
// prints for each channel the steps it took by each launcher and the most
// steps of one launch; exit status 0 if every booking held.
#include <sys/mman.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <sstream>
#include <string>
#include <vector>

#include "lb.h"
#include "lb_internal.h"

using namespace lbnlm;

namespace {
int g_fails = 0;
bool g_recording = false;
std::vector<std::function<void()>> g_capture;
std::map<void *, std::vector<std::function<void()>>> g_graphs;

void failed(int ch, const std::string &what) {
  if (++g_fails <= 20) std::printf("FAILED channel %d: %s\n", ch, what.c_str());
}
hipError_t enqueue(std::function<void()> f) {
  if (g_recording) g_capture.push_back(std::move(f));
  else f();
  return hipSuccess;
}

struct Book {
  const void *last = nullptr;  // buffer the last launch wrote
  long long steps = 0;
  int owed = 0;                // boundaries of the last step not yet applied
  std::map<std::string, long long> by;
  int most = 0;
};
std::map<int, Book> g_books;

// books S steps of every channel of the list; cols: columns of a strip
void book(const std::string &name, const void *A, const void *B, const ChanDev *ch, const Strip *strips, int n, int k,
          int S, bool boundary, const std::function<int(const Strip &, const ChanDev &)> &cols) {
  std::map<int, long long> area;
  for (int i = 0; i < n; ++i) {
    const Strip &s = strips[i];
    const ChanDev &c = ch[s.ch];
    const int w = cols(s, c);
    if (s.x0 < 0 || s.y0 < 0 || s.x0 + w > c.nx || s.y1 > c.ny || w < 1 || s.y1 <= s.y0)
      failed(s.ch, name + ": strip out of the channel");
    area[s.ch] += (long long)w * (s.y1 - s.y0);
  }
  for (auto &[i, nodes] : area) {
    const ChanDev &c = ch[i];
    Book &b = g_books[i];
    if (!c.active) continue;  // (the kernels skip it)
    if (nodes != (long long)c.nx * c.ny) failed(i, name + ": list does not cover the channel");
    if (b.last && b.last != A) failed(i, name + ": reads a buffer the channel is not in");
    if (c.t + k != b.steps) failed(i, name + ": not at the channel's step");
    if (b.owed) failed(i, name + ": the step before has no boundary");
    if (boundary && !c.gpbc) failed(i, name + ": boundary of a channel without one");
    b.owed = c.gpbc && !boundary;
    b.last = B;
    b.steps += S;
    b.by[name] += S;
    b.most = std::max(b.most, S);
  }
}
int rest_of(int x0, int w, int nx) { return std::min(w, nx - x0); }
}  // namespace

// ---- the HIP runtime
extern "C" {
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(8);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
  *p = reinterpret_cast<void *>(256);
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  g_recording = true;
  g_capture.clear();
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  g_recording = false;
  *g = reinterpret_cast<hipGraph_t>(8);
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  static uintptr_t next = 16;
  *e = reinterpret_cast<hipGraphExec_t>(next += 16);
  g_graphs[*e] = g_capture;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  for (auto &f : g_graphs[e]) f();
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}

// ---- the launchers
namespace lbnlm {
hipError_t launch_sweep(int fp32, int cls, bool observe, const SweepArgs &a, hipStream_t) {
  if (observe) return hipSuccess;
  return enqueue([=] {
    book("sweep", a.A, a.B, a.ch, a.strips, a.n_strips, a.k, 1, false, [=](const Strip &s, const ChanDev &c) {
      return is_strip_class(cls) ? rest_of(s.x0, strip_cols(cls, fp32 ? 4 : 8), c.nx) : c.nx;
    });
  });
}
hipError_t launch_tiles(const SweepArgs &a, hipStream_t) {
  return enqueue([=] {
    book("tiles", a.A, a.B, a.ch, a.strips, a.n_strips, a.k, 1, false,
         [](const Strip &s, const ChanDev &c) { return rest_of(s.x0, kMainTileX, c.nx); });
  });
}
hipError_t launch_saf_fused(const double *A, double *B, const ChanDev *ch, const Strip *tiles, int n, int k, int, int,
                            hipStream_t) {
  return enqueue([=] {
    book("tiles", A, B, ch, tiles, n, k, 1, false,
         [](const Strip &s, const ChanDev &c) { return rest_of(s.x0, kSafTileX, c.nx); });
  });
}
hipError_t launch_two_step(bool, const SweepArgs &a, hipStream_t) {
  return enqueue([=] {
    book("two_step", a.A, a.B, a.ch, a.strips, a.n_strips, a.k, 2, false,
         [](const Strip &s, const ChanDev &) { return s.x1 - s.x0; });
  });
}
hipError_t launch_narrow_two_step(bool, int nx, const SweepArgs &a, hipStream_t) {
  return enqueue([=] {
    book("narrow_two_step", a.A, a.B, a.ch, a.strips, a.n_strips, a.k, 2, false,
         [=](const Strip &, const ChanDev &) { return nx; });
  });
}
hipError_t launch_blocks(bool, bool gpbc, bool stress_force, int threads, const SweepArgs &a, int S, hipStream_t) {
  return enqueue([=] {
    const int halo = (stress_force ? 3 : 2) * S;
    for (int i = 0; i < a.n_strips; ++i) {
      const Strip &s = a.strips[i];
      const ChanDev &c = a.ch[s.ch];
      const int w = s.x1 - s.x0 >= c.nx ? c.nx : s.x1 - s.x0 + 2 * halo;
      const int rows = std::min(s.y1 + halo, c.ny) - std::max(s.y0 - halo, 0);
      if ((long long)w * rows > threads) failed(s.ch, "box does not fit its workgroup");
      if (gpbc && S > 1 && rows != c.ny) failed(s.ch, "box without whole columns");
    }
    book("boxes", a.A, a.B, a.ch, a.strips, a.n_strips, a.k, S, gpbc,
         [](const Strip &s, const ChanDev &) { return s.x1 - s.x0; });
  });
}
hipError_t launch_gpbc(int, void *B, const ChanDev *ch, int n, int k, const float *, bool boxed, hipStream_t) {
  return enqueue([=] {
    for (int i = 0; i < n; ++i) {
      if (!column_pass_takes(ch[i], boxed)) continue;
      Book &b = g_books[i];
      if (!b.owed) failed(i, "column pass: no boundary to apply");
      if (b.last != B) failed(i, "column pass: not the buffer just written");
      if (ch[i].t + k + 1 != b.steps) failed(i, "column pass: not of the step just taken");
      b.owed = 0;
      ++b.by["column_pass"];
    }
  });
}
hipError_t launch_advance(ChanDev *ch, int n, int steps, hipStream_t) {
  return enqueue([=] {
    for (int i = 0; i < n; ++i) ch[i].t += steps;
  });
}
hipError_t launch_reduce(const ChanDev *, int, const double *, double *, double *, double *, const float *, int, int,
                         hipStream_t) {
  return hipSuccess;
}
hipError_t launch_rereference(float *, const ChanDev *, int, int, const double *, float *, hipStream_t) {
  return hipSuccess;
}
hipError_t launch_saf_observe(const double *, const ChanDev *, int, long long, int, double *, double *, double *,
                              hipStream_t) {
  return hipSuccess;
}
int narrow_two_step_blocks_per_cu(bool) { return 4; }
int two_step_blocks_per_cu(bool fp32, bool, bool) { return fp32 ? 6 : 4; }
}  // namespace lbnlm

int main(int argc, char **argv) {
  if (argc < 8) return 2;
  lb_options o{};
  o.precision = std::strcmp(argv[1], "fp32") ? LB_FP64 : LB_FP32_SHIFTED;
  o.obs_every = std::atoi(argv[2]);
  o.viscoelastic = std::atoi(argv[3]);
  o.stress_force = std::atoi(argv[4]);
  o.steps_per_sweep = std::atoi(argv[5]);
  std::vector<lb_channel> cs;
  for (int i = 7; i < argc; ++i) {
    int nx, ny, pressure, wall, zh;
    if (std::sscanf(argv[i], "%d,%d,%d,%d,%d", &nx, &ny, &pressure, &wall, &zh) != 5) return 2;
    lb_channel c{};
    c.nx = nx;
    c.ny = ny;
    c.tau_lb = 1.0;
    c.G = 1e-4;
    c.tau0 = 1e3;
    c.gamma_c = 0.1;
    c.t_startup = 1000;
    c.force = pressure ? 0.0 : 1e-6;
    c.pressure_gradient = pressure ? 1e-6 : 0.0;
    c.wall_velocity = wall ? 1e-3 : 0.0;
    c.top_wall = zh ? LB_WALL_ZOU_HE : LB_WALL_HALFWAY;
    cs.push_back(c);
  }
  size_t bytes = 0;
  if (lb_workspace_bytes(cs.data(), (int)cs.size(), &o, &bytes) != LB_OK) return 2;
  // untouched pages of it cost nothing
  void *ws = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (ws == MAP_FAILED) return 2;
  lb_handle *h = nullptr;
  if (lb_create(cs.data(), (int)cs.size(), &o, ws, bytes, nullptr, &h) != LB_OK) return 2;
  long long total = 0;
  std::stringstream steps(argv[6]);
  for (std::string v; std::getline(steps, v, ',');) {
    const long long n = std::atoll(v.c_str());
    if (lb_step(h, n) != LB_OK) failed(-1, std::string("lb_step: ") + lb_last_error(h));
    total += n;
  }
  for (int i = 0; i < (int)cs.size(); ++i) {
    Book &b = g_books[i];
    if (b.steps != total) failed(i, "not every step taken");
    if (b.owed) failed(i, "the last step has no boundary");
    std::printf("channel %d most=%d", i, b.most);
    for (auto &[name, n] : b.by) std::printf(" %s=%lld", name.c_str(), n);
    std::printf("\n");
  }
  lb_destroy(h);
  return g_fails ? 1 : 0;
}
