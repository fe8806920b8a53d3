// Host driver for what the library's calls launch and in which order, without
// a GPU: the HIP runtime's entry points that those calls use are defined here
// (the library, linked dynamically, then calls these), "device" buffers are
// host memory, and of the kernels only what they do to the control block is
// carried out.  Any of the launches and copies of a call can be made to fail.
// Built and run by tests/test_launch_host.py, which names the check to run.
#include <dlfcn.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/ars.h"
#include "../../paper_1903_09043_amd/csrc/ars_fused.h"
#include "../../paper_1903_09043_amd/csrc/ars_internal.h"

namespace {

int ops = 0;             // launches and copies of the present call
int fail_at = -1;        // the one that fails
hipError_t pending = hipSuccess;
double state_rate = 1.0; // rate of every state that a step kernel writes
unsigned last_block = 0; // threads of the last k_batch workgroup
unsigned last_grid = 0;  // workgroups of the last k_step_fused
unsigned best_grid = 0;
int num_cu = 256;

hipError_t op() {
  if (ops++ != fail_at) return hipSuccess;
  pending = hipErrorLaunchFailure;
  return pending;
}

double largest(const ars::RateMax* m) {
  double v = 0.0;
  for (unsigned long long w : m->w) {
    double x;
    std::memcpy(&x, &w, sizeof x);
    v = std::max(v, x);
  }
  return v;
}

void fold(ars::RateMax* m, double v) {
  unsigned long long b;
  std::memcpy(&b, &v, sizeof b);
  m->w[0] = std::max(m->w[0], b);
}

void clear(ars::Control* c) {
  for (auto& m : c->lammax) std::memset(&m, 0, sizeof m);
}

}  // namespace

extern "C" {

hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** a, size_t, hipStream_t) {
  const hipError_t e = op();
  if (e != hipSuccess) return e;
  Dl_info info{};
  const std::string name = dladdr(f, &info) && info.dli_sname ? info.dli_sname : "";
  if (name.find("k_step_fused") != std::string::npos) {
    const ars::Params& P = *(const ars::Params*)a[0];
    const ars::StepIO& io = *(const ars::StepIO*)a[3];
    last_grid = grid.x;
    const double dt = io.rate_in ? P.cfl / largest(io.rate_in) : *io.dt_in;
    if (io.dt_log) *io.dt_log = dt;
    if (io.clear_slot) std::memset(io.clear_slot, 0, sizeof *io.clear_slot);
    if (io.rate_out) fold(io.rate_out, state_rate);
  } else if (name.find("k_ctl_prep") != std::string::npos) {
    if (*(int*)a[1] == 0) clear(*(ars::Control**)a[0]);
  } else if (name.find("k_dt_finish") != std::string::npos) {
    ars::Control* c = *(ars::Control**)a[1];
    **(double**)a[3] = *(double*)a[0] / largest(&c->lammax[*(int*)a[2]]);
    clear(c);
  } else if (name.find("k_batch") != std::string::npos) {
    last_block = block.x;
  }
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  const hipError_t e = op();
  if (e == hipSuccess) std::memcpy(d, s, n);
  return e;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = pending;
  pending = hipSuccess;
  return e;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? num_cu : 0;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 8;
  return hipSuccess;
}

// A call takes the less time, the nearer its workgroups' number is to best_grid.
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::malloc(n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f + (float)std::abs((long)last_grid - (long)best_grid);
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = num_cu;
  return hipSuccess;
}

static struct { dim3 g, b; size_t m; hipStream_t s; } config;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) {
  config = {g, b, m, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = config.g;
  *b = config.b;
  *m = config.m;
  *s = config.s;
  return hipSuccess;
}

}  // extern "C"

namespace {

ars_config rb2d(int nx, int nz) {
  ars_config c{};
  c.dim = 2;
  c.n[0] = nx;
  c.n[1] = nz;
  c.n[2] = 1;
  c.L[0] = 2.0;
  c.L[1] = c.L[2] = 1.0;
  c.gamma = 5.0 / 3.0;
  c.g = 1.0;
  c.mu = 2e-3;
  c.kappa = 3e-3;
  c.K = 1.1;
  c.cfl = 0.4;
  c.low_mach = 1;
  c.bc[1][0] = c.bc[1][1] = ARS_BC_WALL;
  c.wall_noslip = 1;
  c.thermal[0] = c.thermal[1] = ARS_T_FIXED;
  c.T_wall[0] = 1.0;
  c.T_wall[1] = 0.5;
  return c;
}

// A call of n CFL steps that fails at any of its launches or copies, on states
// of rate 100, then one on states of rate 1 with the same workspace: the time
// steps of the second are those of its own states.
int failed_step() {
  int bad = 0;
  const ars_config cfg = rb2d(8, 6);
  ars_ctx* x = nullptr;
  if (ars_create(&cfg, &x) != ARS_OK) return 1;
  const size_t len = ars_state_len(x);
  std::vector<double> A(len), B(len), C(len), D(len), work(ars_workspace_bytes(x) / 8 + 1);
  double t = 0.0, dt = 0.0, log[4];
  for (int to = 0; to < 2; ++to) {
    auto call = [&](int n) {
      ops = 0;
      const int rc = to ? ars_step_to(x, A.data(), B.data(), C.data(), D.data(), work.data(), n, &t, &dt, log, nullptr)
                        : ars_step(x, A.data(), B.data(), work.data(), n, &t, &dt, log, nullptr);
      pending = hipSuccess;
      return rc;
    };
    for (int n = 1; n <= 4; ++n) {
      fail_at = -1;
      ars_workspace_init(x, work.data(), nullptr);
      if (call(n) != ARS_OK) return 1;
      const int total = ops;
      for (int k = 0; k < total; ++k) {
        ars_workspace_init(x, work.data(), nullptr);
        state_rate = 100.0;
        dt = cfg.cfl;
        fail_at = k;
        const int rc = call(n);
        fail_at = -1;
        state_rate = 1.0;
        dt = cfg.cfl;
        const int rc2 = call(4);
        bool ok = rc == ARS_EDEVICE && rc2 == ARS_OK && dt == cfg.cfl;
        for (double d : log) ok = ok && d == cfg.cfl;
        if (!ok) {
          ++bad;
          std::printf("to %d, %d steps, operation %d of %d failed: rc %d, then %d, dts %g %g %g %g, next %g\n", to, n, k,
                      total, rc, rc2, log[0], log[1], log[2], log[3], dt);
        }
      }
    }
  }
  ars_destroy(x);
  return bad;
}

// The tiling that the query reports is the one that the launch takes: its rows
// are the workgroup's, and setting it again changes neither the workgroup nor
// the table.
int batch_tiling() {
  int bad = 0;
  bool seen[2] = {false, false};
  std::vector<ars_config> mixed, one = {rb2d(64, 32), rb2d(64, 32), rb2d(64, 32)}, wide(700, rb2d(20, 12));
  for (int k = 0; k < 96; ++k) mixed.push_back(k % 3 == 0 ? rb2d(64, 32) : k % 3 == 1 ? rb2d(128, 64) : rb2d(256, 128));
  for (const auto& cfgs : {one, mixed, wide}) {
    for (int cus : {256, 32, 4}) {
      num_cu = cus;
      ars_batch* b = nullptr;
      if (ars_batch_create((int)cfgs.size(), cfgs.data(), &b) != ARS_OK) return 1;
      std::vector<double> U(1), T(1);  // addresses only
      std::vector<char> t1(ars_batch_table_bytes(b)), t2(t1.size());
      std::vector<int> zc(cfgs.size());
      int rows = 0;
      auto launch = [&](std::vector<char>& table) {
        last_block = 0;
        if (ars_batch_bind(b, U.data(), T.data(), table.data(), nullptr) != ARS_OK ||
            ars_batch_step(b, table.data(), 1, nullptr) != ARS_OK)
          return -1;
        return (int)last_block / 64;
      };
      const int ran = launch(t1);
      bool ok = ars_batch_get_tiling(b, &rows, zc.data()) == ARS_OK && rows == ran;
      ok = ok && ars_batch_set_tiling(b, rows, zc.data()) == ARS_OK && launch(t2) == ran && t1 == t2;
      seen[rows == 8] = true;
      if (!ok) ++bad;
      std::printf("%d instances, %d CUs: reported %d rows, launched %d, the same table when set: %d\n", (int)cfgs.size(),
                  cus, rows, ran, (int)(t1 == t2));
      ars_batch_destroy(b);
    }
  }
  return bad + !(seen[0] && seen[1]);
}

// The shares of a march's (tile, plane) pairs: every pair once, in order, none
// longer than another by more than one pair; and spread, laid end to end over
// the tiles, they are those of floor(w total / groups), so that no workgroup
// marches more planes, halo planes included, than with those.
int shares() {
  int bad = 0, whole = 0, by_tile = 0;
  auto planes = [](long long a, long long b, int nz, int halo) {
    long long c = 0;
    while (a < b) {
      const long long n = std::min<long long>(nz - a % nz, b - a);
      c += n + halo;
      a += n;
    }
    return c;
  };
  for (long long tiles : {1, 2, 7, 63, 208, 256, 257, 666, 832, 1000})
    for (int nz : {1, 2, 3, 4, 5, 7, 33, 67, 256, 1000})
      for (long long most : {1, 8, 255, 256, 1024, 8192})
        for (long long least : {1, 4, 37})
          for (int form = 0; form < 4; ++form) {
            const int halo = form & 1 ? 2 : 4;
            const bool spread = form & 2;
            const ars::Shares sh = ars::shares_of(tiles, nz, most, least, halo);
            const long long total = tiles * nz, G = sh.groups;
            long long at = 0, busiest = 0, even = 0;
            bool ok = G >= 1 && G <= most;
            for (long long w = 0; w < G && ok; ++w) {
              unsigned cur, stop;
              if (spread)
                ars::share_of<true>(sh, (unsigned)w, (unsigned)nz, cur, stop);
              else
                ars::share_of<false>(sh, (unsigned)w, (unsigned)nz, cur, stop);
              ok = cur == at && stop > cur && stop <= total && stop - cur - sh.share <= 1u;
              at = stop;
              busiest = std::max(busiest, planes(cur, stop, nz, halo));
              even = std::max(even, planes(total * w / G, total * (w + 1) / G, nz, halo));
            }
            ok = ok && at == total;
            if (sh.chunks == G && spread) {
              ++whole;
              ok = ok && busiest <= even;
            } else {
              ++by_tile;
            }
            if (!ok) {
              if (++bad <= 10)
                std::printf("%lld tiles of %d planes, %lld workgroups of at most %lld: up to %lld planes against %lld\n", tiles,
                            nz, G, most, busiest, even);
            }
          }
  return bad + !(whole && by_tile);
}

// Every share has one workgroup, and those of an XCD (workgroups are dealt to
// the eight in turn) are one run of consecutive shares, for any count.
int placement() {
  int bad = 0;
  for (unsigned G = 1; G <= 3000; ++G) {
    std::vector<int> taken(G, 0);
    bool ok = true;
    for (unsigned b = 0; b < G; ++b) {
      const unsigned w = ars::xcd_share(b, G);
      ok = ok && w < G && !taken[w]++ && (b < 8 || w == ars::xcd_share(b - 8, G) + 1);
    }
    if (!ok && ++bad <= 5) std::printf("%u workgroups\n", G);
  }
  return bad;
}

// A 2D step whose pairs, in shares no longer than the default, give each SIMD
// at most one workgroup (a wave) never puts two on one, and shares of one plane
// are left where there are no more pairs than SIMDs.
int one_wave() {
  int bad = 0;
  std::vector<double> work(8192);
  double d[2] = {1e-3, 1e-3};
  for (int cus : {256, 64}) {
    num_cu = cus;
    for (int nz = 3; nz <= 24 * cus; nz += nz / 23 + 1) {
      const ars_config cfg = rb2d(60, nz);
      ars_ctx* x = nullptr;
      if (ars_create(&cfg, &x) != ARS_OK) return 1;
      if (ars_workspace_bytes(x) > work.size() * 8) work.resize(ars_workspace_bytes(x) / 8);
      std::vector<double> A(ars_state_len(x)), B(A.size());
      const int simds = 4 * cus;
      if (nz > simds * ars_get_zchunk(x)) {
        ars_destroy(x);
        break;
      }
      last_grid = 0;
      const bool ok = ars_step_sched(x, A.data(), B.data(), work.data(), 1, d, nullptr, nullptr) == ARS_OK;
      if (!ok || (int)last_grid > simds || (nz <= simds && (int)last_grid != nz)) {
        if (++bad <= 10) std::printf("%d pairs: %u workgroups on %d SIMDs\n", nz, last_grid, simds);
      }
      ars_destroy(x);
    }
  }
  num_cu = 256;
  return bad;
}

// Tuning a 2D step whose untuned launch is the fastest leaves that launch, for
// the context that was tuned and for one that finds it in the cache.
int tuned_2d(const char* cache) {
  int bad = 0;
  for (auto [nx, nz] : {std::pair{512, 256}, {60, 3000}, {64, 32}, {1024, 1024}}) {
    const ars_config cfg = rb2d(nx, nz);
    std::vector<double> work(8192), A, B;
    double d = 1e-3;
    unsigned grid[3];
    for (int k = 0; k < 3; ++k) {  // untuned, tuned, from the cache
      ars_ctx* x = nullptr;
      if (ars_create(&cfg, &x) != ARS_OK) return 1;
      work.resize(std::max(work.size(), ars_workspace_bytes(x) / 8 + 1));
      A.resize(ars_state_len(x));
      B.resize(A.size());
      if (ars_workspace_init(x, work.data(), nullptr) != ARS_OK) return 1;
      ars_tune_result r{};
      if (k && (ars_autotune(x, A.data(), work.data(), 2, cache, nullptr, &r) != ARS_OK || r.from_cache != (k == 2)))
        ++bad;
      if (ars_step_sched(x, A.data(), B.data(), work.data(), 1, &d, nullptr, nullptr) != ARS_OK) return 1;
      grid[k] = last_grid;
      if (k == 0) best_grid = last_grid;
      ars_destroy(x);
    }
    if (grid[1] != grid[0] || grid[2] != grid[0]) {
      ++bad;
      std::printf("%d x %d: %u workgroups untuned, %u tuned, %u from the cache\n", nx, nz, grid[0], grid[1], grid[2]);
    }
  }
  return bad;
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  int bad = 1;
  if (what == "failed_step") bad = failed_step();
  if (what == "batch_tiling") bad = batch_tiling();
  if (what == "shares") bad = shares();
  if (what == "placement") bad = placement();
  if (what == "one_wave") bad = one_wave();
  if (what == "tuned_2d" && argc > 2) bad = tuned_2d(argv[2]);
  std::printf(bad ? "FAILED %d\n" : "ok\n", bad);
  return bad ? 1 : 0;
}
