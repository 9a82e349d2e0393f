// The host side of the C ABI (mhd_api.hip) in a program of its own, with the
// HIP runtime and the kernel launches replaced by stand-ins that move no data
// to a device.  One command per run; test_host_api.py reads what it prints.
#include "../paper_2604_12672_amd/csrc/mhd_api.hip"

#include <map>

namespace {
// the k-th call from now of a kind that fails (0: none)
long fail_malloc = 0, fail_copy = 0, fail_sync = 0;
long fail_new = 0;
bool fails(long &k) { return k > 0 && --k == 0; }
// device allocations of up to 1 MB hold what is copied into them; the others
// are an address only
std::map<void *, size_t> held;
long live = 0;
hipError_t last_error = hipSuccess;  // as the runtime keeps it until it is read
long missing = 0;  // null buffers of diffusion launches
}  // namespace

void *operator new(size_t n) {
  if (fails(fail_new)) throw std::bad_alloc();
  if (void *p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" {
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "success" : "failure"; }
hipError_t hipGetLastError() {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}
hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipMalloc(void **p, size_t bytes) {
  static size_t next = 4096;
  *p = nullptr;
  if (fails(fail_malloc)) return last_error = hipErrorOutOfMemory;
  *p = bytes <= 1 << 20 ? std::calloc(bytes, 1) : reinterpret_cast<void *>(next += 4096);
  const long k = fail_new;  // not of the map's own
  fail_new = 0;
  if (bytes <= 1 << 20) held[*p] = bytes;
  fail_new = k;
  ++live;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  if (p) --live;
  if (held.erase(p)) std::free(p);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t bytes, hipMemcpyKind kind, hipStream_t) {
  if (fails(fail_copy)) return hipErrorUnknown;
  if (kind == hipMemcpyHostToDevice && held.count(dst)) {
    if (held[dst] < bytes) std::abort();
    std::memcpy(dst, src, bytes);
  }
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return fails(fail_sync) ? hipErrorUnknown : hipSuccess; }
}

namespace mhd {
// as the launch bounds and the LDS of the stage kernel leave them
int stage_blocks_per_cu(const Ctx &c) { return c.d.precision == MHD_PREC_SPLIT ? 2 : 1; }
int species_segment(const Ctx &) { return 1; }
int shock_flag_segment(const Ctx &) { return 1; }
size_t mlp_bytes() { return 17632; }
hipError_t noalloc_setup(int) { return hipSuccess; }
hipError_t launch_stage(const Ctx &, const StagePtrs &, double, double, double, double) {
  return hipSuccess;
}
hipError_t launch_signal_speed(const Ctx &, const double *, const double *, const double *,
                               const double *, const double *, double, double *, double *,
                               double *) {
  return hipSuccess;
}
hipError_t launch_init_temperature(const Ctx &, const double *, const double *, const double *,
                                   const double *, const double *, double *) {
  return hipSuccess;
}
hipError_t launch_diagnostics(const Ctx &, const double *, const double *, const double *,
                              const double *, double *) {
  return hipSuccess;
}
hipError_t launch_zero_walls(const Ctx &, double *) { return hipSuccess; }
hipError_t launch_mlp_guess(const Ctx &, const double *, const double *, const double *,
                            const double *, double *, double *, bool, unsigned long long *) {
  return hipSuccess;
}
hipError_t launch_diff_init(const Ctx &, const double *, const double *, const double *,
                            const double *, const double *) {
  return hipSuccess;
}
hipError_t launch_diff_stage(const Ctx &c, const double *, const double *Ta, const double *chia,
                             const double *y0, const double *y1, const double *y2, double *yn,
                             double *Tb, double *chib, int, int, double, double, double, double,
                             double) {
  for (const void *p : {(const void *)Ta, (const void *)chia, (const void *)y0, (const void *)y1,
                        (const void *)y2, (const void *)yn, (const void *)Tb, (const void *)chib,
                        (const void *)c.diff.M0, (const void *)c.diff.cv0})
    missing += !p;
  return hipGetLastError();  // as every launch does
}
hipError_t launch_diff_finish(const Ctx &, double *, const double *, const double *, int,
                              double *) {
  return hipSuccess;
}
hipError_t launch_parabolic_dt(const Ctx &, const double *, const double *, const double *,
                               const double *, const double *, double *, bool) {
  return hipSuccess;
}
hipError_t launch_shock_pressure(const Ctx &, const double *, const double *, const double *,
                                 const double *, const double *, int) {
  return hipSuccess;
}
hipError_t launch_shock_flags(const Ctx &) { return hipSuccess; }
hipError_t launch_species(const Ctx &, const double *, const double *, const double *, double *,
                          double, double, double, double, const double *, const uint8_t *) {
  return hipSuccess;
}
hipError_t launch_eos_solve(const Ctx &, const double *, const double *, const double *,
                            long long, double *, double *, bool) {
  return hipSuccess;
}
hipError_t launch_math_check(hipStream_t, const double *, double *, long long) {
  return hipSuccess;
}
}  // namespace mhd

namespace {

mhd_grid_desc desc(long nx, long ny, long nz, int precision, int eos) {
  mhd_grid_desc d;
  std::memset(&d, 0, sizeof(d));
  d.nx = (int)nx;
  d.ny = (int)ny;
  d.nz = (int)nz;
  for (int a = 0; a < 3; ++a) d.hi[a] = 1.0;
  d.eos = eos;
  d.gamma = 5.0 / 3.0;
  d.mu = d.rgas = d.arad = 1.0;
  d.rk_order = 2;
  d.precision = precision;
  d.newton_tol = 1e-11;
  d.newton_maxit = 50;
  d.mach_cut = 0.6;
  return d;
}

mhd_ctx *grid(long nx, long ny, long nz, int precision) {
  const mhd_grid_desc d = desc(nx, ny, nz, precision, MHD_EOS_IDEAL);
  mhd_ctx *h = nullptr;
  if (mhd_init_grid(&d, nullptr, &h) != MHD_OK) {
    std::printf("init failed: %s\n", mhd_last_error(nullptr));
    std::exit(1);
  }
  return h;
}

// split nx ny nz precision: the stage kernel's work split
int split(char **v) {
  mhd_ctx *h = grid(std::atol(v[0]), std::atol(v[1]), std::atol(v[2]), std::atoi(v[3]));
  std::printf("%d %d %d %d\n", h->c.stage_full, h->c.stage_share, h->c.zseg, h->c.stage_blocks);
  return mhd_destroy(h);
}

// segment tiles nz slots extra: planes per segment of the other marches
int segment(char **v) {
  std::printf("%d\n", mhd::segment_planes(std::atol(v[0]), std::atoi(v[1]), std::atol(v[2]),
                                          std::atoi(v[3])));
  return 0;
}

// dsegment nx ny nz: planes per block of the diffusion stage kernel
int dsegment(char **v) {
  mhd::Phys ph{};
  ph.nx = std::atoi(v[0]);
  ph.ny = std::atoi(v[1]);
  ph.nz = std::atoi(v[2]);
  std::printf("%d\n", mhd::diff_segment(ph, 256));
  return 0;
}

// A call that fails at its k-th `what`, for every k until none is left: the
// sources and the background on the device are those of before the call, also
// after the next successful call has uploaded them again.
int sources(char **v) {
  const std::string what = v[0];
  long &counter = what == "malloc" ? fail_malloc : what == "copy" ? fail_copy : fail_sync;
  const int nz = 4;
  const double heat1[nz] = {1, 2, 3, 4}, heat2[nz] = {5, 6, 7, 8};
  double bg1[4 * nz], bg2[4 * nz], mode[7] = {1, 0, 0, 0.1, 0.2, 0.3, 0.4};
  for (int i = 0; i < 4 * nz; ++i) {
    bg1[i] = 10 + i;
    bg2[i] = 50 + i;
  }
  long failed = 0, wrong = 0;
  for (int call = 0; call < 2; ++call) {
    for (long k = 1;; ++k) {
      mhd_ctx *h = grid(8, 6, nz, MHD_PREC_FP64);
      const double *table = h->c.table;
      auto differs = [&](const double *heat, const double *bg) {
        for (int z = 0; z < nz; ++z) {
          if (table[z * mhd::TAB_N + 4] != heat[z]) return true;
          for (int f = 0; f < 4; ++f)
            if (table[z * mhd::TAB_N + f] != bg[f * nz + z] ||
                table[z * mhd::TAB_N + mhd::TAB_FACE + f] != bg[f * nz + z])
              return true;
        }
        return false;
      };
      if (mhd_set_background(h, bg1, bg1) || mhd_set_sources(h, heat1, nullptr, 0)) return 1;
      const long before = live;
      counter = k;
      const int rc = call ? mhd_set_background(h, bg2, bg2) : mhd_set_sources(h, heat2, mode, 1);
      const bool reached = counter == 0;
      counter = 0;
      if (!reached) {
        wrong += rc != MHD_OK || differs(call ? heat1 : heat2, call ? bg2 : bg1);
        mhd_destroy(h);
        break;
      }
      ++failed;
      wrong += rc == MHD_OK || h->c.fcoef || live != before;
      // the call that is not the failed one, with its values of before
      if (call ? mhd_set_sources(h, heat1, nullptr, 0) : mhd_set_background(h, bg1, bg1)) return 1;
      wrong += differs(heat1, bg1);
      mhd_destroy(h);
    }
  }
  std::printf("%ld %ld %ld\n", failed, wrong, live);
  return 0;
}

// Every host allocation of a call fails in turn: calls, allocations, calls that
// threw, calls that did not report it, device buffers left.
int host_memory(char **) {
  const int nz = 4;
  const double heat[nz] = {1, 2, 3, 4}, bg[4 * nz] = {0.0}, mode[7] = {1, 0, 0, 0.1, 0.2, 0.3, 0.4};
  const std::vector<float> w1(128, 0.5f), b(64, 0.5f);
  const std::vector<uint16_t> w2(64 * 64, 0), w3(64, 0);
  const double norm[6] = {0, 1, 0, 1, 0, 1};
  long reached = 0, thrown = 0, missed = 0;
  const int calls = 5;
  for (int call = 0; call < calls; ++call) {
    for (long k = 1;; ++k) {
      mhd_ctx *h = nullptr;
      mhd_grid_desc d = desc(8, 6, nz, call == 2 ? MHD_PREC_SPLIT : MHD_PREC_FP64, MHD_EOS_GASRAD);
      if (call == 4) d.eos_guess = MHD_GUESS_MLP;
      if (call && mhd_init_grid(&d, nullptr, &h)) return 1;
      int rc = MHD_OK;
      fail_new = k;
      try {
        rc = call == 0   ? mhd_init_grid(&d, nullptr, &h)
             : call == 1 ? mhd_set_background(h, bg, bg)
             : call <= 3 ? mhd_set_sources(h, heat, mode, 1)
                         : mhd_set_eos_mlp(h, w1.data(), b.data(), w2.data(), b.data(), w3.data(),
                                           0.5f, norm);
      } catch (const std::bad_alloc &) {
        ++thrown;
      }
      const bool hit = fail_new == 0;
      fail_new = 0;
      reached += hit;
      missed += hit ? rc == MHD_OK : rc != MHD_OK;
      mhd_destroy(h);
      if (!hit) break;
    }
  }
  std::printf("%d %ld %ld %ld %ld\n", calls, reached, thrown, missed, live);
  return 0;
}

// A grid that could not be created, then a super step whose k-th device allocation fails, then one that succeeds: super
// steps failed, launches with a buffer missing, second ones failed
// (or the next launch after the grid), device buffers left.
int diffusion(char **) {
  long failed = 0, refused = 0, live_after = 0;
  const mhd_grid_desc d = desc(8, 6, 4, MHD_PREC_FP64, MHD_EOS_GASRAD);
  mhd_ctx *h = nullptr;
  fail_malloc = 5;
  if (mhd_init_grid(&d, nullptr, &h) != MHD_ERR_HIP) return 1;
  refused += hipGetLastError() != hipSuccess;
  for (long k = 1;; ++k) {
    std::vector<double> u(5 * 8 * 6 * 4, 1.0);
    if (mhd_init_grid(&d, nullptr, &h) ||
        mhd_set_state(h, u.data(), u.data(), u.data(), u.data(), nullptr, MHD_HOST) ||
        mhd_set_opacity(h, 1.0, 0.0, 0.0, 1.0))
      return 1;
    fail_malloc = k;
    const int rc = mhd_diffuse(h, 1.0, 4, MHD_DIFF_EINT, nullptr);
    const bool hit = fail_malloc == 0;
    fail_malloc = 0;
    failed += hit && rc != MHD_OK;
    refused += mhd_diffuse(h, 1.0, 4, MHD_DIFF_EINT, nullptr) != MHD_OK;
    mhd_destroy(h);
    live_after = live;
    if (!hit) break;
  }
  std::printf("%ld %ld %ld %ld\n", failed, missing, refused, live_after);
  return 0;
}

}  // namespace

int main(int argc, char **argv) {
  const std::map<std::string, std::pair<int, int (*)(char **)>> commands = {
      {"split", {4, split}}, {"segment", {4, segment}}, {"dsegment", {3, dsegment}},
      {"sources", {1, sources}}, {"host_memory", {0, host_memory}},
      {"diffusion", {0, diffusion}}};
  const auto it = argc > 1 ? commands.find(argv[1]) : commands.end();
  if (it == commands.end() || argc - 2 != it->second.first) return 2;
  return it->second.second(argv + 2);
}
