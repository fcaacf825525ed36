// Runs one PCG system three times with the resident kernel, on the same exchange words and with
// growing tags: as rgp_pcg_solve does, then with the given limits, then as at first.  Prints what the
// runs gave, for tests/test_gpu_resident_limits.py.  The limits are fields of the kernel's argument
// block that the host sets; whatever they are, every workgroup ends by itself.
//
//   resident_driver n0 n1 n2 pe f32|f64 maxit rtol spins most grow cus
//
// spins, most, grow: the argument block's (most 0: every workgroup).  cus: the second run's stream has
// the lowest `cus` of each 32 compute units only (0: all), so that not all workgroups are resident.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "rgp_launch.hpp"

using namespace rgp;

#define CHECK(call)                                                                  \
  do {                                                                               \
    const hipError_t e_ = (call);                                                    \
    if (e_ != hipSuccess) {                                                          \
      std::fprintf(stderr, "%s: %s\n", #call, hipGetErrorString(e_));                \
      return 2;                                                                      \
    }                                                                                \
  } while (0)

namespace {

struct Result {
  std::vector<unsigned char> x;
  int32_t iters;
  double relres;
  float ms;
};

struct Limits {
  uint32_t spins;
  int most, grow, cus;
};

template <typename T>
int nans(const Result& r) {
  const T* x = reinterpret_cast<const T*>(r.x.data());
  int n = 0;
  for (size_t i = 0; i < r.x.size() / sizeof(T); ++i) n += std::isnan(x[i]);
  return n;
}

template <typename T>
int run(const int64_t m[3], int pe, DType real, int maxit, double rtol, const Limits& lim) {
  const double h[3] = {1.0, 1.0, 1.0};
  const Geom g = make_geom(m, pe, h);
  const ResPlan R = plan_resident(g, real);
  if (!R.ok) {
    std::fprintf(stderr, "no resident variant\n");
    return 2;
  }
  const size_t nb = (size_t)g.nnode * sizeof(T), pad = (nb + 255) / 256 * 256;
  // a diagonally dominant system
  uint64_t seed = 12345;
  auto rnd = [&]() {
    seed = seed * 6364136223846793005ull + 1442695040888963407ull;
    return (double)(seed >> 11) / 9007199254740992.0;
  };
  std::vector<T> host[3];
  for (auto& v : host) v.resize((size_t)g.nnode);
  for (int64_t i = 0; i < g.nnode; ++i) {
    host[0][i] = (T)(2000.0 + 500.0 * rnd());
    host[1][i] = (T)(-300.0 - 50.0 * rnd());
    host[2][i] = (T)(rnd() - 0.5);
  }
  // diag, off, rhs, x, four vectors of words, two spare ones; sums and control words; outputs
  unsigned char* vec = nullptr;
  CHECK(hipMalloc(&vec, 10 * pad));
  unsigned long long* part = nullptr;
  CHECK(hipMalloc(&part, (size_t)kResSyncWords * 8));
  unsigned char* out = nullptr;
  const size_t so = (sizeof(State) + 255) / 256 * 256;
  CHECK(hipMalloc(&out, so + 256));
  for (int k = 0; k < 3; ++k)
    CHECK(hipMemcpy(vec + k * pad, host[k].data(), nb, hipMemcpyHostToDevice));
  CHECK(hipMemset(out, 0, so + 256));
  hipStream_t s, narrow = nullptr;
  CHECK(hipStreamCreate(&s));
  if (lim.cus > 0) {
    uint32_t mask[8];
    for (uint32_t& w : mask) w = lim.cus >= 32 ? 0xffffffffu : (1u << lim.cus) - 1u;
    CHECK(hipExtStreamCreateWithCUMask(&narrow, 8, mask));
  }
  hipEvent_t e0, e1;
  CHECK(hipEventCreate(&e0));
  CHECK(hipEventCreate(&e1));
  ResArgs a = make_res_args(g, R, 300.0);
  a.diag = vec;
  a.off = vec + pad;
  a.rhs = vec + 2 * pad;
  a.x = vec + 3 * pad;
  a.words = reinterpret_cast<unsigned long long*>(vec + 4 * pad);
  a.part = part;
  a.sync = part + kResSumWords;
  a.spare_r = vec + 8 * pad;
  a.spare_p = vec + 9 * pad;
  a.rhs_sign = 1.0;
  a.rtol = rtol;
  a.st = reinterpret_cast<State*>(out);
  a.iters_out = reinterpret_cast<int32_t*>(out + so);
  a.relres_out = reinterpret_cast<double*>(out + so + 64);
  a.maxit = maxit;
  a.tag = 1;
  CHECK(launch_clear_words(a.words, g.nnode, real, a.part, s));
  Result res[3];
  for (int k = 0; k < 3; ++k) {
    ResArgs b = a;
    if (k == 1) {
      b.spins = lim.spins;
      if (lim.most > 0) b.most = lim.most;
      b.grow = lim.grow;
    }
    const hipStream_t on = k == 1 && narrow ? narrow : s;
    CHECK(hipMemset(a.x, 0x7f, nb));   // (no value of a solve)
    CHECK(hipDeviceSynchronize());
    CHECK(hipEventRecord(e0, on));
    CHECK(launch_pcg_resident_one(b, R, real, on));
    CHECK(hipEventRecord(e1, on));
    CHECK(hipStreamSynchronize(on));
    CHECK(hipEventElapsedTime(&res[k].ms, e0, e1));
    a.tag += (uint32_t)maxit + 1u;
    res[k].x.resize(nb);
    CHECK(hipMemcpy(res[k].x.data(), a.x, nb, hipMemcpyDeviceToHost));
    CHECK(hipMemcpy(&res[k].iters, a.iters_out, sizeof(int32_t), hipMemcpyDeviceToHost));
    CHECK(hipMemcpy(&res[k].relres, a.relres_out, sizeof(double), hipMemcpyDeviceToHost));
  }
  std::printf("{\"units\": %d, \"tier\": %d, \"role\": %d, \"nodes\": %lld, \"runs\": [", a.units,
              R.tier, a.role, (long long)g.nnode);
  for (int k = 0; k < 3; ++k)
    std::printf("%s{\"equal\": %s, \"nans\": %d, \"iters\": %d, \"relres\": \"%.17g\", \"ms\": %.3f}", k ? ", " : "",
                res[k].x == res[0].x ? "true" : "false", nans<T>(res[k]), (int)res[k].iters,
                res[k].relres, res[k].ms);
  std::printf("]}\n");
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 12) {
    std::fprintf(stderr, "usage: resident_driver n0 n1 n2 pe f32|f64 maxit rtol spins most grow cus\n");
    return 2;
  }
  const int64_t m[3] = {std::atoll(argv[1]), std::atoll(argv[2]), std::atoll(argv[3])};
  const int pe = std::atoi(argv[4]), maxit = std::atoi(argv[6]);
  const double rtol = std::atof(argv[7]);
  const Limits lim{(uint32_t)std::strtoul(argv[8], nullptr, 10), std::atoi(argv[9]),
                   std::atoi(argv[10]), std::atoi(argv[11])};
  const bool f64 = std::strcmp(argv[5], "f64") == 0;
  return f64 ? run<double>(m, pe, DType::F64, maxit, rtol, lim)
             : run<float>(m, pe, DType::F32, maxit, rtol, lim);
}
