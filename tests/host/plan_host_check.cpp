// Host tests of the plan code behind the C ABI, over the HIP runtime of fake_hip.hpp: one scenario per run,
// named on the command line; exits with 0 if it holds, else prints what does not.
#include <cmath>
#include <functional>

#include "../../include/fockmi.h"
#include "fake_hip.hpp"

namespace {

int faults = 0;
#define CHECK(c)                                                        \
  do {                                                                  \
    if (!(c)) {                                                         \
      std::printf("line %d: %s does not hold\n", __LINE__, #c);        \
      ++faults;                                                         \
    }                                                                   \
  } while (0)
#define OK(call)                                                                      \
  do {                                                                                \
    const fock_status s_ = (call);                                                    \
    if (s_ != FOCK_OK) {                                                              \
      std::printf("line %d: status %d (%s)\n", __LINE__, (int)s_, fock_last_error()); \
      ++faults;                                                                       \
    }                                                                                 \
  } while (0)

struct CellSpec {
  int n[3], nk, nb;
};

struct TestPlan {
  fockmi_plan h = nullptr;
  std::vector<CellSpec> cells;
  TestPlan(fock_prec prec, std::vector<CellSpec> specs, const char* tune = nullptr) : cells(std::move(specs)) {
    std::vector<std::vector<double>> kp;
    std::vector<fock_cell_desc> d;
    for (const CellSpec& c : cells) {
      kp.emplace_back(3 * c.nk, 0.0);
      for (int k = 0; k < c.nk; ++k) kp.back()[3 * k] = 0.01 * k;
    }
    for (size_t i = 0; i < cells.size(); ++i) {
      fock_cell_desc x{};
      for (int a = 0; a < 3; ++a) {
        x.n[a] = cells[i].n[a];
        x.a[a][a] = 10.26;
      }
      x.nk = cells[i].nk;
      x.kpts = kp[i].data();
      x.nb = cells[i].nb;
      x.omega = 0.11;
      x.gs = 2.0;
      d.push_back(x);
    }
    OK(fock_plan_create(d.data(), (int)d.size(), prec, tune, &h));
  }
  ~TestPlan() { fock_plan_destroy(h); }
  size_t bytes(int cell, int nf) const {
    const CellSpec& c = cells[cell];
    return (size_t)16 * c.n[0] * c.n[1] * c.n[2] * c.nk * nf;
  }
  void* fields(int cell = 0, int nf = 0) const { return fake::user(bytes(cell, nf ? nf : cells[cell].nb)); }
};

CellSpec cube(int n, int nk, int nb) { return CellSpec{{n, n, n}, nk, nb}; }

// the plan's allocations at this moment, none of which may be freed by what follows
struct Held {
  std::map<uintptr_t, size_t> live = fake::st().live;
  size_t lost() const {
    size_t n = 0;
    for (auto& a : live) n += !fake::st().live.count(a.first);
    return n;
  }
};

// A graph captured from a plan refers to the plan's buffers: they stay where they are while eager
// calls of other kinds (an adjoint, more targets, a larger cell) make the plan grow them, and the
// plan frees everything when it is destroyed.
void captured_buffers_stay() {
  struct Form {
    fock_prec prec;
    std::vector<CellSpec> cells;
  };
  const std::vector<Form> forms = {{FOCK_FP32_COMP, {cube(24, 64, 16), cube(24, 64, 20)}},
                                   {FOCK_FP64_FUSED, {cube(24, 64, 16), cube(24, 64, 20)}},
                                   {FOCK_FP64_FUSED, {cube(20, 27, 12), cube(20, 64, 16)}},
                                   {FOCK_FP64, {cube(16, 8, 4), cube(16, 64, 4)}},
                                   {FOCK_FP64, {cube(32, 8, 16), cube(32, 27, 16)}},
                                   {FOCK_FP32_COMP, {cube(32, 27, 16), cube(32, 64, 16)}}};
  for (const Form& f : forms) {
    const size_t before = fake::st().live.size();
    {
      TestPlan p(f.prec, f.cells);
      const hipStream_t q = fake::stream(0);
      void *u = p.fields(), *out = p.fields(), *psi = p.fields();
      OK(fock_apply(p.h, 0, u, u, p.cells[0].nb, out, q));
      OK(fock_orthonormalize(p.h, 0, psi, q));
      fake::st().capturing.insert(q);
      OK(fock_apply(p.h, 0, u, u, p.cells[0].nb, out, q));
      OK(fock_orthonormalize(p.h, 0, psi, q));
      fake::st().capturing.clear();
      const Held held;
      const int nphi = p.cells[0].nb;
      void *phi = p.fields(0, nphi), *g = p.fields(0, nphi), *gu = p.fields(), *gp = p.fields(0, nphi);
      OK(fock_vjp(p.h, 0, u, phi, nphi, g, gu, gp, q));
      void *many = p.fields(0, 40), *mout = p.fields(0, 40);
      OK(fock_apply(p.h, 0, u, many, 40, mout, q));
      void *u1 = p.fields(1), *out1 = p.fields(1);
      OK(fock_apply(p.h, 1, u1, u1, p.cells[1].nb, out1, q));
      OK(fock_orthonormalize(p.h, 1, u1, q));
      double e = 0;
      OK(fock_energy(p.h, 1, u1, &e, nullptr, q));
      CHECK(held.lost() == 0);
      CHECK(fake::st().bad_mallocs == 0);
    }
    CHECK(fake::st().live.size() == before);
  }
}

// Without a capture growth frees what it replaces.
void growth_frees() {
  TestPlan p(FOCK_FP32_COMP, {cube(24, 64, 16)});
  const hipStream_t q = fake::stream(0);
  void *u = p.fields(), *out = p.fields();
  OK(fock_apply(p.h, 0, u, u, 16, out, q));
  const size_t n = fake::st().live.size();
  void *phi = p.fields(), *g = p.fields(), *gu = p.fields(), *gp = p.fields();
  const size_t freed = fake::st().freed.size();
  OK(fock_vjp(p.h, 0, u, phi, 16, g, gu, gp, q));
  CHECK(fake::st().freed.size() > freed);
  CHECK(fake::st().live.size() <= n + 8);
}

const std::map<std::string, std::function<void()>> scenarios = {
    {"captured_buffers_stay", captured_buffers_stay},
    {"growth_frees", growth_frees},
};

}  // namespace

int main(int argc, char** argv) {
  if (argc < 2) {
    for (auto& s : scenarios) std::printf("%s\n", s.first.c_str());
    return 0;
  }
  auto it = scenarios.find(argv[1]);
  if (it == scenarios.end()) {
    std::printf("no scenario %s\n", argv[1]);
    return 2;
  }
  it->second();
  return faults ? 1 : 0;
}
