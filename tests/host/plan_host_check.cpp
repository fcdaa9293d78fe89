// Host tests of the plan code behind the C ABI, over the HIP runtime of fake_hip.hpp: one scenario per run,
// named on the command line; exits with 0 if it holds, else prints what does not.
#include <cmath>
#include <functional>
#include <thread>

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

// A graph captured from a plan refers to the plan's buffers (here all that there are): they stay where they are while eager
// calls of other kinds (an adjoint, more targets, a larger cell) make the plan grow them, and the
// plan frees everything when it is destroyed.
void captured_buffers_stay() {
  struct Form {
    fock_prec prec;
    std::vector<CellSpec> cells;
  };
  const std::vector<Form> forms = {{FOCK_FP32_COMP, {cube(24, 64, 16), cube(24, 64, 20)}},
                                   {FOCK_FP64_FUSED, {cube(24, 64, 16), cube(24, 64, 20)}},
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

// Calls that the header lets run on any streams, and the others that use the same scratch: of each two the
// first records an event behind its last launch, and the second's stream waits for it before its first.
void streams_in_order() {
  for (int n : {16, 20}) {
    TestPlan p(FOCK_FP64_FUSED, {cube(n, 8, 4)});
    void *u = p.fields(), *out = p.fields(), *psi = p.fields(), *phi = p.fields(), *g = p.fields(), *gu = p.fields();
    const double a[3] = {0.0, 0.0, 0.01};
    double e = 0, ga[3];
    using Call = std::function<void(hipStream_t)>;
    const std::vector<Call> calls = {
        [&](hipStream_t q) { OK(fock_apply(p.h, 0, u, u, 4, out, q)); },
        [&](hipStream_t q) { OK(fock_apply(p.h, 0, u, phi, 4, out, q)); },
        [&](hipStream_t q) { OK(fock_apply_krange(p.h, 0, u, 1, 2, phi, 4, out, q)); },
        [&](hipStream_t q) { OK(fock_energy_vjp(p.h, 0, u, 1.0, gu, q)); },
        [&](hipStream_t q) { OK(fock_vjp(p.h, 0, u, phi, 4, g, gu, out, q)); },
        [&](hipStream_t q) { OK(fock_orthonormalize(p.h, 0, psi, q)); },
        [&](hipStream_t q) { OK(fock_energy(p.h, 0, u, &e, nullptr, q)); },
        [&](hipStream_t q) { OK(taylor_step(p.h, 0, psi, nullptr, a, 0.01, 0.25, 2, nullptr, q)); },
        [&](hipStream_t q) { OK(taylor_step_vjp(p.h, 0, psi, nullptr, a, 0.01, 0.25, 2, g, gu, ga, q)); },
        [&](hipStream_t q) { OK(taylor_energy(p.h, 0, psi, nullptr, a, 0.25, &e, gu, ga, q)); }};
    // the calls' kernels that use the shared scratch
    auto shared = [](const fake::Op& o) {
      return o.kind == fake::Op::Launch && (o.name.find("pair_w") != std::string::npos ||
                                            o.name.find("wsum") != std::string::npos ||
                                            o.name.find("mirror_add") != std::string::npos ||
                                            o.name.find("gram") != std::string::npos);
    };
    for (const Call& first : calls)
      for (const Call& second : calls) {
        std::vector<fake::Op>& ops = fake::st().ops;
        ops.clear();
        first(fake::stream(1));
        const size_t cut = ops.size();
        second(fake::stream(2));
        size_t last = cut, next = ops.size(), recorded = 0, waited = ops.size();
        void* ev = nullptr;
        for (size_t i = 0; i < cut; ++i)
          if (shared(ops[i])) last = i;
        for (size_t i = last; i < cut; ++i)
          if (ops[i].kind == fake::Op::Record && ops[i].stream == fake::stream(1)) recorded = i, ev = ops[i].event;
        for (size_t i = ops.size(); i-- > cut;) {
          if (shared(ops[i])) next = i;
          if (ops[i].kind == fake::Op::Wait && ops[i].stream == fake::stream(2) && ops[i].event == ev) waited = i;
        }
        CHECK(last < cut && ev && recorded > last && waited < next && next < ops.size());
      }
  }
}

// Two threads on one plan: the work of one call is enqueued whole before another call's begins.
void threads_one_at_a_time() {
  TestPlan p(FOCK_FP64_FUSED, {cube(16, 8, 4)});
  void* u = p.fields();
  void* outs[2] = {p.fields(), p.fields()};
  void* psis[2] = {p.fields(), p.fields()};
  auto run = [&](int id) {
    for (int i = 0; i < 200; ++i) {
      OK(fock_apply(p.h, 0, u, u, 4, outs[id], fake::stream(id + 1)));
      OK(fock_orthonormalize(p.h, 0, psis[id], fake::stream(id + 1)));
    }
  };
  fake::st().ops.clear();
  std::thread a(run, 0), b(run, 1);
  a.join();
  b.join();
  // a call ends with its record: until then every operation is of one thread
  long owner = 0;
  size_t mixed = 0, records = 0;
  for (const fake::Op& o : fake::st().ops) {
    if (owner && o.thread != owner) ++mixed;
    owner = o.kind == fake::Op::Record ? 0 : o.thread;
    records += o.kind == fake::Op::Record;
  }
  CHECK(mixed == 0);
  CHECK(records == 800);
}

// Captured calls that need no plan memory use none, also on a plan whose buffers are there: their graphs
// may replay on several streams at once.
void captures_without_plan_memory() {
  for (int n : {16, 20}) {
    TestPlan p(FOCK_FP64_FUSED, {cube(n, 8, 4)});
    const hipStream_t q = fake::stream(0);
    void *u = p.fields(), *out = p.fields(), *psi = p.fields(), *phi = p.fields(), *g = p.fields(), *gu = p.fields();
    auto calls = [&] {
      OK(fock_apply(p.h, 0, u, u, 4, out, q));
      OK(fock_apply(p.h, 0, u, phi, 4, out, q));
      OK(fock_apply_krange(p.h, 0, u, 1, 2, phi, 4, out, q));
      OK(fock_vjp(p.h, 0, u, phi, 4, g, gu, out, q));
      OK(fock_energy_vjp(p.h, 0, u, 1.0, gu, q));
      OK(fock_orthonormalize(p.h, 0, psi, q));
    };
    calls();
    CHECK(fake::launches("pair_w") > 0 && fake::launches("gram") > 0);
    const size_t from = fake::st().ops.size();
    fake::st().capturing.insert(q);
    calls();
    fake::st().capturing.clear();
    CHECK(fake::launches("fused64", from) + fake::launches("mgs", from) == fake::launches("", from));
    CHECK(fake::st().bad_mallocs == 0);
    fake::st().ops.clear();
  }
}

// The first sum on a new plan allocates once for the pair form's scratch, in every precision and direction, and
// the same sum again allocates nothing.
void first_sum_allocates_once() {
  struct Form {
    fock_prec prec;
    CellSpec cell;
    size_t shadows;  // complex64 copies, each its own buffer
  };
  for (const Form& f : {Form{FOCK_FP64, cube(16, 8, 4), 0}, Form{FOCK_FP64_FUSED, cube(16, 8, 4), 0},
                        Form{FOCK_FP64, cube(32, 8, 4), 0}, Form{FOCK_FP64, CellSpec{{16, 20, 24}, 12, 6}, 0},
                        Form{FOCK_FP32_COMP, cube(16, 8, 4), 1}}) {
    TestPlan p(f.prec, {f.cell});
    void *u = p.fields(), *out = p.fields();
    const size_t before = fake::st().mallocs;
    OK(fock_apply(p.h, 0, u, u, f.cell.nb, out, fake::stream(0)));
    CHECK(fake::st().mallocs == before + 1 + f.shadows);
    OK(fock_apply(p.h, 0, u, u, f.cell.nb, out, fake::stream(0)));
    CHECK(fake::st().mallocs == before + 1 + f.shadows);
  }
}

// A plan with a tuning cache and no room for the pair form's scratch measures the other forms: 5,000 targets of
// 32^3 under a cap of 4 GiB (mirror sums of 5,000 MiB with rows of 128 targets, 2,500 with rows of 64, which
// then run), and a device whose memory is full but for what the forms that sum on the CU need.
void tuned_call_without_room() {
  const std::string path = std::string(getenv("TMPDIR") ? getenv("TMPDIR") : "/tmp") + "/fockmi_tune_check.json";
  auto launched = [] { return fake::launches("pair_w") > 0; };
  {
    remove(path.c_str());
    setenv("FOCKMI_WORKSPACE_CAP", std::to_string(size_t(4) << 30).c_str(), 1);
    TestPlan p(FOCK_FP32_COMP, {cube(32, 250, 20)}, path.c_str());
    unsetenv("FOCKMI_WORKSPACE_CAP");
    const size_t events = fake::st().events.size();
    void *u = p.fields(), *out = p.fields();
    OK(fock_apply(p.h, 0, u, u, 20, out, fake::stream(0)));
    CHECK(launched() && fake::launches("mirror_add") > 0);
    CHECK(fake::st().events.size() == events);
  }
  fake::st().ops.clear();
  {
    remove(path.c_str());
    TestPlan p(FOCK_FP32_COMP, {cube(32, 8, 16)}, path.c_str());
    const size_t events = fake::st().events.size();
    void *u = p.fields(), *phi = p.fields(0, 4), *out = p.fields(0, 4);
    fake::st().limit = fake::st().used() + (size_t(240) << 20);  // what the three forms that sum on the CU take: 217
    OK(fock_apply(p.h, 0, u, phi, 4, out, fake::stream(0)));
    fake::st().limit = ~size_t(0);
    CHECK(!launched() && fake::launches("split32") + fake::launches("fused") > 0);
    CHECK(fake::st().events.size() == events);
  }
  remove(path.c_str());
}

// A plan created with FOCKMI_SPLIT_SYM=0 runs every pair, in every precision and on every grid; without it
// the same calls use the pair symmetry.
void symmetry_switch() {
  struct Form {
    fock_prec prec;
    CellSpec cell;
  };
  for (const Form& f : {Form{FOCK_FP32_COMP, cube(24, 64, 16)}, Form{FOCK_FP32_COMP, cube(32, 8, 16)},
                        Form{FOCK_FP64, cube(16, 8, 4)}, Form{FOCK_FP64, cube(32, 8, 16)},
                        Form{FOCK_FP64, CellSpec{{16, 20, 24}, 12, 6}}, Form{FOCK_FP64_FUSED, cube(20, 27, 12)},
                        Form{FOCK_FP64_FUSED, cube(24, 64, 16)}})
    for (int sym : {0, 1}) {
      if (!sym) setenv("FOCKMI_SPLIT_SYM", "0", 1);
      TestPlan p(f.prec, {f.cell});
      unsetenv("FOCKMI_SPLIT_SYM");
      void *u = p.fields(), *out = p.fields();
      fake::st().ops.clear();
      OK(fock_apply(p.h, 0, u, u, f.cell.nb, out, fake::stream(0)));
      CHECK((fake::launches("mirror_add") > 0) == (sym == 1));
    }
}

// FP32 at 16^3 to 24^3: where the application to u runs every pair, a k-range of u and a copy of u as targets
// run the same kernel (their bits are the application's). Every count of fields up to 1,100.
void same_kernel_for_a_k_range() {
  for (int n : {16, 20, 24})
    for (int nk : {1, 4, 10, 20})
      for (int nb = 1; nb <= 1100 / nk; nb += nk == 1 ? 7 : 1) {
        TestPlan p(FOCK_FP32_COMP, {cube(n, nk, nb)});
        void *u = p.fields(), *v = p.fields(), *out = p.fields();
        auto kernel = [&](const std::function<void()>& call) {
          fake::st().ops.clear();
          call();
          return fake::launches("mirror_add") ? 2 : (fake::launches("pair_w") ? 1 : 0);
        };
        const int full = kernel([&] { OK(fock_apply(p.h, 0, u, u, nb, out, fake::stream(0))); });
        const int copy = kernel([&] { OK(fock_apply(p.h, 0, u, v, nb, out, fake::stream(0))); });
        const int part = nk == 1 ? copy : kernel([&] { OK(fock_apply_krange(p.h, 0, u, 1, nk - 1, v, nb, out, fake::stream(0))); });
        if (copy != part || (full != 2 && full != copy)) {
          std::printf("%d^3, %d x %d fields: u %d, copy %d, k-range %d\n", n, nk, nb, full, copy, part);
          ++faults;
        }
      }
}

// A captured call whose kind of sum the plan has not run runs in the scratch that is there, or without any:
// after a larger sum of another kind in FP64 (with separate targets on grids of every form; at 16^3 one that
// runs the fused kernel), u as targets, few targets and the adjoint.
void captures_use_what_is_there() {
  for (const CellSpec& c : {cube(32, 8, 8), CellSpec{{16, 20, 24}, 12, 6}, cube(16, 64, 16), cube(24, 8, 16)})
    for (int form : {0, 1}) {
      TestPlan p(form ? FOCK_FP64_FUSED : FOCK_FP64, {c});
      const hipStream_t q = fake::stream(0);
      void *u = p.fields(), *out = p.fields(), *phi = p.fields(0, 40), *big = p.fields(0, 40);
      void *g = p.fields(0, 2), *gp = p.fields(0, 2);
      OK(fock_apply(p.h, 0, u, phi, 40, big, q));
      fake::st().bad_mallocs = 0;
      fake::st().capturing.insert(q);
      OK(fock_apply(p.h, 0, u, u, c.nb, out, q));
      OK(fock_apply(p.h, 0, u, phi, 2, big, q));
      OK(fock_vjp(p.h, 0, u, phi, 2, g, out, gp, q));
      fake::st().capturing.clear();
      CHECK(fake::st().bad_mallocs == 0);
    }
}

// FP64 at 24^3 with a workspace cap below the fused kernel's sums (1,024 targets: 216 MiB): the sum runs in
// blocks, as it did with a tuning file that asks for a batch of 64 MiB.
void fused_sums_beyond_the_cap() {
  setenv("FOCKMI_WORKSPACE_CAP", std::to_string(size_t(100) << 20).c_str(), 1);
  TestPlan p(FOCK_FP64, {cube(24, 64, 16)});
  unsetenv("FOCKMI_WORKSPACE_CAP");
  void *u = p.fields(), *phi = p.fields(), *out = p.fields();
  OK(fock_apply(p.h, 0, u, phi, 16, out, fake::stream(0)));
  CHECK(fake::launches("pair_w") > 0 && fake::launches("fused64") == 0);
}

// A sum that is refused for want of memory leaves the profile record readable, and is not in it.
void refused_sum_is_not_profiled() {
  setenv("FOCKMI_WORKSPACE_CAP", "1000", 1);
  TestPlan p(FOCK_FP64, {CellSpec{{16, 20, 24}, 3, 2}});
  unsetenv("FOCKMI_WORKSPACE_CAP");
  void *u = p.fields(), *out = p.fields(), *g = p.fields(), *gp = p.fields();
  OK(fock_profile_enable(p.h, 1));
  CHECK(fock_apply(p.h, 0, u, u, 2, out, fake::stream(0)) == FOCK_ERR_NOMEM);
  CHECK(fock_vjp(p.h, 0, u, u, 2, g, out, gp, fake::stream(0)) == FOCK_ERR_NOMEM);
  double ms = -1;
  long long n = -1;
  OK(fock_profile_read(p.h, &ms, &n, 1));
  CHECK(n == 0 && ms == 0.0);
}

// Without a tuned choice the batched call runs the faster of its forked cells (a captured graph) and the cells
// in sequence through the pair form, by what both took on the device.
void batched_route() {
  struct Set {
    std::vector<CellSpec> cells;
    bool sequence;
  };
  auto many = [](int n, CellSpec c) { return std::vector<CellSpec>(n, c); };
  for (const Set& s : {Set{many(8, cube(16, 8, 16)), false}, Set{many(8, cube(16, 8, 8)), true},
                       Set{many(8, cube(16, 8, 4)), true}, Set{many(4, cube(20, 8, 8)), true},
                       Set{many(8, cube(20, 8, 8)), true}, Set{many(8, cube(24, 4, 8)), true},
                       Set{{cube(16, 64, 16), cube(16, 8, 16)}, false}, Set{{cube(24, 64, 16), cube(16, 1, 1)}, true},
                       Set{{cube(24, 125, 16), cube(20, 64, 12), cube(16, 27, 8)}, true},
                       Set{{cube(16, 8, 8), cube(20, 4, 8), cube(24, 2, 8)}, true},
                       Set{many(8, cube(16, 1, 4)), true}, Set{many(2, cube(16, 216, 16)), false}}) {
    TestPlan p(FOCK_FP32_COMP, s.cells);
    std::vector<const void*> u;
    std::vector<void*> out;
    std::vector<int> np;
    for (size_t i = 0; i < s.cells.size(); ++i) {
      u.push_back(p.fields((int)i));
      out.push_back(p.fields((int)i));
      np.push_back(s.cells[i].nb);
    }
    fake::st().ops.clear();
    OK(fock_apply_batched(p.h, u.data(), u.data(), np.data(), out.data(), fake::stream(0)));
    CHECK((fake::launches("graph") == 0) == s.sequence);
  }
}

// A plan created with the split form's wait limit set runs it at 32^3, with its mirror copies where u is the
// targets.
void wait_limit_runs_the_split_form() {
  setenv("FOCKMI_SPLIT_WAIT_TICKS", "5000000", 1);
  TestPlan p(FOCK_FP32_COMP, {cube(32, 8, 3)});
  unsetenv("FOCKMI_SPLIT_WAIT_TICKS");
  void *u = p.fields(), *phi = p.fields(), *out = p.fields();
  fake::st().ops.clear();
  OK(fock_apply(p.h, 0, u, u, 3, out, fake::stream(0)));
  CHECK(fake::launches("split32_kernel") == 1 && fake::launches("sym_combine") == 1 && fake::launches("pair_w") == 0);
  fake::st().ops.clear();
  OK(fock_apply(p.h, 0, u, phi, 3, out, fake::stream(0)));
  CHECK(fake::launches("split32_kernel") == 1 && fake::launches("sym_combine") == 0 && fake::launches("pair_w") == 0);
}

// What test_gpu_grid_forms.py runs: the fused kernels, by a tuning file in FP32 and by the rule for separate
// targets in FP64, against symmetric pairs with u as targets.
void grid_forms_of_the_device_tests() {
  const std::string path = std::string(getenv("TMPDIR") ? getenv("TMPDIR") : "/tmp") + "/fockmi_grid_forms.json";
  for (const CellSpec& c : {cube(16, 54, 19), cube(20, 28, 19), cube(24, 17, 19)}) {
    FILE* f = fopen(path.c_str(), "w");
    fprintf(f, "{\"gfx950/fp32/fused/n%dx%dx%d/nt%d/ns%d/nb%d/nx%d\": {\"variant\": 0, \"xcd_map\": 1}}\n", c.n[0], c.n[0],
            c.n[0], c.nk, c.nk, c.nb, c.nb);
    fclose(f);
    TestPlan p(FOCK_FP32_COMP, {c}, path.c_str());
    void *u = p.fields(), *out = p.fields();
    fake::st().ops.clear();
    OK(fock_apply(p.h, 0, u, u, c.nb, out, fake::stream(0)));
    CHECK(fake::launches("fused_apply") == 1 && fake::launches("pair_w") == 0);
  }
  remove(path.c_str());
  for (const CellSpec& c : {cube(16, 27, 19), cube(20, 14, 18), cube(24, 8, 32)}) {
    TestPlan p(FOCK_FP64_FUSED, {c});
    void *u = p.fields(), *v = p.fields(), *out = p.fields();
    fake::st().ops.clear();
    OK(fock_apply(p.h, 0, u, v, c.nb, out, fake::stream(0)));
    CHECK(fake::launches("fused64") == 1 && fake::launches("pair_w") == 0);
    OK(fock_apply(p.h, 0, u, u, c.nb, out, fake::stream(0)));
    CHECK(fake::launches("mirror_add") == 1);
  }
}

// The same in FP32, whose sums on the CU need buffers that the pair form leaves unsized: a k-range, the energy
// gradient and separate targets captured after an eager adjoint (the choice of the form falls on the fused
// kernel for the k-range), and in a plan with a tuning cache, which measures nothing inside a capture.
void fp32_captures_use_what_is_there() {
  const std::string path = std::string(getenv("TMPDIR") ? getenv("TMPDIR") : "/tmp") + "/fockmi_capture_check.json";
  for (const CellSpec& c : {cube(20, 103, 2), cube(16, 40, 20), cube(32, 61, 1)})
    for (int tuned : {0, 1}) {
      remove(path.c_str());
      TestPlan p(FOCK_FP32_COMP, {c}, tuned ? path.c_str() : nullptr);
      const hipStream_t q = fake::stream(0);
      void *u = p.fields(), *out = p.fields(), *phi = p.fields(), *g = p.fields(), *gu = p.fields(), *gp = p.fields();
      OK(fock_vjp(p.h, 0, u, phi, c.nb, g, gu, gp, q));
      fake::st().bad_mallocs = 0;
      fake::st().ops.clear();
      fake::st().capturing.insert(q);
      OK(fock_energy_vjp(p.h, 0, u, 1.0, gu, q));
      OK(fock_apply_krange(p.h, 0, u, 1, c.nk / 2, phi, c.nb, out, q));
      OK(fock_apply(p.h, 0, u, phi, c.nb, out, q));
      fake::st().capturing.clear();
      CHECK(fake::st().bad_mallocs == 0);
    }
  remove(path.c_str());
}

// On a device with little memory left the pair scratch gives way to the buffers that other calls need, takes
// no more than the batch of a sum in one block, and shrinks as far as it has to where there is no other form.
void device_nearly_full() {
  const hipStream_t q = fake::stream(0);
  {
    TestPlan p(FOCK_FP32_COMP, {cube(24, 64, 16)});
    void *u = p.fields(), *out = p.fields(), *psi = p.fields();
    const double a[3] = {0.0, 0.0, 0.01};
    fake::st().limit = fake::st().used() + (size_t(2) << 30);
    OK(fock_apply(p.h, 0, u, u, 16, out, q));
    OK(taylor_step(p.h, 0, psi, nullptr, a, 0.01, 0.25, 4, nullptr, q));
    OK(fock_apply(p.h, 0, u, u, 16, out, q));
    fake::st().limit = ~size_t(0);
  }
  {
    TestPlan p(FOCK_FP64, {CellSpec{{16, 20, 24}, 3, 5}});
    void *u = p.fields(), *phi = p.fields(), *out = p.fields();
    fake::st().limit = fake::st().used() + 15 * 15 * 7680 * 16;  // the batch of all pairs
    OK(fock_apply(p.h, 0, u, phi, 5, out, q));
    fake::st().limit = ~size_t(0);
  }
  {
    TestPlan p(FOCK_FP64, {cube(32, 8, 16)});
    void *u = p.fields(), *phi = p.fields(), *out = p.fields();
    fake::st().limit = fake::st().used() + (size_t(20) << 20);
    OK(fock_apply(p.h, 0, u, phi, 16, out, q));
    fake::st().limit = ~size_t(0);
  }
}

const std::map<std::string, std::function<void()>> scenarios = {
    {"device_nearly_full", device_nearly_full},
    {"fp32_captures_use_what_is_there", fp32_captures_use_what_is_there},
    {"grid_forms_of_the_device_tests", grid_forms_of_the_device_tests},
    {"wait_limit_runs_the_split_form", wait_limit_runs_the_split_form},
    {"batched_route", batched_route},
    {"refused_sum_is_not_profiled", refused_sum_is_not_profiled},
    {"captures_use_what_is_there", captures_use_what_is_there},
    {"fused_sums_beyond_the_cap", fused_sums_beyond_the_cap},
    {"same_kernel_for_a_k_range", same_kernel_for_a_k_range},
    {"symmetry_switch", symmetry_switch},
    {"tuned_call_without_room", tuned_call_without_room},
    {"first_sum_allocates_once", first_sum_allocates_once},
    {"streams_in_order", streams_in_order},
    {"threads_one_at_a_time", threads_one_at_a_time},
    {"captures_without_plan_memory", captures_without_plan_memory},
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
