// Checks of the library's host code over the fake runtime of fake_hip.h, one
// a run: host_calls NAME.  Exit status 0 when the check holds.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <string>
#include <thread>
#include <vector>

#include "fake_hip.h"
#include "nflbm.h"

using fake::state;

static int failures = 0;
#define CHECK(cond)                                                        \
  do {                                                                     \
    if (!(cond)) {                                                         \
      std::fprintf(stderr, "line %d: %s does not hold\n", __LINE__, #cond); \
      ++failures;                                                          \
    }                                                                      \
  } while (0)

struct Problem {
  std::vector<double> sigma, tau;
  nflbm_config cfg;
  Problem(int lattice, int nx, int ny, int nz, int N, int precision, int flags = 0) : sigma(size_t(N) * N, 0.006), tau(N, 1.0) {
    for (int i = 0; i < N; ++i) sigma[size_t(i) * N + i] = 0.0;
    std::memset(&cfg, 0, sizeof(cfg));
    cfg.lattice = lattice;
    cfg.nx = nx;
    cfg.ny = ny;
    cfg.nz = nz;
    cfg.ncomp = N;
    cfg.implicit_comp = -1;
    cfg.sigma = sigma.data();
    cfg.tau = tau.data();
    cfg.width_D = 4.0;
    cfg.m = (flags & NFLBM_FLAG_C2C2_MOBILITY) ? 10.0 : 0.05;
    cfg.precision = precision;
    cfg.flags = flags;
  }
  Problem(const Problem&) = delete;
};

static nflbm_sim* make(const Problem& p) {
  nflbm_sim* s = nullptr;
  CHECK(nflbm_create(&p.cfg, &s) == NFLBM_OK);
  return s;
}

// A state taken from elsewhere may hold velocities also where the run does
// not evolve the flow; only a single step reads them.
static void restored_velocities() {
  Problem p(NFLBM_D2Q9, 64, 48, 1, 3, NFLBM_FP32, NFLBM_FLAG_NO_HYDRO);
  nflbm_sim* s = make(p);
  CHECK(nflbm_step(s, 9) == NFLBM_OK);
  CHECK(state().count("fused2d") > 0);
  size_t bytes = 0;
  CHECK(nflbm_state_bytes(s, &bytes) == NFLBM_OK);
  std::vector<unsigned char> raw(bytes);
  CHECK(nflbm_get_state(s, raw.data()) == NFLBM_OK);
  CHECK(nflbm_set_state(s, raw.data()) == NFLBM_OK);
  state().launches.clear();
  CHECK(nflbm_step(s, 8) == NFLBM_OK);
  CHECK(state().launches.front().kind == "conc");
  CHECK(state().count("conc") < 3 && state().count("fused2d") > 0);
  nflbm_destroy(s);
}

// A captured step reads and writes fixed record sets, so every call leaves
// the state where as many single steps would.
static void state_parity() {
  Problem p(NFLBM_D2Q9, 64, 48, 1, 3, NFLBM_FP32);
  nflbm_sim* s = make(p);
  nflbm_batch* b = nullptr;
  CHECK(nflbm_batch_create(&p.cfg, 1, &b) == NFLBM_OK);
  auto sim_source = [&] {      // C set that one more step reads
    CHECK(nflbm_step(s, 1) == NFLBM_OK);
    const auto& l = state().launches;
    return l[l.size() - 2].step.cprev;
  };
  auto batch_source = [&] {
    CHECK(nflbm_batch_step(b, 1, NFLBM_BATCH_LAUNCH) == NFLBM_OK);
    return state().launches.back().step.cprev;
  };
  const void* const s0 = sim_source();
  const void* const b0 = batch_source();
  long long total = 1;
  for (long long n : {3, 2, 7, 9, 500}) {
    CHECK(nflbm_step(s, n) == NFLBM_OK);
    CHECK(nflbm_batch_step(b, n, NFLBM_BATCH_LAUNCH) == NFLBM_OK);
    total += n;
    CHECK((sim_source() == s0) == (total % 2 == 0));
    CHECK((batch_source() == b0) == (total % 2 == 0));
    ++total;
  }
  CHECK(state().count("fused2d") > 0 && state().count("fused2d_batch") > 0);
  nflbm_destroy(s);
  nflbm_batch_destroy(b);
}

// Stepping queues launches: it allocates nothing, and a batch waits for
// nothing once the first step after set_fields is done.
static void stepping_allocates_nothing() {
  const int forms[] = {0, NFLBM_FLAG_NO_HYDRO, NFLBM_FLAG_NO_HYDRO | NFLBM_FLAG_C2C2_MOBILITY, NFLBM_FLAG_F_POPULATIONS};
  for (int flags : forms)
    for (int precision : {NFLBM_FP64, NFLBM_FP32, NFLBM_FP16S}) {
      Problem p(NFLBM_D2Q9, 70, 50, 1, 3, precision, flags);
      nflbm_sim* s = make(p);
      nflbm_batch* b = nullptr;
      CHECK(nflbm_batch_create(&p.cfg, 1, &b) == NFLBM_OK);
      std::vector<double> C(3 * 70 * 50, 1.0 / 3.0), out(C.size());
      CHECK(nflbm_set_fields(s, C.data(), nullptr, nullptr) == NFLBM_OK);
      CHECK(nflbm_batch_set_fields(b, 0, C.data(), nullptr, nullptr) == NFLBM_OK);
      for (bool read : {false, true}) {
        if (read) {
          CHECK(nflbm_get_field(s, NFLBM_FIELD_C, out.data()) == NFLBM_OK);
          CHECK(nflbm_batch_get_field(b, 0, NFLBM_FIELD_C, out.data()) == NFLBM_OK);
        }
        long long before = state().mallocs;
        CHECK(nflbm_step(s, 1) == NFLBM_OK && nflbm_step(s, 9) == NFLBM_OK);
        CHECK(nflbm_batch_step(b, 1, NFLBM_BATCH_LAUNCH) == NFLBM_OK);
        CHECK(state().mallocs == before);
        const long long waits = state().syncs;
        CHECK(nflbm_batch_step(b, 9, NFLBM_BATCH_LAUNCH) == NFLBM_OK && nflbm_batch_step(b, 2, NFLBM_BATCH_LAUNCH) == NFLBM_OK);
        CHECK(state().mallocs == before && state().syncs == waits);
        double ms = 0.0;
        CHECK(nflbm_step_timed(s, 6, &ms, nullptr) == NFLBM_OK);
        CHECK(state().mallocs == before);
      }
      nflbm_destroy(s);
      nflbm_batch_destroy(b);
    }
  CHECK(state().count("fused2d") > 0 && state().count("fused2d_batch") > 0 && state().count("fused_mob") > 0);
  CHECK(state().device.empty() && state().pinned.empty() && state().events == 0);
}

// The other record set of the fused steps: no more than its values, and a
// simulation without room for it steps through the two kernels.
static void other_record_set() {
  for (int N = 2; N <= 8; ++N)
    for (int precision : {NFLBM_FP64, NFLBM_FP32, NFLBM_FP16S}) {
      Problem p(NFLBM_D2Q9, 128, 96, 1, N, precision);
      const size_t n = 128 * 96, rs = precision == NFLBM_FP64 ? 8 : (precision == NFLBM_FP32 ? 4 : 2);
      size_t planned = 0;
      CHECK(nflbm_device_bytes(&p.cfg, &planned) == NFLBM_OK);
      nflbm_sim* s = make(p);
      const size_t used = state().device_bytes();
      CHECK(nflbm_step(s, 1) == NFLBM_OK && nflbm_step(s, 8) == NFLBM_OK);
      CHECK(state().count("fused2d") > 0);
      CHECK(state().device_bytes() == used);
      CHECK(used <= planned + (8 + size_t(N - 1)) * n * rs + (64 << 10));
      nflbm_destroy(s);
    }
  state().launches.clear();
  Problem p(NFLBM_D2Q9, 128, 96, 1, 3, NFLBM_FP64);
  state().fail_at = (8 + 2) * size_t(128 * 96) * 8;
  nflbm_sim* s = make(p);
  nflbm_batch* b = nullptr;
  CHECK(nflbm_batch_create(&p.cfg, 1, &b) == NFLBM_OK);
  state().fail_at = 0;
  const long long before = state().mallocs;
  CHECK(nflbm_step(s, 9) == NFLBM_OK && nflbm_batch_step(b, 9, NFLBM_BATCH_LAUNCH) == NFLBM_OK);
  CHECK(state().mallocs == before);
  CHECK(state().count("conc") == 9 && state().count("batch") == 9);
  nflbm_destroy(s);
  nflbm_batch_destroy(b);
}

// The batch autotuner chooses the tile width of the two kernels, so it times
// those and not the fused launches, which have tiles of their own.
static void batch_autotune_times_its_kernels() {
  Problem p(NFLBM_D2Q9, 128, 96, 1, 3, NFLBM_FP32);
  nflbm_batch* b = nullptr;
  CHECK(nflbm_batch_create(&p.cfg, 1, &b) == NFLBM_OK);
  std::vector<double> C(3 * 128 * 96, 1.0 / 3.0);
  CHECK(nflbm_batch_set_fields(b, 0, C.data(), nullptr, nullptr) == NFLBM_OK);
  CHECK(nflbm_batch_step(b, 3, NFLBM_BATCH_GRAPH) == NFLBM_OK);
  CHECK(state().count("fused2d_batch") > 0);
  state().launches.clear();
  CHECK(nflbm_batch_autotune(b, nullptr) == NFLBM_OK);
  CHECK(state().count("fused2d_batch") == 0);
  CHECK(state().count("batch") > 0 && state().count("graph") > 0);
  state().launches.clear();
  CHECK(nflbm_batch_step(b, 4, NFLBM_BATCH_GRAPH) == NFLBM_OK);
  CHECK(state().count("fused2d_batch") > 0);
  nflbm_batch_destroy(b);
}

// So does a simulation's own, its warm-up steps included: they load the
// kernels of the shape that the timed steps take.
static void autotune_warms_its_kernels() {
  for (int flags : {0, int(NFLBM_FLAG_NO_HYDRO), NFLBM_FLAG_NO_HYDRO | NFLBM_FLAG_C2C2_MOBILITY}) {
    Problem p(NFLBM_D2Q9, 128, 96, 1, 3, NFLBM_FP32, flags);
    nflbm_sim* s = make(p);
    CHECK(nflbm_step(s, 1) == NFLBM_OK);
    state().launches.clear();
    CHECK(nflbm_autotune(s, nullptr) == NFLBM_OK);
    CHECK(state().count("fused2d") + state().count("fused_mob") == 0);
    CHECK(state().count("update") > 0);
    nflbm_destroy(s);
  }
}

// A large read-back without pinned memory for its slots copies plainly and
// gives back the events it made for them.
static void readback_without_pinned_memory() {
  Problem p(NFLBM_D3Q19, 128, 128, 86, 3, NFLBM_FP32);
  nflbm_sim* s = make(p);
  std::vector<double> out(3 * size_t(128 * 128 * 86));
  state().pinned_fails = true;
  for (int i = 0; i < 2; ++i) {
    std::fill(out.begin(), out.end(), -1.0);
    CHECK(nflbm_get_field(s, NFLBM_FIELD_C, out.data()) == NFLBM_OK);
    for (size_t q = 0; q < out.size(); ++q) CHECK(out[q] == double(q));
  }
  nflbm_destroy(s);
  CHECK(state().device.empty() && state().pinned.empty() && state().events == 0);
}

// Two threads that read fields of one simulation each get their own whole.
static void readback_from_two_threads() {
  const size_t n = 128 * 128 * 86;
  Problem p(NFLBM_D3Q19, 128, 128, 86, 3, NFLBM_FP32);
  nflbm_sim* s = make(p);
  std::vector<double> first(3 * n);
  CHECK(nflbm_get_field(s, NFLBM_FIELD_P, first.data()) == NFLBM_OK);
  std::vector<long long> wrong(2, 0);
  auto read = [&](int t) {
    const int field = t ? NFLBM_FIELD_V : NFLBM_FIELD_C;      // rows 3.. and 0.. of the fields
    const size_t off = t ? 3 * n : 0;
    std::vector<double> out(3 * n);
    for (int i = 0; i < 8; ++i) {
      std::fill(out.begin(), out.end(), -1.0);
      if (nflbm_get_field(s, field, out.data()) != NFLBM_OK) ++wrong[t];
      for (size_t q = 0; q < out.size(); ++q) wrong[t] += out[q] != double(off + q);
    }
  };
  std::thread a(read, 0), b(read, 1);
  a.join();
  b.join();
  CHECK(wrong[0] == 0 && wrong[1] == 0);
  nflbm_destroy(s);
  CHECK(state().device.empty() && state().pinned.empty() && state().events == 0);
}

// Solid nodes take 4 bytes a node, 8 while a face is open or the outflow's;
// where the second map does not fit, nothing changes.
static void solid_memory() {
  Problem p(NFLBM_D3Q19, 32, 24, 20, 3, NFLBM_FP32);
  p.cfg.wall[0] = 1;
  const size_t n = 32 * 24 * 20;
  nflbm_sim* s = make(p);
  std::vector<unsigned char> solid(n, 0);
  for (size_t q = 0; q < n; ++q) solid[q] = (q / 32) % 24 < 3;
  const double v[3] = {0.01, 0.0, 0.0}, c[3] = {0.5, 0.25, 0.25};
  const size_t base = state().device_bytes();
  CHECK(nflbm_set_solid(s, solid.data()) == NFLBM_OK);
  CHECK(state().device_bytes() == base + 4 * n);
  state().fail_at = 4 * n;
  CHECK(nflbm_set_open_face(s, 0, v, c) == NFLBM_ENOMEM);
  CHECK(nflbm_set_outflow(s, 1) == NFLBM_ENOMEM);
  CHECK(nflbm_set_solid(s, nullptr) == NFLBM_OK);
  CHECK(nflbm_set_solid(s, solid.data()) == NFLBM_ENOMEM);
  CHECK(state().device_bytes() == base);
  CHECK(nflbm_step(s, 1) == NFLBM_OK);
  CHECK(!state().launches.back().step.bb && !state().launches.back().step.faces);
  state().fail_at = 0;
  CHECK(nflbm_set_open_face(s, 0, v, c) == NFLBM_OK);
  const size_t open = state().device_bytes();
  CHECK(open < base + 4 * n);
  CHECK(nflbm_set_solid(s, solid.data()) == NFLBM_OK);
  CHECK(state().device_bytes() == open + 8 * n && state().count("build_ob") == 1);
  CHECK(nflbm_set_outflow(s, 1) == NFLBM_OK && state().count("build_ob") == 2);
  CHECK(nflbm_step(s, 1) == NFLBM_OK);
  // the outflow moves to the other face
  CHECK(nflbm_set_open_face(s, 0, nullptr, nullptr) == NFLBM_OK && nflbm_set_outflow(s, 0) == NFLBM_OK);
  CHECK(nflbm_step(s, 1) == NFLBM_OK);
  CHECK(nflbm_set_outflow(s, 1) == NFLBM_OK && nflbm_set_open_face(s, 0, v, c) == NFLBM_OK);
  CHECK(nflbm_step(s, 1) == NFLBM_OK);
  for (const fake::Launch& l : state().launches)
    if (l.kind == "conc" && l.step.faces) CHECK(l.step.bb && l.step.ob);
  CHECK(nflbm_set_outflow(s, -1) == NFLBM_OK && nflbm_set_open_face(s, 0, nullptr, nullptr) == NFLBM_OK);
  CHECK(state().device_bytes() == base + 4 * n);
  CHECK(nflbm_set_solid(s, nullptr) == NFLBM_OK);
  CHECK(state().device_bytes() == base);
  nflbm_destroy(s);
  CHECK(state().device.empty() && state().pinned.empty() && state().events == 0);
}

// A batch launch takes one storage form of f for all members.
static void batch_shares_the_form_of_f() {
  Problem a(NFLBM_D2Q9, 64, 48, 1, 3, NFLBM_FP32), b(NFLBM_D2Q9, 40, 48, 1, 3, NFLBM_FP32),
      c(NFLBM_D2Q9, 32, 32, 1, 3, NFLBM_FP32, NFLBM_FLAG_NO_HYDRO);
  b.tau.assign(3, 0.8);
  const std::vector<std::vector<nflbm_config>> mixes = {{a.cfg, b.cfg}, {b.cfg, a.cfg}, {a.cfg, c.cfg}, {c.cfg, a.cfg},
                                                        {a.cfg, a.cfg}, {c.cfg, c.cfg}};
  for (const auto& m : mixes) {
    nflbm_batch* h = nullptr;
    CHECK(nflbm_batch_create(m.data(), int(m.size()), &h) == NFLBM_OK);
    const int form = nflbm_f_storage_form(nflbm_batch_member(h, 0));
    for (int i = 0; i < nflbm_batch_count(h); ++i) CHECK(nflbm_f_storage_form(nflbm_batch_member(h, i)) == form);
    CHECK(form == (&m == &mixes[4]));
    CHECK(nflbm_batch_step(h, 9, NFLBM_BATCH_LAUNCH) == NFLBM_OK);
    nflbm_batch_destroy(h);
  }
}

// The shape and number of the workgroups of four steps of an nx x ny lattice
// (threads 0 where the two kernels take them).
static fake::Launch four_steps(int nx, int ny, int N, int precision, double omega, int flags = 0) {
  Problem p(NFLBM_D2Q9, nx, ny, 1, N, precision, flags);
  p.cfg.omega_stab = omega;
  nflbm_sim* s = make(p);
  CHECK(nflbm_step(s, 1) == NFLBM_OK);
  state().launches.clear();
  CHECK(nflbm_step(s, 4) == NFLBM_OK);
  const fake::Launch l = state().launches.back();
  nflbm_destroy(s);
  return l;
}

// Beyond one round of workgroups the fused steps are taken where they measured
// faster than the two kernels.
static void fused_shapes() {
  const size_t lds = 160 << 10;
  for (int precision : {NFLBM_FP64, NFLBM_FP32, NFLBM_FP16S})
    for (int N = 2; N <= 8; ++N)
      for (double omega : {0.0, 0.05})
        for (int flags : {0, int(NFLBM_FLAG_NO_HYDRO)}) {
          const bool f64 = precision == NFLBM_FP64, half = precision == NFLBM_FP16S, options = omega != 0.0;
          const fake::Launch big = four_steps(1100, 1000, N, precision, omega, flags);
          const bool two = !flags && (f64 ? N == 7 && options
                                          : N == 8 || (N == 7 && (half || options)) || (half && (N == 5 || N == 6) && options));
          CHECK((big.kind == "fused2d") == !two);
          if (two) continue;
          CHECK(big.shape.lds <= lds);
          if (!f64 && N >= 4 && !flags) CHECK(big.shape.threads == 512 && 2 * big.shape.lds <= lds);
          if (f64 && N >= 7 && !flags) CHECK(big.fused.tile_h >= 11);
          // a small lattice is one round of small tiles in every form
          const fake::Launch small = four_steps(90, 70, N, precision, omega, flags);
          CHECK(small.kind == "fused2d" && small.shape.blocks <= 256);
        }
  // a second round of few workgroups
  CHECK(four_steps(560, 540, 5, NFLBM_FP32, 0.0).kind != "fused2d");
  CHECK(four_steps(700, 650, 5, NFLBM_FP32, 0.0).kind == "fused2d");
  // the shortest tile of one round
  CHECK(four_steps(420, 430, 4, NFLBM_FP32, 0.0).fused.tile_h <= 16);
  // N = 7 in FP16S: one round of tall tiles, then the two kernels
  CHECK(four_steps(370, 370, 7, NFLBM_FP16S, 0.0).kind == "fused2d");
  CHECK(four_steps(420, 430, 7, NFLBM_FP16S, 0.0).kind != "fused2d");
}

// N = 8 in FP64 with the concentration-dependent mobility: one step a launch,
// by tiles of 12 rows once those of 8 are more than a round of workgroups.
static void mobility_shapes() {
  const int flags = NFLBM_FLAG_NO_HYDRO | NFLBM_FLAG_C2C2_MOBILITY;
  const fake::Launch small = four_steps(60, 64, 8, NFLBM_FP64, 0.05, flags);
  CHECK(small.kind == "fused_mob" && small.nsteps == 1 && small.shape.blocks == 3 * 8);
  const fake::Launch big = four_steps(480, 480, 8, NFLBM_FP64, 0.05, flags);
  CHECK(big.kind == "fused_mob" && big.nsteps == 1 && big.shape.blocks == 18 * 40);
  CHECK(four_steps(480, 480, 4, NFLBM_FP32, 0.05, flags).nsteps == 2);
}

// The z runs of a batch fill the workgroup slots over all members, also where
// each alone would take long ones; a run that was set stays.
static void batch_runs_share_the_slots() {
  state().groups_per_cu = 3;
  Problem p(NFLBM_D3Q19, 137, 78, 179, 5, NFLBM_FP32), q(NFLBM_D3Q19, 60, 40, 30, 5, NFLBM_FP32);
  const long long slots = 3 * 256;
  for (int count : {1, 2, 3, 5, 8}) {
    std::vector<nflbm_config> cfgs(count, p.cfg);
    cfgs.push_back(q.cfg);
    nflbm_batch* b = nullptr;
    CHECK(nflbm_batch_create(cfgs.data(), int(cfgs.size()), &b) == NFLBM_OK);
    int tx = 0;
    CHECK(nflbm_batch_get_launch(b, &tx, nullptr, nullptr) == NFLBM_OK && tx == 6);
    CHECK(nflbm_batch_step(b, 1, NFLBM_BATCH_LAUNCH) == NFLBM_OK);
    const fake::Launch l = state().launches.back();
    const long long tiles = count * 3LL * 20, small = 10;
    long long best = 0;
    for (int zc = 1; zc <= 179; ++zc) {
      const long long groups = tiles * ((179 + zc - 1) / zc) + small * ((30 + zc - 1) / zc);
      const long long cost = (groups + slots - 1) / slots * (zc + 2);
      if (zc == 1 || cost < best) best = cost;
    }
    CHECK((l.shape.blocks + slots - 1) / slots * (l.step.zchunk + 2) == best);
    nflbm_batch_destroy(b);
  }
  nflbm_config cfgs[2] = {p.cfg, p.cfg};
  nflbm_batch* b = nullptr;
  CHECK(nflbm_batch_create(cfgs, 2, &b) == NFLBM_OK);
  CHECK(nflbm_set_launch(nflbm_batch_member(b, 0), 6, 7) == NFLBM_OK);
  CHECK(nflbm_batch_step(b, 1, NFLBM_BATCH_LAUNCH) == NFLBM_OK);
  CHECK(state().launches.back().step.zchunk == 7);
  nflbm_batch_destroy(b);
}

// Calls of two and three steps beyond one round: one step a launch, where that
// measured faster than the two kernels.
static void short_calls() {
  for (int precision : {NFLBM_FP64, NFLBM_FP32, NFLBM_FP16S})
    for (int N = 2; N <= 8; ++N)
      for (int side : {90, 1000}) {
        Problem p(NFLBM_D2Q9, side, side, 1, N, precision);
        nflbm_sim* s = make(p);
        nflbm_batch* b = nullptr;
        CHECK(nflbm_batch_create(&p.cfg, 1, &b) == NFLBM_OK);
        CHECK(nflbm_step(s, 1) == NFLBM_OK && nflbm_batch_step(b, 1, NFLBM_BATCH_LAUNCH) == NFLBM_OK);
        const bool few = side == 90 || (precision != NFLBM_FP64 && N <= 4);
        for (int n : {2, 3}) {
          state().launches.clear();
          CHECK(nflbm_step(s, n) == NFLBM_OK && nflbm_batch_step(b, n, NFLBM_BATCH_LAUNCH) == NFLBM_OK);
          CHECK(state().count("fused2d") == (few ? 2 : 0) && state().count("fused2d_batch") == (few ? 2 : 0));
        }
        nflbm_destroy(s);
        nflbm_batch_destroy(b);
      }
}

// The table of the open faces is replaced by a copy on the default stream,
// which does not wait for steps queued on the simulation's: the call does.
static void open_faces_wait_for_queued_steps() {
  Problem p(NFLBM_D3Q19, 20, 12, 10, 3, NFLBM_FP32);
  p.cfg.wall[0] = 1;
  nflbm_sim* s = make(p);
  const double v[3] = {0.01, 0.0, 0.0}, c[3] = {0.5, 0.25, 0.25};
  CHECK(nflbm_set_open_face(s, 0, v, c) == NFLBM_OK && nflbm_set_open_face(s, 1, v, c) == NFLBM_OK);
  for (bool open : {true, false}) {
    CHECK(nflbm_step(s, 3) == NFLBM_OK);
    const long long waits = state().syncs;
    CHECK(nflbm_set_open_face(s, 0, open ? v : nullptr, open ? c : nullptr) == NFLBM_OK);
    CHECK(state().copied_after > waits);
  }
  nflbm_destroy(s);
}

// The first step after set_fields takes f from each node's own record; batch
// steps after it do not, also where the members took it on their own or were
// given a state.
static void batch_after_members_stepped() {
  for (int lattice : {int(NFLBM_D2Q9), int(NFLBM_D3Q19)}) {
    Problem p(lattice, 20, 18, lattice == NFLBM_D2Q9 ? 1 : 9, 3, NFLBM_FP32);
    std::vector<unsigned char> raw;
    for (int how = 0; how < 3; ++how) {
      nflbm_batch* b = nullptr;
      CHECK(nflbm_batch_create(&p.cfg, 1, &b) == NFLBM_OK);
      nflbm_sim* m = nflbm_batch_member(b, 0);
      if (how == 0) CHECK(nflbm_batch_step(b, 2, NFLBM_BATCH_PER_SIM) == NFLBM_OK);
      if (how == 1) CHECK(nflbm_step(m, 3) == NFLBM_OK);
      if (how == 2) CHECK(nflbm_set_state(m, raw.data()) == NFLBM_OK);
      for (int i = 0; i < 3; ++i) {
        CHECK(nflbm_batch_step(b, 1, NFLBM_BATCH_LAUNCH) == NFLBM_OK);
        CHECK(state().launches.back().kind == "batch");
        CHECK(!(state().launches.back().step.flags & nflbm::kFlagFLocal));
      }
      size_t bytes = 0;
      CHECK(nflbm_state_bytes(m, &bytes) == NFLBM_OK);
      raw.resize(bytes);
      CHECK(nflbm_get_state(m, raw.data()) == NFLBM_OK);
      nflbm_batch_destroy(b);
    }
  }
}

int main(int argc, char** argv) {
  const std::string name = argc > 1 ? argv[1] : "";
  if (name == "restored_velocities") restored_velocities();
  else if (name == "state_parity") state_parity();
  else if (name == "stepping_allocates_nothing") stepping_allocates_nothing();
  else if (name == "batch_autotune_times_its_kernels") batch_autotune_times_its_kernels();
  else if (name == "autotune_warms_its_kernels") autotune_warms_its_kernels();
  else if (name == "readback_without_pinned_memory") readback_without_pinned_memory();
  else if (name == "readback_from_two_threads") readback_from_two_threads();
  else if (name == "solid_memory") solid_memory();
  else if (name == "batch_shares_the_form_of_f") batch_shares_the_form_of_f();
  else if (name == "fused_shapes") fused_shapes();
  else if (name == "mobility_shapes") mobility_shapes();
  else if (name == "batch_runs_share_the_slots") batch_runs_share_the_slots();
  else if (name == "short_calls") short_calls();
  else if (name == "open_faces_wait_for_queued_steps") open_faces_wait_for_queued_steps();
  else if (name == "batch_after_members_stepped") batch_after_members_stepped();
  else if (name == "other_record_set") other_record_set();
  else {
    std::fprintf(stderr, "no check named '%s'\n", name.c_str());
    return 2;
  }
  return failures ? 1 : 0;
}
