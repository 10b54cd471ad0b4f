// Checks of the library's host code over the fake runtime of fake_hip.h, one
// a run: host_calls NAME.  Exit status 0 when the check holds.
#include <cstdio>
#include <cstring>
#include <string>
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

// C set last by the launches so far: where the next single step reads from
static const void* next_source(nflbm_sim* s) {
  CHECK(nflbm_step(s, 1) == NFLBM_OK);
  const auto& l = state().launches;
  CHECK(l.size() >= 2 && l[l.size() - 2].kind == "conc");
  return l[l.size() - 2].step.cprev;
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

int main(int argc, char** argv) {
  const std::string name = argc > 1 ? argv[1] : "";
  if (name == "restored_velocities") restored_velocities();
  else {
    std::fprintf(stderr, "no check named '%s'\n", name.c_str());
    return 2;
  }
  (void)next_source;
  return failures ? 1 : 0;
}
