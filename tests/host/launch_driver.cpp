// Checks of the launch sequences of the host side of the library on the CPU device of
// device_double.cpp.  Run with the name of a check; exits non-zero if it fails.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <memory>
#include <utility>

#include "device_double.h"
#include "lbm_ch.h"

static int fails = 0;
#define EXPECT(cond, ...)                                              \
  do {                                                                 \
    if (!(cond)) {                                                     \
      fprintf(stderr, "%s:%d: expected %s: ", __FILE__, __LINE__, #cond); \
      fprintf(stderr, __VA_ARGS__);                                    \
      fprintf(stderr, "\n");                                           \
      ++fails;                                                         \
    }                                                                  \
  } while (0)

static lbm_ch_params params(int nx, int ny, double tau = 1.0) {
  lbm_ch_params p;
  memset(&p, 0, sizeof p);
  p.nx = nx; p.ny = ny; p.model = 2; p.tau_g = tau; p.mobility = 0.01;
  p.sigma = 0.01; p.width = 4.0; p.phi_a = 1.0; p.phi_b = -1.0;
  p.rho_a = 1.0; p.rho_b = 1.0; p.tau_f = 0.8;
  return p;
}

struct Lattice {
  lbm_ch_params p;
  void* ws;
  lbm_ch_ctx* c = nullptr;
  std::vector<float> phi;
  std::vector<char> state;
  explicit Lattice(const lbm_ch_params& q, const std::vector<double>& tf = {}) : p(q) {
    const size_t n = lbm_ch_workspace_bytes(&p);
    ws = aligned_alloc(256, n);
    phi.resize((size_t)p.nx * p.ny);
    lbm_ch_velocity v;
    memset(&v, 0, sizeof v);
    v.time_factor = tf.empty() ? nullptr : tf.data();
    v.n_time_factor = (int64_t)tf.size();
    EXPECT(lbm_ch_init(&c, &p, &v, ws, n, phi.data(), nullptr) == LBM_CH_OK, "init");
    state.resize(lbm_ch_state_bytes(c));
  }
  Lattice(const Lattice&) = delete;
  ~Lattice() {
    lbm_ch_destroy(c);
    free(ws);
  }
  // steps taken by the state as the read-out sees it (-1: refused)
  double seen() {
    return lbm_ch_moments(c, phi.data(), nullptr, nullptr, nullptr, nullptr, nullptr) == LBM_CH_OK
               ? phi[0] : -1.0;
  }
  // and as its saved populations hold it
  double saved() {
    if (lbm_ch_save_state(c, state.data(), state.size(), nullptr) != LBM_CH_OK) return -1.0;
    double v;
    memcpy(&v, state.data(), sizeof v);
    return v;
  }
};

// Sums, populations and step counter of a usable context say the same, now and later.
static void consistent(Lattice& l, const char* what) {
  for (int n : {0, 3, 2, 1, 4}) {
    EXPECT(lbm_ch_step(l.c, n, nullptr) == LBM_CH_OK, "%s", what);
    const double at = (double)lbm_ch_step_count(l.c);
    EXPECT(l.seen() == at && l.saved() == at, "%s: step %g, phi of %g, populations of %g", what,
           at, l.seen(), l.saved());
  }
}

// A launch that fails in the middle of a call either leaves state and step counter
// consistent, or a context that refuses every call on its state until one is loaded.
static void failed_launch() {
  for (int walls : {0, 1})
    for (double tau : {1.0, 0.8})
      for (auto [nx, ny] : {std::pair<int, int>{64, 60}, {300, 60}, {700, 60}, {64, 2100}})
        for (int graphs : {0, 1})
          for (int record : {0, 1})
            for (int n = 1; n <= 9; ++n)
              for (int at = 0; at < 2 * n + 1; ++at) {
                if (ny > 60 && (walls || tau != 1.0 || graphs)) continue;  // tiles in the last launch
                lbm_ch_params p = params(nx, ny, tau);
                p.walls = walls;
                Lattice l(p);
                lbm_ch_set_graphs(l.c, graphs);
                EXPECT(lbm_ch_step(l.c, 2, nullptr) == LBM_CH_OK, "step");
                EXPECT(l.saved() == 2.0, "saved");
                const std::vector<char> two = l.state;
                std::vector<float> traj(record ? (size_t)n * nx * ny : 0);
                dbl::fail_in = at;
                const int r = record ? lbm_ch_record(l.c, n, traj.data(), nullptr)
                                     : lbm_ch_step(l.c, n, nullptr);
                if (dbl::fail_in >= 0 || r == LBM_CH_OK) {  // fewer launches than that
                  dbl::fail_in = -1;
                  EXPECT(r == LBM_CH_OK && l.seen() == 2 + n, "no failure");
                  continue;
                }
                char what[120];
                snprintf(what, sizeof what, "walls %d tau %g %d x %d graphs %d record %d: launch %d of %d steps",
                         walls, tau, nx, ny, graphs, record, at, n);
                EXPECT(r == LBM_CH_EHIP, "%s", what);
                if (l.seen() >= 0) {
                  consistent(l, what);
                  continue;
                }
                float us;
                EXPECT(at > 0, "%s: nothing was overwritten", what);
                EXPECT(lbm_ch_step(l.c, 1, nullptr) == LBM_CH_ESTATE, "%s", what);
                EXPECT(lbm_ch_record(l.c, 0, nullptr, nullptr) == LBM_CH_ESTATE, "%s", what);
                EXPECT(lbm_ch_check_finite(l.c, nullptr) == LBM_CH_ESTATE, "%s", what);
                EXPECT(l.saved() == -1.0, "%s", what);
                EXPECT(lbm_ch_autotune(l.c, l.state.data(), l.state.size(), 1, nullptr, &us) ==
                           LBM_CH_ESTATE, "%s", what);
                EXPECT(lbm_ch_load_state(l.c, two.data(), two.size(), 2, nullptr) == LBM_CH_OK, "%s", what);
                consistent(l, what);
              }
}

// The same for a batch, and for a load that fails between its copies and its sums.
static void failed_batch_and_load() {
  for (int n = 1; n <= 6; ++n)
    for (int at = 0; at < 2 * n; ++at) {
      Lattice a(params(64, 48)), b(params(80, 50, 0.9));
      lbm_ch_ctx* cs[2] = {a.c, b.c};
      const size_t nb = lbm_ch_batch_workspace_bytes(2);
      void* ws = aligned_alloc(256, (nb + 255) / 256 * 256);
      lbm_ch_batch* batch = nullptr;
      EXPECT(lbm_ch_batch_create(&batch, cs, 2, ws, nb) == LBM_CH_OK, "create");
      EXPECT(lbm_ch_batch_step(batch, 3, 0, nullptr) == LBM_CH_OK, "batch step");
      EXPECT(a.saved() == 3.0 && b.saved() == 3.0, "batch");
      dbl::fail_in = at;
      EXPECT(lbm_ch_batch_step(batch, n, 0, nullptr) == LBM_CH_EHIP, "launch %d of %d", at, n);
      for (Lattice* l : {&a, &b}) {
        EXPECT((l->seen() < 0) == (at > 0), "launch %d of %d", at, n);
        if (at == 0) continue;
        EXPECT(lbm_ch_batch_step(batch, 1, 0, nullptr) == LBM_CH_ESTATE, "lost member");
        EXPECT(lbm_ch_load_state(l->c, l->state.data(), l->state.size(), 3, nullptr) == LBM_CH_OK, "load");
      }
      EXPECT(lbm_ch_batch_step(batch, n, 0, nullptr) == LBM_CH_OK, "launch %d of %d", at, n);
      EXPECT(a.saved() == 3 + n && b.saved() == 3 + n && a.seen() == 3 + n, "launch %d of %d", at, n);
      lbm_ch_batch_destroy(batch);
      free(ws);
    }
  for (int at = 0; at < 2; ++at) {
    Lattice l(params(64, 48));
    EXPECT(l.saved() == 0.0, "saved");
    const std::vector<char> zero = l.state;
    EXPECT(lbm_ch_step(l.c, 5, nullptr) == LBM_CH_OK, "step");
    dbl::fail_in = at;
    const int r = lbm_ch_load_state(l.c, zero.data(), zero.size(), 0, nullptr);
    dbl::fail_in = -1;
    if (r != LBM_CH_OK && l.seen() < 0)
      EXPECT(lbm_ch_load_state(l.c, zero.data(), zero.size(), 0, nullptr) == LBM_CH_OK, "load");
    consistent(l, "load");
  }
}

// One step on one stream beside a read-out of the state before it on another, whatever the
// order in which their launches meet: the read-out sees its state, and the step is whole.
static void readout_beside_a_step() {
  const hipStream_t other = (hipStream_t)&fails;
  for (int walls : {0, 1})
    for (double tau : {1.0, 0.8})
      for (int what = 0; what < 3; ++what)
        for (size_t before = 0; before < 3; ++before) {  // launches that run before the step
          lbm_ch_params p = params(130, 60, tau);
          p.walls = walls;
          Lattice l(p);
          EXPECT(lbm_ch_step(l.c, 3, nullptr) == LBM_CH_OK, "step");
          std::vector<float> mu(130 * 60, -1.0f);
          double d[8] = {-1.0};
          dbl::side = other;
          float* phi = what == 1 ? l.phi.data() : nullptr;
          const int r = what == 2 ? lbm_ch_diagnostics(l.c, nullptr, d, other)
                                  : lbm_ch_moments(l.c, phi, mu.data(), nullptr, nullptr, nullptr, other);
          EXPECT(r == LBM_CH_OK, "read-out");
          size_t k = 0;
          for (; k < before && k < dbl::waiting.size(); ++k) dbl::waiting[k]();
          EXPECT(lbm_ch_step(l.c, 1, nullptr) == LBM_CH_OK, "step");
          for (; k < dbl::waiting.size(); ++k) dbl::waiting[k]();
          dbl::waiting.clear();
          dbl::side = nullptr;
          const double got = what == 2 ? d[0] : mu[0];
          EXPECT(got == 3.0, "walls %d tau %g read-out %d, %zu launches before: of step %g", walls, tau,
                 what, before, got);
          consistent(l, "after the read-out");
        }
}

static std::pair<int, int> tiles(const lbm_ch_ctx* c) {
  int32_t tx = 0, ty = 0;
  EXPECT(lbm_ch_get_tiles(c, &tx, &ty) == LBM_CH_OK, "get_tiles");
  return {tx, ty};
}
static std::pair<int, int> default_tiles(const lbm_ch_params& p) {
  int32_t tx = 0, ty = 0;
  EXPECT(lbm_ch_default_tiles(&p, &tx, &ty) == LBM_CH_OK, "default_tiles");
  return {tx, ty};
}
// kind of launch that one step is made of
static std::string step_kind(Lattice& l) {
  dbl::count.clear();
  EXPECT(lbm_ch_step(l.c, 1, nullptr) == LBM_CH_OK, "step");
  return dbl::count.size() == 1 ? dbl::count.begin()->first : "several";
}

// The autotuner sets what it has timed to be the fastest: the march or a tile where both
// serve, and nothing where no shape has an effect.  Setting the shape it reports on another
// context gives that context the same step, and the default shape the step of a new one.
static void autotune() {
  const std::pair<int, int> fast{128, 8};
  for (double tau : {1.0, 0.8})
    for (int walls : {0, 1})
      for (int march_wins : {0, 1}) {
        lbm_ch_params p = params(300, 200, tau);
        p.walls = walls;
        Lattice l(p);
        const auto def = default_tiles(p);
        EXPECT(def != fast, "the default is not the tile that the test makes the fastest");
        if (tau == 1.0) EXPECT(lbm_ch_set_tiles(l.c, 256, 4) == LBM_CH_OK, "set_tiles");
        EXPECT(lbm_ch_step(l.c, 3, nullptr) == LBM_CH_OK, "step");
        // later launches are quicker, so that the last of equal ones would win
        float drift = 0.0f;
        dbl::cost = [&](const std::string& kind, int shape) {
          drift -= 1e-4f;
          if (kind == "pop_march") return (march_wins ? 4.0f : 9.0f) + drift;
          return (kind == "tile" && shape == fast.first * 1000 + fast.second ? 6.0f : 12.0f) + drift;
        };
        float us = 0.0f;
        dbl::count.clear();
        EXPECT(lbm_ch_autotune(l.c, l.state.data(), l.state.size(), 4, nullptr, &us) == LBM_CH_OK, "autotune");
        dbl::cost = nullptr;
        EXPECT(lbm_ch_step_count(l.c) == 3 && l.seen() == 3.0, "restored");
        const auto set = tiles(l.c);
        if (tau == 1.0) {
          EXPECT(set == std::make_pair(256, 4), "%d x %d", set.first, set.second);
          EXPECT(dbl::count["march"] + dbl::count["block"] <= 1 + 4, "one trial");
          continue;
        }
        EXPECT(set == (march_wins ? def : fast), "%d x %d", set.first, set.second);
        EXPECT(us > (march_wins ? 3.9f : 5.9f) && us < (march_wins ? 4.1f : 6.1f), "%g us", us);
        const std::string want = march_wins ? "pop_march" : "tile";
        EXPECT(step_kind(l) == want, "%s", step_kind(l).c_str());
        Lattice other(p);
        EXPECT(lbm_ch_set_tiles(other.c, set.first, set.second) == LBM_CH_OK, "set_tiles");
        EXPECT(step_kind(other) == want, "%s", step_kind(other).c_str());
        EXPECT(lbm_ch_set_tiles(l.c, def.first, def.second) == LBM_CH_OK, "set_tiles");
        EXPECT(step_kind(l) == "pop_march", "%s", step_kind(l).c_str());
      }
}

// The batch autotuner sets the fastest schedule and tile of the lattices that have them, and
// nothing for a batch whose lattices all march; lattices of every kind step together.
static void batch_autotune() {
  for (int mixed : {0, 1}) {
    std::vector<std::unique_ptr<Lattice>> ls;
    std::vector<lbm_ch_ctx*> cs;
    for (int i = 0; i < 7; ++i) {
      lbm_ch_params p = params(40 + 70 * i, 50 + i, mixed && i % 2 ? 0.9 : 1.0);
      p.model = 1 + (i / 2) % 2;
      ls.push_back(std::make_unique<Lattice>(p));
      cs.push_back(ls.back()->c);
    }
    const size_t nb = lbm_ch_batch_workspace_bytes(7);
    void* ws = aligned_alloc(256, nb);
    lbm_ch_batch* b = nullptr;
    EXPECT(lbm_ch_batch_create(&b, cs.data(), 7, ws, nb) == LBM_CH_OK, "create");
    EXPECT(lbm_ch_batch_set_tiles(b, 128, 8) == LBM_CH_OK, "set_tiles");
    EXPECT(lbm_ch_batch_set_schedule(b, 1) == LBM_CH_OK, "set_schedule");
    EXPECT(lbm_ch_batch_step(b, 3, 0, nullptr) == LBM_CH_OK, "step");
    float drift = 0.0f;
    dbl::cost = [&](const std::string& kind, int shape) {
      drift -= 1e-4f;
      return (kind == "tile_batch" && shape == 2560 ? 6.0f : 12.0f) + drift;
    };
    const size_t nst = lbm_ch_batch_state_bytes(b);
    void* backup = aligned_alloc(256, nst);
    float us = 0.0f;
    dbl::count.clear();
    EXPECT(lbm_ch_batch_autotune(b, backup, nst, 4, nullptr, &us) == LBM_CH_OK, "autotune");
    dbl::cost = nullptr;
    int32_t tx = 0, ty = 0;
    EXPECT(lbm_ch_batch_get_tiles(b, &tx, &ty) == LBM_CH_OK, "get_tiles");
    const int persistent = lbm_ch_batch_get_schedule(b);
    if (mixed) {
      EXPECT(tx == 256 && persistent == 0, "%d x %d, schedule %d", tx, ty, persistent);
    } else {
      EXPECT(tx == 128 && ty == 8 && persistent == 1, "%d x %d, schedule %d", tx, ty, persistent);
      EXPECT(dbl::count["march_batch"] == 2 * (1 + 4), "%d launches", dbl::count["march_batch"]);
      EXPECT(dbl::count["occupancy"] == 0, "a launch that has no tiles was sized for them");
    }
    for (int n : {1, 2, 5}) EXPECT(lbm_ch_batch_step(b, n, n == 2, nullptr) == LBM_CH_OK, "step");
    for (auto& l : ls)
      EXPECT(lbm_ch_step_count(l->c) == 11 && l->seen() == 11.0 && l->saved() == 11.0, "nx %d: %g, %g",
             l->p.nx, l->seen(), l->saved());
    lbm_ch_batch_destroy(b);
    free(backup);
    free(ws);
  }
}

// A state is loaded by one kernel from this device's memory at 4-byte alignment where the sums
// are kept, and by a copy (and, with sums, a pass over it) from everywhere else.
static void load_routes() {
  for (double tau : {1.0, 0.8})
    for (int dev : {0, 1, -1, -2})
      for (int off : {0, 1, 2, 4}) {
        Lattice l(params(64, 48, tau));
        EXPECT(lbm_ch_step(l.c, 3, nullptr) == LBM_CH_OK && l.saved() == 3.0, "saved");
        std::vector<char> buf(l.state.size() + 8);
        memcpy(buf.data() + off, l.state.data(), l.state.size());
        EXPECT(lbm_ch_step(l.c, 2, nullptr) == LBM_CH_OK, "step");
        dbl::source_device = dev;
        dbl::count.clear();
        EXPECT(lbm_ch_load_state(l.c, buf.data() + off, l.state.size(), 3, nullptr) == LBM_CH_OK, "load");
        dbl::source_device = 0;
        const bool kernel = tau == 1.0 && dev == 0 && off % 4 == 0;
        EXPECT(dbl::count["load_sum"] == kernel && dbl::count["copy"] == !kernel &&
                   dbl::count["sum_field"] == (tau == 1.0 && !kernel), "device %d offset %d", dev, off);
        EXPECT(l.seen() == 3.0, "loaded");
        consistent(l, "loaded");
      }
}

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> checks = {{"failed_launch", failed_launch},
                                                    {"failed_batch_and_load", failed_batch_and_load},
                                                    {"readout_beside_a_step", readout_beside_a_step},
                                                    {"autotune", autotune},
                                                    {"batch_autotune", batch_autotune},
                                                    {"load_routes", load_routes}};
  const auto it = argc > 1 ? checks.find(argv[1]) : checks.end();
  if (it == checks.end()) return 2;
  it->second();
  printf("%s: %d failed expectations\n", argv[1], fails);
  return fails ? 1 : 0;
}
