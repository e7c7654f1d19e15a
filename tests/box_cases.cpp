// Cases of the library's box object (csrc/box.hip) on the stand-in runtime, with
// stand-ins for the kernels' launchers; argv[1] names one.  Exit status 0: as
// it should be.
#define FAKE_HIP_MAIN
#include "fake_hip.hpp"

#include <vector>

#include "../paper_1601_03815_amd/csrc/runtime.hpp"

extern "C" {
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = fake::stream(0); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { delete reinterpret_cast<fake::Stream *>(s); return hipSuccess; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorUnknown; }
}

namespace {
int steps_launched = 0, failing_step = -1;
std::vector<double *> summed;  // where sums were added up, in order
}  // namespace

namespace dhit {
int fused_dugks_blocks(const dhit_params &, int *, int *, int *, int *) { return 8; }
int fused_auto_chunk(const dhit_params &) { return 8; }
int lbe_items(int64_t, const LbeSplit &) { return 8; }
LbeSplit lbe_split(int, int, int) { return {1, 128}; }
void spectrum_free(dhit_box &) {}
void timer_free(dhit_box &) {}
void copy_to_host(std::initializer_list<HostCopy>, hipStream_t) {}
void box_made() {}
void box_gone() {}
void lbe_table_entries(const dhit_box &, BatchBox (&e)[2]) { std::memset(&e, 0, sizeof(e)); }
void fused_table_entries(const dhit_box &b, BatchBox (&e)[2]) {
  std::memset(&e, 0, sizeof(e));
  for (BatchBox &x : e) {
    x.mesh_width = b.mesh;
    x.mesh_coef = b.mesh ? b.mesh + 3 * b.n : nullptr;
  }
}
void launch_finalize_sums(dhit_box &, const double *, int, double *out) { summed.push_back(out); }
static void step(dhit_box &b, double *out, bool defer, PendingSums *pend) {
  if (steps_launched == failing_step) throw Error(DHIT_EDEVICE, "launch failed");
  ++steps_launched;
  if (pend && pend->nblocks > 0) summed.push_back(pend->out);  // by the launch's extra block
  if (pend) *pend = {nullptr, 0, nullptr};
  if (defer)
    *pend = {b.partials, 8, out};
  else
    launch_finalize_sums(b, b.partials, 8, out);
}
void launch_lbe_step(dhit_box &b, const void *, void *, double *out, bool defer, PendingSums *pend) {
  step(b, out, defer, pend);
}
void launch_dugks_step(dhit_box &b, const void *, void *, double *out, bool defer, PendingSums *pend) {
  step(b, out, defer, pend);
}
}  // namespace dhit

#define CHECK(x)                                             \
  do {                                                       \
    if (!(x)) {                                              \
      std::fprintf(stderr, "line %d: %s\n", __LINE__, #x);   \
      return 1;                                              \
    }                                                        \
  } while (0)

// A launch that fails in a run of steps: the steps before it are taken, and
// their sums are in the history.
static int failing_launch() {
  for (int method : {DHIT_LBE_BGK, DHIT_DUGKS})
    for (int fails : {0, 1, 2, 5}) {
      dhit_params p;
      CHECK(default_params(8, method, DHIT_FP64, 0.01, &p) == DHIT_OK);
      dhit_box *b = nullptr;
      CHECK(create_box(&p, &b) == DHIT_OK);
      steps_launched = 0;
      failing_step = fails;
      summed.clear();
      CHECK((method == DHIT_DUGKS ? step_dugks(b, 6) : step_lbe(b, 6)) == DHIT_EDEVICE);
      CHECK(std::string(dhit_last_error()).find("launch failed") != std::string::npos);
      CHECK(steps_taken(b) == fails && (int)summed.size() == fails);
      for (int k = 0; k < fails; ++k) CHECK(summed[k] == b->hist + 5 * k);
      destroy_box(b);
    }
  return 0;
}

// A copy that fails in set_mesh: whatever kernel the box's next step chooses
// (b->mesh) finds the tables that kernel reads in the step's table.
static int failing_mesh() {
  const int n = 8;
  const std::vector<double> w(3 * n, 1.0), w2(3 * n, 1.25);
  for (int variant : {DHIT_VARIANT_DEFAULT, DHIT_VARIANT_TWO_PASS})
    for (bool stretched : {false, true})
      for (int fails = 0; fails < 3; ++fails) {
        dhit_params p;
        CHECK(default_params(n, DHIT_DUGKS, DHIT_FP64, 0.01, &p) == DHIT_OK);
        p.variant = variant;
        dhit_box *b = nullptr;
        CHECK(create_box(&p, &b) == DHIT_OK);
        if (stretched) CHECK(set_mesh(b, w.data()) == DHIT_OK);
        auto whole = [&] {
          if (!b->mesh) return true;
          for (int e = 0; e < 2; ++e)
            if (b->step_table[e].mesh_width != b->mesh || b->step_table[e].mesh_coef != b->mesh + 3 * n) return false;
          return true;
        };
        fake::copies_until_failure = fails;
        const int32_t st = set_mesh(b, w2.data());
        const bool ran_out = fake::copies_until_failure == 0;
        fake::copies_until_failure = -1;
        CHECK(st == DHIT_OK || (st == DHIT_EDEVICE && ran_out));
        CHECK(whole() && (st == DHIT_OK || (b->mesh != nullptr) == stretched));
        CHECK(set_mesh(b, w2.data()) == DHIT_OK && b->mesh && whole() && b->mesh[0] == 1.25);
        CHECK(set_mesh(b, nullptr) == DHIT_OK && !b->mesh);
        CHECK(set_mesh(b, w.data()) == DHIT_OK && b->mesh && whole());
        destroy_box(b);
      }
  return 0;
}

int main(int argc, char **argv) {
  const std::string c = argc > 1 ? argv[1] : "";
  if (c == "failing_launch") return failing_launch();
  if (c == "failing_mesh") return failing_mesh();
  return 2;
}
