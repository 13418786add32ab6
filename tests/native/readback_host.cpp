// Host side of the readbacks and of the step modes, on the HIP runtime of
// fake_hip.h.
// readback_host CASE runs one case and says "ok".
#include "fake_hip.h"

#include <string>
#include <thread>

#include "lbib.h"

#define CHECK(cond)                                                               \
  do {                                                                            \
    if (!(cond)) {                                                                \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #cond);      \
      std::exit(1);                                                               \
    }                                                                             \
  } while (0)

// A running context of one body on a stream of the given device, the workspace in
// host memory.
struct Ctx {
  lbib_ctx* h = nullptr;
  char* ws = nullptr;
  int nx, ny, nv;

  explicit Ctx(hipStream_t s) : Ctx(64, 32, 20, s, 0.0) {}
  Ctx(int nx_, int ny_, int nv_, int device, int k = 0, double repulsion = 0.0)
      : Ctx(nx_, ny_, nv_, fake::stream_of(device, k), repulsion) {}
  Ctx(int nx_, int ny_, int nv_, hipStream_t stream, double repulsion) : nx(nx_), ny(ny_), nv(nv_) {
    lbib_lattice_desc d;
    std::memset(&d, 0, sizeof(d));
    d.nx = nx;
    d.ny = ny;
    d.tau = 1.0;
    CHECK(lbib_create(&d, &h) == LBIB_OK);
    lbib_body_desc b;
    std::memset(&b, 0, sizeof(b));
    b.kind = LBIB_PARTICLE_RIGID;
    b.nv = nv;
    b.density_ratio = 1.1;
    std::vector<double> xy(2 * nv);
    for (int k = 0; k < nv; ++k) {
      xy[2 * k] = 0.5 * nx + 6.0 * __builtin_cos(2 * 3.14159265358979 * k / nv);
      xy[2 * k + 1] = 0.5 * ny + 6.0 * __builtin_sin(2 * 3.14159265358979 * k / nv);
    }
    CHECK(lbib_add_body(h, &b, xy.data(), nullptr) == LBIB_OK);
    CHECK(lbib_set_repulsion(h, repulsion, 2.0) == LBIB_OK);
    size_t n = 0;
    CHECK(lbib_workspace_query(h, &n) == LBIB_OK);
    CHECK(posix_memalign((void**)&ws, 256, n) == 0);
    std::memset(ws, 0x5a, n);
    CHECK(lbib_bind(h, ws, n, stream) == LBIB_OK);
    CHECK(lbib_finalize_setup(h) == LBIB_OK);
  }
  void close() {
    CHECK(lbib_destroy(h) == LBIB_OK);
    std::free(ws);
  }
  void read_all() {
    const size_t N = (size_t)nx * ny;
    std::vector<double> r(N), u(N), v(N), xy(2 * nv);
    CHECK(lbib_get_fields(h, r.data(), u.data(), v.data()) == LBIB_OK);
    CHECK(lbib_get_markers(h, 0, xy.data()) == LBIB_OK);
    CHECK(lbib_get_marker_forces(h, 0, xy.data()) == LBIB_OK);
    lbib_diag d;
    CHECK(lbib_diagnostics(h, &d) == LBIB_OK);
    CHECK(state().size() > 0);
  }
  std::vector<char> state() {
    size_t n = 0;
    CHECK(lbib_get_state(h, nullptr, &n) == LBIB_OK);
    std::vector<char> s(n, 0x11);
    CHECK(lbib_get_state(h, s.data(), &n) == LBIB_OK);
    return s;
  }
};

// A context on a stream of device 1 while device 0 is current.
static void device() {
  fake::current = 0;
  Ctx c(200, 90, 40, 1);
  c.read_all();
  CHECK(fake::current == 0);
  fake::current = 1;
  Ctx d(64, 32, 20, 0);
  d.read_all();
  c.read_all();
  CHECK(fake::current == 1);
  // a stream whose device the runtime does not tell: the current device's
  fake::unknown_stream = true;
  fake::current = 0;
  d.read_all();
  CHECK(hipGetLastError() == hipSuccess);
  fake::unknown_stream = false;
  // the null stream, the legacy and the per-thread one
  for (uintptr_t h = 0; h < 3; ++h) {
    Ctx e((hipStream_t)h);
    e.read_all();
    e.close();
  }
  c.close();
  d.close();
}

// Closing a context frees no pinned memory (that waits for all streams of the
// device) while another is open; of what the readbacks of the last one used,
// 2 MB stay for the next.
static void close_one() {
  fake::current = 0;
  for (int round = 0; round < 3; ++round) {
    Ctx a(200, 90, 40, 0, 0), b(64, 32, 20, 0, 1), c(300, 100, 30, 0, 2);
    a.read_all();
    b.read_all();
    c.read_all();
    a.close();
    b.close();
    CHECK(fake::frees == 0);
    c.close();
    size_t held = 0;
    for (auto& m : fake::pinned) held += m.second;
    CHECK(held <= (2u << 20));
  }
}

// Contexts on threads of their own, more than there are rings: right data, at
// most 8 MB pinned at a time.
static void threads() {
  fake::current = 0;
  fake::wait_us = 300;
  constexpr int n = 12;
  std::vector<Ctx> cs;
  std::vector<std::vector<char>> want;
  for (int k = 0; k < n; ++k) {
    cs.emplace_back(180 + 7 * k, 80, 24 + k, 0, k);
    want.push_back(cs[k].state());
  }
  CHECK(want[0] != want[1]);
  std::vector<std::thread> ts;
  for (int k = 0; k < n; ++k)
    ts.emplace_back([&, k] {
      for (int i = 0; i < 15; ++i) {
        CHECK(cs[k].state() == want[k]);
        cs[k].read_all();
      }
    });
  for (auto& t : ts) t.join();
  size_t held = 0;
  for (auto& m : fake::pinned) held += m.second;
  CHECK(held <= (8u << 20));
  for (auto& c : cs) c.close();
  held = 0;
  for (auto& m : fake::pinned) held += m.second;
  CHECK(held <= (2u << 20));
}

// Pinned memory refused, then granted.
static void refused() {
  fake::current = 0;
  fake::refuse_malloc = 1000;
  Ctx a(200, 90, 40, 0);
  const std::vector<char> direct = a.state();
  a.read_all();
  CHECK(fake::pinned.empty());
  CHECK(hipGetLastError() == hipSuccess);
  fake::refuse_malloc = 0;
  Ctx b(200, 90, 40, 0, 1);
  CHECK(b.state() == direct);
  a.close();
  b.close();
}

// A copy that fails leaves nothing under way that would still write to the ring.
static void failed() {
  fake::current = 0;
  Ctx a(700, 300, 40, 0);
  const std::vector<char> want = a.state();
  for (int k : {1, 2, 5, 9}) {
    std::vector<char> s(want.size());
    size_t n = 0;
    CHECK(lbib_get_state(a.h, nullptr, &n) == LBIB_OK);
    fake::fail_copy = k;
    CHECK(lbib_get_state(a.h, s.data(), &n) == LBIB_EHIP);
    CHECK(hipGetLastError() != hipSuccess);
    const fake::Stream& q = fake::streams[fake::stream_of(0)];
    CHECK(q.done == q.issued);
    CHECK(a.state() == want);
  }
  a.close();
}

// An error that a call of the program's own left behind is not the marker
// read's, and stays for the program to see.
static void stale_error() {
  fake::current = 0;
  Ctx a(64, 32, 20, 0);
  std::vector<double> xy(40);
  CHECK(hipSetDevice(7) != hipSuccess);
  CHECK(lbib_get_markers(a.h, 0, xy.data()) == LBIB_OK);
  CHECK(lbib_get_marker_forces(a.h, 0, xy.data()) == LBIB_OK);
  CHECK(hipGetLastError() == hipErrorInvalidDevice);
  fake::refuse_launch = 1;
  CHECK(lbib_get_markers(a.h, 0, xy.data()) == LBIB_EHIP);
  (void)hipGetLastError();
  CHECK(lbib_get_markers(a.h, 0, xy.data()) == LBIB_OK);
  a.close();
}

// A state blob in pinned memory is written by the copy engine itself.
static void pinned_blob() {
  fake::current = 0;
  Ctx a(700, 300, 40, 0);
  const std::vector<char> want = a.state();
  std::vector<char> s(want.size());
  size_t n = 0;
  CHECK(lbib_get_state(a.h, nullptr, &n) == LBIB_OK);
  for (bool pinned : {true, false}) {
    if (pinned) fake::user_pinned.insert(s.data());
    else fake::user_pinned.clear();
    std::fill(s.begin(), s.end(), 0);
    fake::d2h.clear();
    CHECK(lbib_get_state(a.h, s.data(), &n) == LBIB_OK);
    CHECK(s == want);
    size_t direct = 0;
    for (auto& d : fake::d2h)
      if (d.first >= s.data() && d.first < s.data() + s.size()) direct += d.second;
    CHECK(pinned ? direct > 0.99 * n : direct == 0);
  }
  a.close();
}

// What lbib_get_step_mode answers for each mode asked for: the name that the
// form of that mode has had throughout (automatic: 2 where 2 is possible).
static void modes() {
  fake::current = 0;
  Ctx small(64, 32, 512, 0), large(64, 32, 513, 0), crowd(64, 32, 40, 0, 0, 1e-5);
  const struct {
    Ctx* c;
    int want[4];
  } rows[] = {{&small, {2, 1, 2, 3}}, {&large, {1, 1, 1, 3}}, {&crowd, {1, 1, 1, 3}}};
  for (auto& r : rows) {
    int32_t got = -1;
    CHECK(lbib_get_step_mode(r.c->h, &got) == LBIB_OK && got == r.want[0]);
    for (int m : {3, 1, 2, 0}) {
      CHECK(lbib_set_step_mode(r.c->h, m) == LBIB_OK);
      CHECK(lbib_get_step_mode(r.c->h, &got) == LBIB_OK && got == r.want[m]);
    }
    r.c->close();
  }
}

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "device") device();
  else if (what == "close") close_one();
  else if (what == "threads") threads();
  else if (what == "refused") refused();
  else if (what == "failed") failed();
  else if (what == "error") stale_error();
  else if (what == "pinned") pinned_blob();
  else if (what == "modes") modes();
  else return 2;
  std::puts("ok");
  return 0;
}
