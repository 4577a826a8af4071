// Host checks of what the C ABI asks of the device: tables and memory, what
// runs while a stream is captured, which kernels a call launches.  No kernel
// runs (fake_device.hpp).
// Usage: device_calls_check SCENARIO
#include <cstring>
#include <functional>

#include "atlas_nabla.h"
#include "fake_device.hpp"

static int bad = 0;
#define EXPECT(c)                                                                       \
  do {                                                                                  \
    if (!(c)) {                                                                         \
      ++bad;                                                                            \
      std::printf("line %d: %s (last error: %s)\n", __LINE__, #c, atlas_last_error());  \
    }                                                                                   \
  } while (0)

// fields at made-up device addresses, far apart
static void* field(int k) { return reinterpret_cast<void*>((uintptr_t(k) + 1) << 44); }
static hipStream_t stream(int k) { return reinterpret_cast<hipStream_t>(uintptr_t(0x100 + k)); }

struct Mesh {
  atlas_mesh_t h = nullptr;
  int64_t V = 0;
  explicit Mesh(const char* grid) {
    EXPECT(atlas_mesh_build(grid, 6371220.0, 0, &h) == ATLAS_OK);
    EXPECT(atlas_mesh_sizes(h, &V, nullptr, nullptr, nullptr, nullptr, nullptr) == ATLAS_OK);
  }
  ~Mesh() { atlas_mesh_free(h); }
};

// Columns of 8 to 32 levels of a field of 2.6 million values take the tiles;
// where memory is short they run on the gather, and what they could not
// complete is given back and not tried again.
static void short_columns_out_of_memory() {
  Mesh m("O200");
  const int L = 19;
  EXPECT(atlas_nabla_gradient(m.h, ATLAS_F32, 3, field(0), field(1), nullptr) == ATLAS_OK);   // the gather's order
  const size_t held = dev().live;
  // room for some of the tiling's tables and for all but the records
  for (size_t room : {size_t(1) << 20, size_t(8) * m.V, size_t(60) * m.V}) {
    Mesh n("O200");
    EXPECT(atlas_nabla_gradient(n.h, ATLAS_F32, 3, field(0), field(1), nullptr) == ATLAS_OK);
    const size_t before = dev().live;
    dev().limit = before + room;
    dev().launches.clear();
    EXPECT(atlas_nabla_gradient(n.h, ATLAS_F32, L, field(0), field(1), nullptr) == ATLAS_OK);
    EXPECT(dev().refused > 0 && dev().count("k_op<") == 1 && dev().count("k_tile<") == 0);
    EXPECT(dev().live == before);
    const int asked = dev().mallocs;
    for (int i = 0; i < 3; ++i)
      EXPECT(atlas_nabla_gradient(n.h, ATLAS_F32, L, field(0), field(1), nullptr) == ATLAS_OK);
    EXPECT(dev().mallocs == asked && dev().live == before && dev().count("k_op<") == 4);
    dev().limit = SIZE_MAX;
    dev().refused = 0;
    // another operator is not held back by it
    EXPECT(atlas_nabla_divergence(n.h, ATLAS_F32, L, field(0), field(2), nullptr) == ATLAS_OK);
    EXPECT(dev().count("k_tile<") == 1);
  }
  EXPECT(dev().live == held);
  // long columns: an error, as ever, and nothing kept of the attempt
  dev().limit = held + 60 * m.V;
  for (int i = 0; i < 3; ++i)
    EXPECT(atlas_nabla_gradient(m.h, ATLAS_F32, 60, field(0), field(1), nullptr) == ATLAS_ENOMEM);
  EXPECT(dev().live == held);
  dev().limit = SIZE_MAX;
  EXPECT(atlas_nabla_gradient(m.h, ATLAS_F32, 60, field(0), field(1), nullptr) == ATLAS_OK);
}

// After one call on short columns, whichever path it took, calls of other
// short columns and operators can be captured: those without tiles of their
// own record the gather, whose node order is there.
static void short_columns_captured() {
  for (int warm : {3, 19}) {
    Mesh m("O200");
    EXPECT(atlas_nabla_gradient(m.h, ATLAS_F32, warm, field(0), field(1), nullptr) == ATLAS_OK);
    dev().launches.clear();
    dev().here.insert(stream(1));
    for (int L : {7, 18, 20}) {
      EXPECT(atlas_nabla_gradient(m.h, ATLAS_F32, L, field(0), field(1), stream(1)) == ATLAS_OK);
      EXPECT(atlas_nabla_divergence_curl(m.h, ATLAS_F64, L, field(0), field(2), field(3), stream(1)) == ATLAS_OK);
    }
    EXPECT(dev().count("k_op<") == 9 && dev().launches.size() == 9 && dev().broken == 0);
    dev().here.clear();
  }
}

// First calls of short columns while another thread captures a stream in the
// global mode, or this thread another stream: nothing they ask for may break
// that capture, and the tiles are built.
static void short_columns_beside_a_capture() {
  for (int whose = 0; whose < 2; ++whose) {
    Mesh m("O200");
    EXPECT(atlas_nabla_gradient(m.h, ATLAS_F32, 3, field(0), field(1), nullptr) == ATLAS_OK);
    dev().launches.clear();
    if (whose == 0) dev().elsewhere = true;
    else dev().here.insert(stream(1));
    for (int L : {18, 20}) {
      EXPECT(atlas_nabla_gradient(m.h, ATLAS_F32, L, field(0), field(1), stream(2)) == ATLAS_OK);
      EXPECT(atlas_nabla_gradient(m.h, ATLAS_F32, L, field(0), field(1), nullptr) == ATLAS_OK);
    }
    EXPECT(dev().count("k_tile<") == 4 && dev().broken == 0 && dev().mode == hipStreamCaptureModeGlobal);
    dev().elsewhere = false;
    dev().here.clear();
  }
}

// What short columns keep of tables grows with the level counts in use, up to
// a sixteenth of the device's memory a mesh; further ones run on the gather,
// the ones that have tables keep them.
static void short_columns_table_budget() {
  dev().total = size_t(1) << 30;
  Mesh m("O200");
  EXPECT(atlas_nabla_gradient(m.h, ATLAS_F32, 3, field(0), field(1), nullptr) == ATLAS_OK);
  const size_t held = dev().live;
  int tiles = 0;
  for (int pass = 0; pass < 2; ++pass) {
    dev().launches.clear();
    for (int L = 16; L <= 32; ++L)
      EXPECT(atlas_nabla_gradient(m.h, ATLAS_F32, L, field(0), field(1), nullptr) == ATLAS_OK);
    if (pass == 0) tiles = dev().count("k_tile<");
    EXPECT(tiles > 1 && tiles < 17 && dev().count("k_tile<") == tiles && dev().count("k_op<") == 17 - tiles);
    // the table that reaches the bound is the last
    const size_t kept = dev().live - held, one = kept / tiles;
    EXPECT(kept >= dev().total / 16 && kept <= dev().total / 16 + 2 * one);
  }
  // long columns have no such bound
  for (int L = 60; L < 64; ++L)
    EXPECT(atlas_nabla_gradient(m.h, ATLAS_F32, L, field(0), field(1), nullptr) == ATLAS_OK);
  EXPECT(dev().count("k_win<") == 0);
}

struct Plan {
  atlas_batch_t h = nullptr;
  int rc = 0;
  Plan(const Mesh& m, std::vector<int> levels, const atlas_tune_t* tune = nullptr, int dtype = ATLAS_F32,
       uint32_t ops = 0xF) {
    std::vector<atlas_tracer_desc_t> d(levels.size());
    for (size_t t = 0; t < d.size(); ++t) {
      d[t].nlev = levels[t];
      // field, wind, and an output of each operator
      d[t].in[0] = d[t].in[3] = field(10 * (int)t);
      d[t].in[1] = d[t].in[2] = field(10 * (int)t + 1);
      for (int o = 0; o < 4; ++o) d[t].out[o] = field(10 * (int)t + 2 + o);
    }
    rc = atlas_batch_create(m.h, dtype, d.data(), (int)d.size(), ops, tune, &h);
  }
  ~Plan() { atlas_batch_free(h); }
};

// A plan of large fields whose field launches' tables (one set a level count)
// do not fit takes the persistent form, whose tracers share tilings; what was
// built for the other is given back.
static void plan_out_of_memory() {
  const std::vector<int> levels = {130, 132, 133, 134, 135, 136, 137};
  size_t fields, shared;
  {
    Mesh m("O200");
    const size_t held = dev().live;
    Plan p(m, levels);
    EXPECT(p.rc == ATLAS_OK && atlas_batch_run(p.h, nullptr) == ATLAS_OK);
    EXPECT(dev().count("k_tile<") == 3 * 7 && dev().count("k_tile_batched<") == 0);
    fields = dev().live - held;
  }
  {
    Mesh m("O200");
    const size_t held = dev().live;
    atlas_tune_t t{};
    t.batch_mode = 1;
    Plan p(m, levels, &t);
    EXPECT(p.rc == ATLAS_OK);
    shared = dev().live - held;
  }
  EXPECT(shared < fields / 2);
  Mesh m("O200");
  const size_t held = dev().live;
  dev().limit = held + shared + shared / 4;
  {
    dev().launches.clear();
    Plan p(m, levels);
    EXPECT(p.rc == ATLAS_OK && dev().refused > 0);
    EXPECT(dev().live - held == shared);
    const int asked = dev().mallocs;
    EXPECT(atlas_batch_run(p.h, nullptr) == ATLAS_OK);
    EXPECT(dev().count("k_tile_batched<") == 3 && dev().count("k_tile<") == 0 && dev().mallocs == asked);
  }
  // neither fits
  dev().limit = SIZE_MAX;
  Mesh n("O200");
  dev().limit = dev().live + shared / 2;
  Plan p(n, levels);
  EXPECT(p.rc == ATLAS_ENOMEM);
  // what its short columns went without they are not denied later
  dev().limit = dev().live + (size_t(1) << 20);
  Plan q(n, {19, 300});
  EXPECT(q.rc == ATLAS_ENOMEM);
  dev().limit = SIZE_MAX;
  dev().launches.clear();
  EXPECT(atlas_nabla_gradient(n.h, ATLAS_F32, 19, field(0), field(1), nullptr) == ATLAS_OK);
  EXPECT(dev().count("k_tile<") == 1);
}

// A plan in the field form by request, whose operators' tables are there from
// single calls (or from tuning) but not the divergence pair's: captured, and
// short of memory, it runs the two operators; else the pair.
static void field_plan_pair() {
  for (int captured = 0; captured < 2; ++captured) {
    Mesh m("O33");
    EXPECT(atlas_nabla_divergence(m.h, ATLAS_F32, 60, field(1), field(0), nullptr) == ATLAS_OK);
    EXPECT(atlas_nabla_gradient_adjoint(m.h, ATLAS_F32, 60, field(1), field(0), nullptr) == ATLAS_OK);
    atlas_tune_t t{};
    t.batch_mode = 2;
    Plan p(m, {60, 60}, &t, ATLAS_F32, ATLAS_OP_DIVERGENCE | ATLAS_OP_GRADIENT_ADJOINT);
    EXPECT(p.rc == ATLAS_OK);
    const size_t held = dev().live;
    dev().launches.clear();
    if (captured) dev().here.insert(stream(1));
    else dev().limit = held;
    EXPECT(atlas_batch_run(p.h, stream(1)) == ATLAS_OK);
    EXPECT(dev().count("k_tile<float, 1,") == 2 && dev().count("k_tile<float, 2,") == 2 && dev().launches.size() == 4);
    EXPECT(dev().broken == 0 && dev().live == held);
    dev().here.clear();
    dev().limit = SIZE_MAX;
    dev().launches.clear();
    EXPECT(atlas_batch_run(p.h, stream(1)) == ATLAS_OK);
    EXPECT(dev().count("k_tile<float, 8,") == (captured ? 2 : 0));
  }
}

// atlas_nabla_describe names the kernel that a call launches, and the shape it
// reports, set on the mesh, keeps that kernel.
static void described_kernels() {
  struct Call {
    uint32_t code, bit;
    std::function<int(atlas_mesh_t, int, int)> run;
  };
  const auto one = [](int (*fn)(atlas_mesh_t, int, int32_t, const void*, void*, void*)) {
    return [fn](atlas_mesh_t m, int dt, int L) { return fn(m, dt, L, field(0), field(1), nullptr); };
  };
  const auto two = [](int (*fn)(atlas_mesh_t, int, int32_t, const void*, void*, void*, void*)) {
    return [fn](atlas_mesh_t m, int dt, int L) { return fn(m, dt, L, field(0), field(1), field(2), nullptr); };
  };
  const std::vector<Call> calls = {
      {ATLAS_OP_GRADIENT, ATLAS_OP_GRADIENT, one(atlas_nabla_gradient)},
      {ATLAS_OP_DIVERGENCE, ATLAS_OP_DIVERGENCE, one(atlas_nabla_divergence)},
      {ATLAS_OP_CURL_ADJOINT, ATLAS_OP_CURL_ADJOINT, one(atlas_nabla_curl_adjoint)},
      {ATLAS_OP_LAPLACIAN, ATLAS_OP_LAPLACIAN,
       [](atlas_mesh_t m, int dt, int L) { return atlas_nabla_laplacian(m, dt, L, field(0), field(1), nullptr, nullptr); }},
      {ATLAS_OP_GRADIENT_LAPLACIAN, ATLAS_OP_LAPLACIAN, two(atlas_nabla_gradient_laplacian)},
      {ATLAS_OP_DIVERGENCE_CURL, ATLAS_OP_DIVERGENCE, two(atlas_nabla_divergence_curl)},
      {ATLAS_OP_DIVERGENCE_GRADIENT_ADJOINT, ATLAS_OP_DIVERGENCE, two(atlas_nabla_divergence_gradient_adjoint)},
  };
  Mesh m("O200");
  const auto launched = [&](const Call& c, int dt, int L) {
    EXPECT(c.run(m.h, dt, L) == ATLAS_OK);   // tables
    dev().launches.clear();
    EXPECT(c.run(m.h, dt, L) == ATLAS_OK);
    return dev().launches.size() == 1 ? dev().launches[0] : std::string("two calls");
  };
  for (int dt : {ATLAS_F64, ATLAS_F32, ATLAS_BF16})
    for (int L : {7, 16, 32, 33, 96, 137, 180})
      for (const Call& c : calls) {
        char name[128];
        atlas_tune_t t{};
        EXPECT(atlas_nabla_describe(m.h, dt, c.code, L, &t, name, sizeof name) == ATLAS_OK);
        const std::string run = launched(c, dt, L);
        if (run != name) {
          ++bad;
          std::printf("op %x dtype %d x %d: %s described, %s launched\n", c.code, dt, L, name, run.c_str());
        }
        EXPECT(atlas_nabla_set_tune(m.h, dt, c.bit, &t) == ATLAS_OK);
        const std::string again = launched(c, dt, L);
        if (again != run) {
          ++bad;
          std::printf("op %x dtype %d x %d: %s, with the described shape set %s\n", c.code, dt, L, run.c_str(),
                      again.c_str());
        }
        EXPECT(atlas_nabla_set_tune(m.h, dt, c.bit, nullptr) == ATLAS_OK);
      }
}

// Orders of one-tile workgroups: shapes that ask for the form alone go around
// single bands as the library's own do, and the autotuner's sweeps of several
// bands are timed in the order that they change, a part of it per XCD.
static void tile_orders() {
  Mesh m("O33");
  for (uint32_t op : {ATLAS_OP_GRADIENT, ATLAS_OP_DIVERGENCE, ATLAS_OP_LAPLACIAN})
    for (int dt : {ATLAS_F64, ATLAS_F32, ATLAS_BF16}) {
      atlas_tune_t own{}, t{}, got{};
      EXPECT(atlas_nabla_describe(m.h, dt, op, 60, &own, nullptr, 0) == ATLAS_OK);
      t.lds_tiles = 3;
      EXPECT(atlas_nabla_set_tune(m.h, dt, op, &t) == ATLAS_OK);
      EXPECT(atlas_nabla_describe(m.h, dt, op, 60, &got, nullptr, 0) == ATLAS_OK);
      EXPECT(own.run_nodes == 1 && got.run_nodes == own.run_nodes && got.xcd_remap == own.xcd_remap);
      // a sweep that is asked for stays
      t.run_nodes = 8;
      EXPECT(atlas_nabla_set_tune(m.h, dt, op, &t) == ATLAS_OK);
      EXPECT(atlas_nabla_describe(m.h, dt, op, 60, &got, nullptr, 0) == ATLAS_OK && got.run_nodes == 8);
      EXPECT(atlas_nabla_set_tune(m.h, dt, op, nullptr) == ATLAS_OK);
    }
  atlas_tune_t best{};
  dev().orders.clear();
  EXPECT(atlas_nabla_tune(m.h, ATLAS_F32, ATLAS_OP_DIVERGENCE, 60, field(0), field(1), 1, nullptr, &best, nullptr) ==
         ATLAS_OK);
  int eighths = 0;
  for (int r : dev().orders) eighths += r == 1;
  EXPECT(eighths == 3 * 2);   // three sweeps, a warm-up launch and a timed one each
}

// Which plans run the tracers' field launches: all-default ones of at least 5 x
// 2^22 values a tracer and at most eight level counts, on default shapes
// whatever the mesh's are; with the divergence pair, where nothing overlaps.
static void plan_rule() {
  Mesh m("O200");   // 167,200 nodes: 126 levels are past 5 x 2^22
  EXPECT(m.V * 125 < 5 * (1 << 22) && m.V * 126 >= 5 * (1 << 22));
  const auto forms = [&](const std::vector<int>& levels, const atlas_tune_t* t, uint32_t ops) {
    Plan p(m, levels, t, ATLAS_F32, ops);
    dev().launches.clear();
    EXPECT(p.rc == ATLAS_OK && atlas_batch_run(p.h, nullptr) == ATLAS_OK);
    return std::make_pair(dev().count("k_tile<"), dev().count("k_tile_batched<"));
  };
  const uint32_t one = ATLAS_OP_GRADIENT;
  using P = std::pair<int, int>;
  EXPECT(forms({126, 126}, nullptr, one) == P(2, 0));
  EXPECT(forms({125, 125}, nullptr, one) == P(0, 1));
  EXPECT(forms({1, 251}, nullptr, one).second == 0);   // a mean of 126 levels
  EXPECT(forms({126, 127, 128, 129, 130, 131, 132, 133}, nullptr, one) == P(8, 0));
  EXPECT(forms({126, 127, 128, 129, 130, 131, 132, 133, 134}, nullptr, one) == P(0, 1));
  atlas_tune_t t{};
  t.tile_kb = 64;
  EXPECT(forms({126, 126}, &t, one) == P(0, 1));
  t = {};
  t.batch_mode = 1;
  EXPECT(forms({126, 126}, &t, one) == P(0, 1));
  t.batch_mode = 2;
  EXPECT(forms({5, 33}, &t, one).second == 0);
  EXPECT(forms({126, 126}, nullptr, 0xF) == P(3 * 2, 0) && dev().count("k_tile<float, 8,") == 2);
  EXPECT(forms({125, 125}, nullptr, 0xF) == P(0, 3) && dev().count("k_tile_batched<float, 8,") == 1);
  t = {};
  t.lds_tiles = 2;
  EXPECT(atlas_nabla_set_tune(m.h, ATLAS_F32, one, &t) == ATLAS_OK);
  EXPECT(forms({126, 126}, nullptr, one) == P(2, 0));
}

int main(int argc, char** argv) {
  const std::map<std::string, std::function<void()>> scenarios = {
      {"short_columns_out_of_memory", short_columns_out_of_memory},
      {"short_columns_captured", short_columns_captured},
      {"short_columns_beside_a_capture", short_columns_beside_a_capture},
      {"short_columns_table_budget", short_columns_table_budget},
      {"plan_out_of_memory", plan_out_of_memory},
      {"field_plan_pair", field_plan_pair},
      {"described_kernels", described_kernels},
      {"tile_orders", tile_orders},
      {"plan_rule", plan_rule},
  };
  if (argc != 2 || !scenarios.count(argv[1])) return 2;
  scenarios.at(argv[1])();
  std::printf(bad ? "FAILED\n" : "OK\n");
  return bad ? 1 : 0;
}
