// The host driver with its kernels replaced by what a test makes them do
// (hip/hip_runtime.h beside this file).  One check per command-line argument.
#include "dpo_host.hip"

#include <cstdio>

namespace dpo {
const void* parent_kernel_ptr(int, int, bool) { return fake::kernel("parent"); }
const void* child_kernel_ptr(int, bool, bool) { return fake::kernel("child"); }
const void* serial_kernel_ptr(int p, int g, bool) {
  return p == PROB_BFS || g == AGG_FLAT ? nullptr : fake::kernel("serial");
}
const void* harvest_kernel_ptr(int, bool) { return fake::kernel("harvest"); }
const void* init_kernel_ptr(int) { return fake::kernel("init"); }
const void* narrow_kernel_ptr(int32_t) { return fake::kernel("narrow"); }
const void* near_kernel_ptr() { return fake::kernel("near"); }
const void* solo_kernel_ptr(bool) { return fake::kernel("solo"); }
const void* symmetry_kernel_ptr(bool) { return fake::kernel("symmetry"); }
const void* bottom_up_kernel_ptr() { return fake::kernel("bottom_up"); }
const void* tally_kernel_ptr() { return fake::kernel("tally"); }
const void* bottom_up_words_kernel_ptr() { return fake::kernel("words"); }
const void* bottom_up_queries_kernel_ptr() { return fake::kernel("bottom_up_queries"); }
const void* clear_tally_kernel_ptr() { return fake::kernel("clear_tally"); }
const void* settle_symmetry_kernel_ptr() { return fake::kernel("settle"); }
const void* start_kernel_ptr(int) { return fake::kernel("start"); }
const void* admit_kernel_ptr(int) { return fake::kernel("admit"); }
const void* admit_sources_kernel_ptr() { return fake::kernel("admit_sources"); }
const void* retire_kernel_ptr() { return fake::kernel("retire"); }
const void* clear_found_kernel_ptr() { return fake::kernel("clear_found"); }
const void* advance_kernel_ptr() { return fake::kernel("advance"); }
}  // namespace dpo

using namespace dpo;

static int failures = 0;
#define CHECK(x) \
  do { \
    if (!(x)) { \
      printf("%s:%d: %s\n", __FILE__, __LINE__, #x); \
      ++failures; \
    } \
  } while (0)

static fake::Runtime& F = fake::rt();

// A narrow kernel that posts the given verdicts one after the other.
static void post_in_turn(std::vector<uint32_t> codes) {
  auto left = std::make_shared<std::deque<uint32_t>>(codes.begin(), codes.end());
  F.kernels["narrow"] = [left](void** p) -> std::function<void()> {
    const uint32_t ticket = *(uint32_t*)p[2];
    uint32_t* verdict = *(uint32_t**)p[3];
    State* st = ((Args*)p[0])->st;
    return [=] {
      const uint32_t code = left->front();
      left->pop_front();
      st->plan = code;
      st->done = code == V_DONE;
      if (verdict) *verdict = ticket << 8 | code;
    };
  };
}

struct Single {
  std::vector<int32_t> rp, col;
  std::vector<uint32_t> w, out;
  std::vector<char> ws;
  dpo_options o;
  dpo_csr g;
  Single(int32_t n, int32_t m) : rp(n + 1), col(m), w(m, 1), out(n) {
    dpo_default_options(&o);
    g = dpo_csr{n, m, rp.data(), col.data(), w.data()};
    ws.resize(dpo_workspace_bytes(&g, &o));
  }
  dpo_status bfs() {
    return dpo_bfs(&g, 0, &o, (int32_t*)out.data(), ws.data(), ws.size(), nullptr, nullptr);
  }
  dpo_status sssp() { return dpo_sssp(&g, 0, &o, out.data(), ws.data(), ws.size(), nullptr, nullptr); }
};

// The verdict of a solo (near-far) SSSP stays in the word the narrow kernel's
// verdicts are polled in; no later traversal may take it for its own, whatever
// the launch ticket has come to.
static void stale_verdict(const char* kernel, int32_t n, int32_t m) {
  Single s(n, m);
  F.kernels[kernel] = [=](void** p) -> std::function<void()> {
    uint32_t* verdict = *(uint32_t**)p[strcmp(kernel, "near") ? 3 : 2];
    return [=] { *verdict = V_DONE; };
  };
  CHECK(s.sssp() == DPO_OK);
  CHECK(F.launched[kernel] == 1);
  rt().ticket = 0xFFFFFF;
  post_in_turn({V_TOP_DOWN, V_DONE});
  CHECK(s.bfs() == DPO_OK);
  CHECK(F.launched["narrow"] == 2);
  CHECK(F.launched["parent"] == 1);
}

// Launches that post nothing leave a verdict behind whose ticket comes round.
static void stale_verdict_unposted() {
  Single s(100, 10);
  post_in_turn({V_DONE});
  CHECK(s.bfs() == DPO_OK);  // posts ticket t
  const uint32_t t = rt().ticket;
  post_in_turn({V_DONE});
  CHECK(dpo_bfs_noalloc(&s.g, 0, &s.o, (int32_t*)s.out.data(), nullptr) == DPO_OK);
  rt().ticket = t - 1;  // as 2^24 - 2 more of them would
  post_in_turn({V_TOP_DOWN, V_DONE});
  CHECK(s.bfs() == DPO_OK);
  CHECK(F.launched["parent"] == 1);
}

// A run of wide levels takes as many level steps at a time as it has had;
// a narrow or bottom-up level in between ends the run.
static void wide_run(bool noalloc) {
  Single s(5000, 10);
  auto after = std::make_shared<std::vector<uint32_t>>();
  const std::vector<uint32_t> codes = {V_STILL, V_STILL, V_STILL, V_STILL, V_STILL, V_STILL, V_TOP_DOWN,
                                       V_STILL, V_BOTTOM_UP, 0, V_STILL, V_STILL, V_DONE};
  post_in_turn(codes);
  auto post = F.kernels["narrow"];
  F.kernels["narrow"] = [=](void** p) {
    after->push_back(*(uint32_t*)p[1]);
    return post(p);
  };
  auto steps = std::make_shared<std::vector<uint32_t>>();
  F.kernels["parent"] = [=](void** p) -> std::function<void()> {
    steps->push_back(*(uint32_t*)p[1]);
    return nullptr;
  };
  CHECK((noalloc ? dpo_bfs_noalloc(&s.g, 0, &s.o, (int32_t*)s.out.data(), nullptr) : s.bfs()) == DPO_OK);
  const uint32_t B = AFTER_BOTTOM_UP;
  CHECK((*after == std::vector<uint32_t>{0, 1, 1, 2, 4, 8, 16, 1, 1, B, B, 1, 1}));
  std::vector<uint32_t> expected;
  for (uint32_t k : {1, 1, 2, 4, 8, 16, 1, 1, 1, 1})
    for (uint32_t i = 0; i < k; ++i) expected.push_back(i);
  CHECK(*steps == expected);
}

// An engine over graphs of the given sizes whose replays end every query.
struct Served {
  std::vector<int32_t> vbase, rp, col;
  std::vector<uint32_t> w;
  std::vector<char> ws, out_arena;
  std::vector<std::vector<uint32_t>> outs;
  dpo_options o;
  dpo_arena ar;
  dpo_engine* e = nullptr;
  Served(std::vector<int32_t> sizes, int32_t m, int kind, int64_t slots = 1 << 16) : vbase{0}, col(m), w(m, 1) {
    for (int32_t n : sizes) vbase.push_back(vbase.back() + n);
    rp.resize(vbase.back() + 1);
    dpo_default_options(&o);
    o.steps_per_replay = 2;
    ar = dpo_arena{(int32_t)sizes.size(), vbase.data(), {vbase.back(), m, rp.data(), col.data(), w.data()}};
    ws.resize(dpo_engine_workspace_bytes(&o, 64, slots));
    out_arena.resize(slots * 4);
    for (int64_t i = 0; i < slots; ++i) ((uint32_t*)out_arena.data())[i] = (uint32_t)i + 1000;
    F.kernels["advance"] = [](void** p) -> std::function<void()> {
      uint32_t* flags = *(uint32_t**)p[2];
      return [=] {
        flags[0] += 2;
        flags[1] = 1;
      };
    };
    F.kernels["retire"] = [](void** p) -> std::function<void()> {
      const uint32_t* from = *(const uint32_t**)p[0];
      const uint4* list = *(const uint4**)p[1];
      const int32_t count = *(int32_t*)p[3];
      return [=] {
        for (int32_t k = 0; k < count; ++k)
          memcpy((void*)((uint64_t)list[k].y << 32 | list[k].x), from + list[k].z, (size_t)list[k].w * 4);
      };
    };
    CHECK(dpo_engine_create(&ar, kind, &o, 1, nullptr, 64, slots, ws.data(), ws.size(), out_arena.data(), nullptr,
                            &e) == DPO_OK);
  }
  uint64_t submit(int32_t graph) {
    outs.emplace_back(vbase[graph + 1] - vbase[graph], 7u);
    uint64_t t = 0;
    CHECK(dpo_engine_submit(e, graph, 0, outs.back().data(), &t) == DPO_OK);
    return t;
  }
  std::vector<uint64_t> poll() {
    uint64_t t[64];
    const int32_t k = dpo_engine_poll(e, t, 64);
    return std::vector<uint64_t>(t, t + k);
  }
  ~Served() { dpo_engine_destroy(e); }
};

// A step whose copy of finished results fails reports no ticket; the results are
// copied by the next step that can.
static void failed_copy() {
  Served s({40, 100}, 300, 1);
  s.outs.reserve(8);
  s.submit(0);
  s.submit(1);
  int32_t running = 0, pending = 0;
  CHECK(dpo_engine_step(s.e, &running, &pending) == DPO_OK && running == 2);
  F.fail_launch = "retire";
  CHECK(dpo_engine_step(s.e, &running, &pending) == DPO_ERR_HIP);
  CHECK(s.poll().empty());
  CHECK(running == 2);
  F.fail_launch = "";
  CHECK(dpo_engine_step(s.e, &running, &pending) == DPO_OK && running == 0);
  CHECK(s.poll().size() == 2);
  for (auto& out : s.outs)
    for (size_t i = 0; i < out.size(); ++i) CHECK(out[i] == out[0] + i && out[i] >= 1000);
}

// Results whose array a kernel on the engine's device may not store to (another
// device's, the host's, not at a word's boundary) are copied, beside those that
// the kernel stores.
static void foreign_outputs() {
  Served s({40, 100, 33, 70, 64}, 300, 0);
  std::vector<uint32_t> far(40, 7u), host(100, 7u), own(64, 7u), managed(70, 7u);
  std::vector<char> odd(33 * 4 + 1, 7);
  F.attributes[far.data()] = {hipMemoryTypeDevice, 1};
  F.attributes[host.data()] = {hipMemoryTypeHost, 0};
  F.attributes[managed.data()] = {hipMemoryTypeManaged, 0};
  void* outs[5] = {far.data(), host.data(), odd.data() + 1, managed.data(), own.data()};
  for (int k = 0; k < 5; ++k) {
    uint64_t t;
    CHECK(dpo_engine_submit(s.e, k, 0, outs[k], &t) == DPO_OK);
  }
  for (int i = 0; i < 2; ++i) CHECK(dpo_engine_step(s.e, nullptr, nullptr) == DPO_OK);
  CHECK(s.poll().size() == 5);
  CHECK(F.copies["device"] == 4);
  CHECK(F.launched["retire"] == 1);
  for (int k = 0; k < 5; ++k) {
    uint32_t first, v;
    memcpy(&first, outs[k], 4);
    CHECK(first >= 1000);
    for (int32_t i = 0; i < s.vbase[k + 1] - s.vbase[k]; ++i) {
      memcpy(&v, (char*)outs[k] + 4 * i, 4);
      CHECK(v == first + (uint32_t)i);
    }
  }
}

static void answer_symmetry(uint32_t code) {
  F.kernels["settle"] = [=](void** p) -> std::function<void()> {
    const uint32_t ticket = *(uint32_t*)p[1];
    uint32_t* verdict = *(uint32_t**)p[2];
    return [=] { *verdict = ticket << 8 | code; };
  };
}

// A large batch asks for its arena's symmetry and runs the level steps with
// bottom-up nodes only if the answer is yes.
static void batch_symmetry(bool symmetric) {
  const int32_t n = 1000, m = 1 << 20, nq = 25;
  std::vector<int32_t> vbase{0, n}, rp(n + 1), col(m), out((size_t)round32(n) * nq);
  dpo_arena ar{1, vbase.data(), {n, m, rp.data(), col.data(), nullptr}};
  std::vector<dpo_query> q(nq, dpo_query{0, 0, 0});
  dpo_options o;
  dpo_default_options(&o);
  std::vector<char> ws(dpo_batch_workspace_bytes(&ar, q.data(), nq, &o));
  answer_symmetry(symmetric ? V_BOTTOM_UP : V_TOP_DOWN);
  F.kernels["advance"] = [](void** p) -> std::function<void()> {
    uint32_t* flags = *(uint32_t**)p[2];
    return [=] { flags[1] = 1; };
  };
  CHECK(dpo_bfs_batch(&ar, q.data(), nq, &o, 1, out.data(), ws.data(), ws.size(), nullptr, nullptr) == DPO_OK);
  CHECK(F.launched["symmetry"] == 1 && F.launched["settle"] == 1);
  CHECK(F.launched["parent"] == kBatchSteps && F.launched["harvest"] == kBatchSteps);
  for (const char* k : {"tally", "words", "bottom_up_queries"}) CHECK(F.launched[k] == (symmetric ? kBatchSteps : 0));
}

// A batch's replays by default: short ones, two at a time from the third on, on a
// dense graph; long ones on a sparse one, or as the options say.
static void batch_replays() {
  const int32_t n = 1000;
  std::vector<int32_t> vbase{0, n}, rp(n + 1), col(1 << 14), out(1024);
  std::vector<uint32_t> w(1 << 14);
  dpo_query q{0, 0, 0};
  struct { int32_t m, steps, k, at_once; } forms[] = {{1 << 14, 0, 8, 2}, {2000, 0, 16, 1}, {1 << 14, 8, 8, 1}, {1 << 14, 4, 4, 1}};
  for (auto& f : forms) {
    dpo_arena ar{1, vbase.data(), {n, f.m, rp.data(), col.data(), w.data()}};
    dpo_options o;
    dpo_default_options(&o);
    o.steps_per_replay = f.steps;
    std::vector<char> ws(dpo_batch_workspace_bytes(&ar, &q, 1, &o));
    auto ends = std::make_shared<int>(0);  // replays run
    F.kernels["advance"] = [=](void** p) -> std::function<void()> {
      uint32_t* flags = *(uint32_t**)p[2];
      return [=] { flags[1] = ++*ends >= 5; };
    };
    F.launched.clear();
    CHECK(dpo_sssp_batch(&ar, &q, 1, &o, 1, (uint32_t*)out.data(), ws.data(), ws.size(), nullptr, nullptr) == DPO_OK);
    CHECK(F.launched["advance"] == (f.at_once == 2 ? 6 : 5));  // 1, 1, 2, 2
    CHECK(F.launched["parent"] == F.launched["advance"] * f.k);
    std::lock_guard<std::mutex> lock(rt().mu);
    rt().graphs.clear();  // their nodes keep this form's counter
  }
}

// An engine's replays have bottom-up nodes while its running queries are enough
// work, whatever it has served before, and none once its arena is known to be
// asymmetric.
static void engine_symmetry(bool symmetric) {
  Served s({1000, 200000}, 25 << 20, 0, 1 << 20);
  s.outs.reserve(64);
  answer_symmetry(symmetric ? V_BOTTOM_UP : V_TOP_DOWN);
  // queries of the first graph end with their second replay, of the second with
  // their third
  Query* table = s.e->sr.a.q;
  uint32_t* flags = s.e->hflags;
  const auto end_small = [=] {
    for (int32_t q = 0; q < 64; ++q)
      if (++table[q].lstart < (table[q].n > 1000 ? 3 : 2)) table[q].last = (int32_t)flags[0] - 1;
      else table[q].last = -1;
    flags[1] = 0;
  };
  s.e->exec->nodes.push_back({"end", end_small});
  if (s.e->plain) s.e->plain->nodes.push_back({"end", end_small});
  auto step = [&] {
    const int before = F.launched["tally"];
    CHECK(dpo_engine_step(s.e, nullptr, nullptr) == DPO_OK);
    return F.launched["tally"] - before;
  };
  s.submit(0);
  CHECK(step() == 0 && F.launched["symmetry"] == 0);  // too little work
  s.submit(1);
  s.submit(0);
  CHECK(step() == 2 && F.launched["symmetry"] == 1);
  CHECK(F.launched["clear_tally"] == 0);
  s.submit(0);
  CHECK(step() == (symmetric ? 2 : 0));
  s.submit(0);
  CHECK(step() == (symmetric ? 2 : 0));
  for (int i = 0; i < 30; ++i) {  // the large one has ended: a trickle of small ones, never idle
    s.submit(0);
    CHECK(step() == 0);
  }
  s.submit(1);
  s.submit(0);
  CHECK(step() == (symmetric ? 2 : 0));
  CHECK(F.launched["clear_tally"] == (symmetric ? 1 : 0));
  CHECK(F.launched["symmetry"] == 1);
  for (int i = 0; i < 5; ++i) step();
}

int main(int argc, char** argv) {
  const std::string name = argc > 1 ? argv[1] : "";
  if (name == "stale_solo") stale_verdict("solo", 100, 200);
  else if (name == "stale_near") stale_verdict("near", 20000, 40000);
  else if (name == "stale_unposted") stale_verdict_unposted();
  else if (name == "wide_run") wide_run(false);
  else if (name == "wide_run_noalloc") wide_run(true);
  else if (name == "batch_replays") batch_replays();
  else if (name == "batch_symmetric") batch_symmetry(true);
  else if (name == "batch_directed") batch_symmetry(false);
  else if (name == "engine_symmetric") engine_symmetry(true);
  else if (name == "engine_directed") engine_symmetry(false);
  else if (name == "failed_copy") failed_copy();
  else if (name == "foreign_outputs") foreign_outputs();
  else { printf("no check %s\n", name.c_str()); return 2; }
  if (!failures) printf("ok\n");
  return failures != 0;
}
