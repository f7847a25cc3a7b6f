// team_model.cpp -- a CPU model of the bitset traversal's teams (paper §IV-A, §IV-C), for
// ThreadSanitizer and random interleavings. Test infrastructure: the library does not use it.
//
// Each std::thread plays one wavefront; `waves` of them are a team (a workgroup). Two protocols,
// with the device's atomic operations and memory orders:
//  - inside a team: `active` (sub-trees the team holds), the `idle` bits, and one box with a mail
//    flag per wavefront. A wavefront without work lowers `active` and sets its idle bit; one with
//    deferred children clears idle bits (the claim), raises `active`, fills the boxes and sets
//    their flags. `active` reads zero only when the team has finished all it took; all of its
//    wavefronts then meet at a barrier and the first one looks for work for the team;
//  - between teams: the worklist of worklist_model.cpp, with up to four nodes donated at once: one
//    reservation of m consecutive tickets, whose slots are all waited for before any of the m
//    nodes is published (the lanes of a wavefront leave such a wait together).
// A wavefront has its own bounded stack ring; pops take the newest entry, handovers and donations
// the oldest. A full ring makes room first.
//
// The trees are seeded and imbalanced (two, one or no children). Checked after every thread has
// ended: every node of every tree visited exactly once, every counter back at zero, every slot free
// for its next lap, no mail left in a box.
//
//   team_model TEAMS WAVES CAP THRESHOLD INSTANCES MAX_DEPTH STACK SEED
// exits 0 when every check holds, 1 with a message otherwise.
//
// -DVC_MODEL_MUTATION=1: a handover does not raise `active`; =2: mail flags are set with a relaxed
// store; =3: idle bits are claimed with a relaxed operation. The tests check that the checks, or
// ThreadSanitizer, notice.

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <random>
#include <thread>
#include <vector>

#ifndef VC_MODEL_MUTATION
#define VC_MODEL_MUTATION 0
#endif

namespace {

constexpr int kMaxWaves = 16;
constexpr int kDonateMost = 4;
constexpr int kDonateNodes = 4;
constexpr auto relaxed = std::memory_order_relaxed;
constexpr auto acquire = std::memory_order_acquire;
constexpr auto release = std::memory_order_release;

struct Tree {
  std::vector<int32_t> left, right;  // child indices, -1 if none
};

// Node 0 is the root; depth-first construction with a seeded generator.
Tree make_tree(uint64_t seed, int max_depth) {
  Tree t{{-1}, {-1}};
  std::mt19937_64 rng(seed);
  std::vector<std::pair<int32_t, int>> todo{{0, 0}};
  while (!todo.empty()) {
    const auto [node, depth] = todo.back();
    todo.pop_back();
    if (depth >= max_depth) continue;
    const double u = std::uniform_real_distribution<double>(0.0, 1.0)(rng);
    const int kids = u < 0.62 ? 2 : (u < 0.85 ? 1 : 0);
    for (int c = 0; c < kids; ++c) {
      const int32_t id = static_cast<int32_t>(t.left.size());
      t.left.push_back(-1);
      t.right.push_back(-1);
      (c == 0 ? t.left : t.right)[node] = id;
      todo.push_back({id, depth + 1});
    }
  }
  return t;
}

struct Node {
  int32_t inst = -1, node = 0;
};

struct Team {
  std::atomic<int32_t> active{0};
  std::atomic<uint32_t> idle{0};
  std::atomic<int32_t> mail[kMaxWaves] = {};
  Node box[kMaxWaves];
  Node taken;      // what the team's first wavefront found (plain: read after a barrier)
  int status = 0;
  std::atomic<int> arrived{0}, phase{0};
};

struct Shared {
  uint32_t cap = 0, threshold = 0;
  int32_t num_inst = 0, waves = 1, stack = 1;
  std::vector<Tree> trees;
  std::vector<std::vector<std::atomic<uint8_t>>> visited;
  std::vector<std::unique_ptr<Team>> teams;
  std::atomic<int32_t> count{0}, work{0}, root_next{0};
  std::atomic<uint64_t> head{0}, tail{0};
  std::vector<std::atomic<int32_t>> inst_work;
  std::vector<std::atomic<uint32_t>> seq;
  std::vector<Node> payload;
  std::atomic<int64_t> visits{0}, given{0}, donated{0};
  std::atomic<int> failed{0};
  Shared(size_t n_inst, size_t slots) : inst_work(n_inst), seq(slots), payload(slots) {}
};

void fail(Shared& s, const char* what) {
  if (s.failed.exchange(1) == 0) std::fprintf(stderr, "team model: %s\n", what);
}

// A random pause between protocol steps: nothing, a yield, or a few microseconds.
struct Jitter {
  std::mt19937 rng;
  explicit Jitter(uint32_t seed) : rng(seed) {}
  void operator()() {
    const uint32_t r = rng() % 64;
    if (r == 0) std::this_thread::sleep_for(std::chrono::microseconds(1 + rng() % 20));
    else if (r < 8) std::this_thread::yield();
  }
};

// The team's barrier (left early once a check has failed).
void barrier(Shared& s, Team& t) {
  const int phase = t.phase.load(acquire);
  if (t.arrived.fetch_add(1, std::memory_order_acq_rel) == s.waves - 1) {
    t.arrived.store(0, relaxed);
    t.phase.store(phase + 1, release);
    return;
  }
  while (t.phase.load(acquire) == phase && !s.failed.load()) std::this_thread::yield();
}

struct Wave {
  Shared& s;
  Team& t;
  int wave;
  Jitter j;
  std::vector<Node> ring;
  int top = 0, bot = 0;  // [bot, top): pops at top, handovers and donations from bot
  Node entry(int at) const { return ring[static_cast<size_t>(at % s.stack)]; }

  // bits_enqueue: donate the m oldest entries; false if the worklist is at its threshold.
  bool donate(int inst, int m) {
    if (s.count.load(relaxed) >= static_cast<int32_t>(s.threshold)) return false;
    s.inst_work[static_cast<size_t>(inst)].fetch_add(m, relaxed);
    s.work.fetch_add(m, relaxed);
    j();
    s.count.fetch_add(m, relaxed);
    const uint64_t first = s.tail.fetch_add(static_cast<uint64_t>(m), relaxed);
    for (int i = 0; i < m; ++i) {
      const uint64_t ticket = first + static_cast<uint64_t>(i);
      const uint32_t lap = static_cast<uint32_t>(ticket / s.cap);
      while (s.seq[ticket % s.cap].load(acquire) != 2u * lap) {
        if (s.failed.load()) return true;
        std::this_thread::yield();
      }
    }
    for (int i = 0; i < m; ++i) {
      const uint64_t ticket = first + static_cast<uint64_t>(i);
      s.payload[ticket % s.cap] = entry(bot + i);
      j();
      s.seq[ticket % s.cap].store(2u * static_cast<uint32_t>(ticket / s.cap) + 1u, release);
    }
    s.donated.fetch_add(m, relaxed);
    return true;
  }

  // worklist_take / bits_dequeue, the team's first wavefront: 1 a queued node, 2 a root, 0 the end.
  int dequeue(Node* out) {
    for (;;) {
      if (s.failed.load()) return 0;
      if (s.count.load(relaxed) > 0) {
        if (s.count.fetch_add(-1, relaxed) > 0) {
          const uint64_t h = s.head.fetch_add(1, relaxed);
          const uint32_t lap = static_cast<uint32_t>(h / s.cap);
          while (s.seq[h % s.cap].load(acquire) != 2u * lap + 1u) {
            if (s.failed.load()) return 0;
            std::this_thread::yield();
          }
          *out = s.payload[h % s.cap];
          j();
          s.seq[h % s.cap].store(2u * (lap + 1u), release);
          return 1;
        }
        j();
        s.count.fetch_add(1, relaxed);  // lost the race: give the reservation back
        continue;
      }
      if (s.root_next.load(relaxed) < s.num_inst) {
        const int32_t r = s.root_next.fetch_add(1, relaxed);
        if (r < s.num_inst) {
          *out = Node{r, 0};
          return 2;
        }
        continue;
      }
      if (s.work.load(relaxed) == 0) return 0;
      std::this_thread::yield();
    }
  }

  // team_wait: true with this wavefront's box filled, false once the whole team has finished.
  bool wait(bool held) {
    if (held) {
      const int32_t before = t.active.fetch_add(-1, relaxed);
      if (before < 1) fail(s, "the team's count of sub-trees went below zero");
      if (before == 1) return false;
    }
    t.idle.fetch_or(1u << wave, release);
    for (;;) {
      j();
      if (t.mail[wave].load(acquire)) {
        t.mail[wave].store(0, relaxed);
        return true;
      }
      if (t.active.load(acquire) == 0 || s.failed.load()) return false;
      std::this_thread::yield();
    }
  }

  // team_give: the oldest entries to idle wavefronts, one each; returns how many.
  int give(uint32_t idle, int avail) {
    std::vector<int> to;
    for (int w = 0; w < s.waves && static_cast<int>(to.size()) < avail; ++w) {
      if (!(idle >> w & 1u)) continue;
      const auto order = VC_MODEL_MUTATION == 3 ? relaxed : acquire;
      if (t.idle.fetch_and(~(1u << w), order) >> w & 1u) to.push_back(w);
    }
    if (to.empty()) return 0;
    j();
    if (VC_MODEL_MUTATION != 1) t.active.fetch_add(static_cast<int32_t>(to.size()), relaxed);
    for (size_t e = 0; e < to.size(); ++e) {
      t.box[to[e]] = entry(bot + static_cast<int>(e));
      j();
      t.mail[to[e]].store(1, VC_MODEL_MUTATION == 2 ? relaxed : release);
    }
    s.given.fetch_add(static_cast<int64_t>(to.size()), relaxed);
    return static_cast<int>(to.size());
  }

  void run() {
    bool have = false, held = false, first = true;
    bool holding = false;  // the team's first wavefront: the team holds a sub-tree of the launch
    int quiet = 0;
    int last_inst = -1;
    Node cur;
    while (!s.failed.load()) {
      if (!have) {
        if (top > bot) {
          cur = entry(--top);
        } else if (s.waves > 1 && !first && wait(held)) {
          held = true;
          cur = t.box[wave];
        } else {
          held = false;
          barrier(s, t);
          if (wave == 0) {
            if (holding) {
              if (s.inst_work[static_cast<size_t>(last_inst)].fetch_add(-1, relaxed) < 1 ||
                  s.work.fetch_add(-1, relaxed) < 1)
                fail(s, "an outstanding-work counter went below zero");
            }
            t.status = dequeue(&t.taken);
            holding = t.status > 0;
            last_inst = t.taken.inst;
            t.active.store(1, relaxed);
            t.idle.store(0, relaxed);
          }
          barrier(s, t);
          first = false;
          if (s.failed.load() || t.status == 0) return;
          if (wave != 0) continue;
          held = true;
          cur = t.taken;
        }
        have = true;
      }
      const uint32_t idle = t.idle.load(relaxed);  // read before the node's work, used after it
      if (s.visited[static_cast<size_t>(cur.inst)][static_cast<size_t>(cur.node)].exchange(1, relaxed))
        fail(s, "a node was visited twice");
      s.visits.fetch_add(1, relaxed);
      const Tree& tree = s.trees[static_cast<size_t>(cur.inst)];
      const int32_t a = tree.left[static_cast<size_t>(cur.node)];
      const int32_t b = tree.right[static_cast<size_t>(cur.node)];
      j();
      if (a < 0) {
        have = false;
        continue;
      }
      if (b >= 0) {
        const auto defer = [&]() { ring[static_cast<size_t>(top++ % s.stack)] = Node{cur.inst, b}; };
        const bool full = top - bot >= s.stack;
        if (!full) defer();
        int given = 0;
        ++quiet;
        if (s.waves > 1 && idle) given = give(idle, top - bot);
        if (given == 0 && (full || (!idle && (s.waves == 1 || (top - bot > 1 && quiet >= kDonateNodes))))) {
          const int m = std::min(kDonateMost, (top - bot + 1) / 2);
          if (donate(cur.inst, m)) given = m;
          quiet = 0;
        }
        bot += given;
        if (full) {
          if (given == 0) {
            fail(s, "stack ring overflow");
            return;
          }
          defer();
        }
      }
      cur.node = a;
    }
  }
};

}  // namespace

int main(int argc, char** argv) {
  if (argc != 9) {
    std::fprintf(stderr, "usage: %s TEAMS WAVES CAP THRESHOLD INSTANCES MAX_DEPTH STACK SEED\n", argv[0]);
    return 2;
  }
  const int teams = std::atoi(argv[1]), waves = std::atoi(argv[2]);
  const uint32_t cap = static_cast<uint32_t>(std::atoi(argv[3]));
  const uint32_t threshold = static_cast<uint32_t>(std::atoi(argv[4]));
  const int insts = std::atoi(argv[5]), max_depth = std::atoi(argv[6]), stack = std::atoi(argv[7]);
  const uint64_t seed = std::strtoull(argv[8], nullptr, 10);
  // the ring must hold every reservation: (kDonateMost + 1) for each wavefront beyond the threshold
  if (teams < 1 || waves < 1 || waves > kMaxWaves || cap == 0 || (cap & (cap - 1)) || stack < 1 ||
      threshold + static_cast<uint32_t>((kDonateMost + 1) * teams * waves) > cap) {
    std::fprintf(stderr, "bad sizes: cap must be a power of two >= threshold + 5 * wavefronts\n");
    return 2;
  }
  Shared s(static_cast<size_t>(insts), cap);
  s.cap = cap;
  s.threshold = threshold;
  s.num_inst = insts;
  s.waves = waves;
  s.stack = stack;
  int64_t total = 0;
  for (int i = 0; i < insts; ++i) {
    s.trees.push_back(make_tree(seed * 1000 + static_cast<uint64_t>(i), max_depth));
    total += static_cast<int64_t>(s.trees.back().left.size());
    s.visited.emplace_back(s.trees.back().left.size());
  }
  for (int t = 0; t < teams; ++t) s.teams.push_back(std::make_unique<Team>());
  for (auto& w : s.inst_work) w.store(1);  // one root each
  s.work.store(insts);
  for (auto& q : s.seq) q.store(0);
  std::vector<std::thread> pool;
  for (int i = 0; i < teams * waves; ++i)
    pool.emplace_back([&s, i, seed] {
      Wave w{s, *s.teams[static_cast<size_t>(i / s.waves)], i % s.waves,
             Jitter(static_cast<uint32_t>(seed * 7919 + static_cast<uint64_t>(i))),
             std::vector<Node>(static_cast<size_t>(s.stack))};
      w.run();
    });
  for (auto& th : pool) th.join();
  if (s.failed.load()) return 1;
  int64_t seen = 0;
  for (auto& tree : s.visited)
    for (auto& x : tree) seen += x.load();
  if (seen != total || s.visits.load() != total) {
    std::fprintf(stderr, "team model: %lld of %lld nodes visited (%lld visits)\n",
                 static_cast<long long>(seen), static_cast<long long>(total),
                 static_cast<long long>(s.visits.load()));
    return 1;
  }
  if (s.work.load() != 0 || s.count.load() != 0 || s.head.load() != s.tail.load()) {
    std::fprintf(stderr, "team model: counters not back at zero\n");
    return 1;
  }
  for (auto& w : s.inst_work)
    if (w.load() != 0) {
      std::fprintf(stderr, "team model: an instance is not finished\n");
      return 1;
    }
  for (auto& t : s.teams)
    for (auto& m : t->mail)
      if (m.load() != 0) {
        std::fprintf(stderr, "team model: mail left in a box\n");
        return 1;
      }
  const uint64_t done = s.tail.load();
  for (uint32_t slot = 0; slot < cap; ++slot) {
    const uint64_t used = done / cap + (slot < done % cap ? 1 : 0);
    if (s.seq[slot].load() != 2u * static_cast<uint32_t>(used)) {
      std::fprintf(stderr, "team model: slot %u not free for its next lap\n", slot);
      return 1;
    }
  }
  std::printf("ok %lld nodes, %lld handed over, %lld donated\n", static_cast<long long>(total),
              static_cast<long long>(s.given.load()), static_cast<long long>(s.donated.load()));
  return 0;
}
