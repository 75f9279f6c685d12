// fork_join on a model of streams and events: whatever fails, the work that was launched on a side stream
// comes before anything that follows on the common stream, or has been waited for on the host.  And
// deal_lanes: every active member once, keys together, one stream while launches are timed.
#include <cstdio>
#include <map>
#include <set>
#include <string>

#include "lanes.h"

struct Model {
  using Stream = int;
  using Event = int;
  using Status = int;
  std::map<int, std::set<int>> done;       // per stream: the work whose end its next operation waits for
  std::map<int, std::set<int>> recorded;   // per event
  std::set<int> host;                      // work the host has waited for
  int calls = 0, fail_at = -1;             // the stream or event call that fails
  int ok() const { return 0; }
  int step() { return calls++ == fail_at ? 7 : 0; }
  int record(int e, int s) { if (int r = step()) return r; recorded[e] = done[s]; return 0; }
  int wait(int s, int e) { if (int r = step()) return r; done[s].insert(recorded[e].begin(), recorded[e].end()); return 0; }
  int sync(int s) { host.insert(done[s].begin(), done[s].end()); return 0; }
  void launch(int s, int id) { done[s].insert(id); }
};

static int failures = 0, checks = 0;
static void check(bool ok, const std::string &what) {
  ++checks;
  if (!ok) { ++failures; std::printf("FAIL %s\n", what.c_str()); }
}

static void check_deal() {
  for (unsigned seed = 1; seed <= 200; ++seed) {
    unsigned r = seed * 2654435761u;
    auto next = [&](unsigned n) { r = r * 1664525u + 1013904223u; return (r >> 16) % n; };
    std::vector<qf::LaneMember> ms;
    const unsigned count = 1 + next(12);
    for (unsigned j = 0; j < count; ++j) ms.push_back({(int)next(6), 1e-6 * (1 + next(500)), next(5) != 0, next(20) == 0});
    const int n = 1 + (int)next(4);
    const auto lanes = qf::deal_lanes(ms, n);
    const std::string at = "deal " + std::to_string(seed);
    std::map<size_t, int> where;
    std::set<int> keys;
    bool timed = false, together = true;
    size_t dealt = 0, used = 0;
    for (size_t l = 0; l < lanes.size(); ++l) {
      used += !lanes[l].empty();
      for (size_t j : lanes[l]) { where[j] = (int)l; ++dealt; }
    }
    size_t active = 0;
    for (size_t j = 0; j < ms.size(); ++j)
      if (ms[j].active) {
        ++active;
        keys.insert(ms[j].key);
        timed = timed || ms[j].timed;
        for (size_t i = 0; i < j; ++i)
          if (ms[i].active && ms[i].key == ms[j].key) together = together && where[i] == where[j];
      }
    check((int)lanes.size() == n && dealt == active && where.size() == active, at + ": every active member once");
    check(together, at + ": members of a key together");
    if (timed) check(lanes[0].size() == active, at + ": timed launches on the common stream");
    else check(used == std::min(keys.size(), (size_t)n), at + ": every stream used");
  }
}

int main() {
  check_deal();
  for (int nside = 0; nside <= 3; ++nside)
    for (int run_fails = -1; run_fails <= 2 * nside; ++run_fails)       // the launch that fails, -1: none
      for (int fail_at = -1; fail_at <= 1 + 3 * nside; ++fail_at) {     // the stream or event call that fails
        Model m;
        m.fail_at = fail_at;
        m.launch(0, 1000);                     // earlier work of the common stream
        std::vector<qf::SideStream<Model>> sides;
        for (int i = 0; i < nside; ++i) sides.push_back({10 + i, 100 + i});
        std::set<int> launched;
        bool ran = false, early = false;
        const int s = qf::fork_join(m, 0, 99, sides, [&]() -> int {
          ran = true;
          for (int q = 0; q <= 2 * nside; ++q) {
            if (q == run_fails) return 5;
            const int st = q % (nside + 1) ? 9 + q % (nside + 1) : 0;
            early = early || !m.done[st].count(1000);
            m.launch(st, q);
            launched.insert(q);
          }
          return 0;
        });
        const std::string at = "sides " + std::to_string(nside) + ", launch " + std::to_string(run_fails) + ", call " +
                               std::to_string(fail_at);
        check(!early, at + ": side work waits for the common stream");
        for (int q : launched) check(m.done[0].count(q) || m.host.count(q), at + ": launch " + std::to_string(q) + " joined");
        const bool call_failed = fail_at >= 0 && fail_at < m.calls;
        const int want = fail_at == 0 || (call_failed && fail_at <= nside) ? 7 : run_fails >= 0 ? 5 : call_failed ? 7 : 0;
        check(s == want, at + ": status " + std::to_string(s));
        check(ran == !(fail_at >= 0 && fail_at <= nside), at + ": runs if the fork is complete");
      }
  std::printf("%d checks, %d failures\n", checks, failures);
  return failures != 0;
}
