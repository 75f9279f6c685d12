// Work forked from one stream to others and joined to it again (host code; the stream and event calls
// come through `Api`, so that it runs without a device too).
//
// Api: Stream, Event and Status types, Status ok(), and record(event, stream), wait(stream, event) and
// sync(stream), which return a Status.
#pragma once

#include <algorithm>
#include <vector>

namespace qf {

template <class Api> struct SideStream {
  typename Api::Stream stream;
  typename Api::Event join;
};

// The side streams wait for `fork`, recorded on `st`; run() launches on them and on st; st waits for all
// of them.  They are joined also where run() fails: what it launched before that runs on, and a caller
// that synchronises st alone (or frees what the work uses after doing so) must find it done.  Returns
// run()'s failure, else the first one of the calls here.
template <class Api, class Run>
typename Api::Status fork_join(Api &api, typename Api::Stream st, typename Api::Event fork,
                               const std::vector<SideStream<Api>> &sides, Run run) {
  using Status = typename Api::Status;
  Status s = api.record(fork, st);
  if (s != api.ok()) return s;
  size_t forked = 0;
  while (forked < sides.size() && s == api.ok()) {
    s = api.wait(sides[forked].stream, fork);
    if (s == api.ok()) ++forked;
  }
  if (s == api.ok()) s = run();
  for (size_t i = 0; i < forked; ++i) {
    Status j = api.record(sides[i].join, sides[i].stream);
    if (j == api.ok()) j = api.wait(st, sides[i].join);
    if (j != api.ok()) (void)api.sync(sides[i].stream);   // no join on the device: wait here
    if (s == api.ok()) s = j;
  }
  return s;
}

// One member of a batch: members of one key share launches and so a stream; cost: a step's time; active: it
// takes part; timed: its launches are timed.
struct LaneMember {
  int key;
  double cost;
  bool active, timed;
};

// The active members (their indices) of each of n streams: those of one key on the same one, the costliest
// key first to the least loaded stream, the first stream being the common one.  While the launches of any
// of them are timed all of them are on the first, so that every timed launch has the device to itself (as
// under a profiler) and its duration is the kernel's own.
inline std::vector<std::vector<size_t>> deal_lanes(const std::vector<LaneMember> &ms, int n) {
  struct Share { int key; double cost; };
  std::vector<Share> shares;
  bool timed = false;
  for (const LaneMember &m : ms) {
    if (!m.active) continue;
    timed = timed || m.timed;
    auto it = std::find_if(shares.begin(), shares.end(), [&](const Share &x) { return x.key == m.key; });
    if (it == shares.end()) { shares.push_back({m.key, 8e-6}); it = shares.end() - 1; }   // two launches
    it->cost += m.cost;
  }
  std::sort(shares.begin(), shares.end(), [](const Share &x, const Share &y) {
    return x.cost != y.cost ? x.cost > y.cost : x.key < y.key;
  });
  std::vector<double> load(n, 0.0);
  std::vector<std::vector<size_t>> lanes(n);
  for (const Share &x : shares) {
    const size_t l = timed ? 0 : std::min_element(load.begin(), load.end()) - load.begin();
    load[l] += x.cost;
    for (size_t j = 0; j < ms.size(); ++j)
      if (ms[j].active && ms[j].key == x.key) lanes[l].push_back(j);
  }
  return lanes;
}

}  // namespace qf
