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

}  // namespace qf
