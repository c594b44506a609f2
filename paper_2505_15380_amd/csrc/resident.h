// Which launches whose workgroups wait for each other may run side by side (host only).
//
// Such launches hold compute units while they do: of two that do not fit the device together each would hold what the other one waits for until their
// bounded waits give up.  So a launch is ordered behind those of other streams that it may not fit beside.  What has to fit is every XCD's share: workgroup w of a
// launch runs on XCD w % 8 and has a compute unit to itself, so 218 and 37 workgroups are 255 of 256 units, but 28 + 5 of the 32 of the first XCDs.  A launch is
// counted as its largest share; sums of shares that fit here also fit where a partition of the device has fewer XCDs.
// A stream's launches are ordered among themselves; what is kept per stream is the most that its launches, and those of other streams that they were ordered
// behind and that may still run, take together; it goes over to a stream that waits for it.  The sum over the streams of a device never exceeds it.
#pragma once
#include <algorithm>

namespace ssd {

struct ResidentTable {
  static constexpr int CAP = 32, XCDS = 8;
  // stream: its handle, or an odd number for a thread's own one (hipStreamPerThread, which names another stream in each thread).  done: event behind the last
  // launch of a stream that other threads cannot name.
  struct Entry { int device; const void* stream; int share; void* done; };
  Entry e[CAP];
  int n = 0;

  // A launch of `wgs` workgroups on `stream`; wait_for(entry) orders it behind what that entry's stream has been given.  Returns the stream's entry, until the
  // next call (null: the table is full of other devices' streams).
  template <typename WAIT>
  Entry* admit(int device, const void* stream, int wgs, int cus, WAIT wait_for) {
    int share = (wgs + XCDS - 1) / XCDS, others = 0;
    const int room = (cus + XCDS - 1) / XCDS;
    Entry* own = nullptr;
    for (int i = 0; i < n; ++i) {
      if (e[i].device != device) continue;
      if (e[i].stream == stream) own = &e[i];
      else others += e[i].share;
    }
    if (own && own->share >= share) return own;                // (it fits: the sum does)
    if (others + share > room || (!own && n >= CAP)) {
      share = std::max(share, others + (own ? own->share : 0));      // (they may all still run)
      int kept = 0;
      for (int i = 0; i < n; ++i) {
        const Entry x = e[i];
        if (x.device != device || x.stream == stream) e[kept++] = x;
        else wait_for(x);
      }
      n = kept;
    }
    for (int i = 0; i < n; ++i)
      if (e[i].stream == stream && e[i].device == device) { e[i].share = std::max(e[i].share, share); return &e[i]; }
    if (n >= CAP) return nullptr;
    e[n] = {device, stream, share, nullptr};
    return &e[n++];
  }
};

}  // namespace ssd
