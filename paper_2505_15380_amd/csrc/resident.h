// Which launches whose workgroups wait for each other may run side by side on a device (host only).
//
// Such launches hold compute units while they do: of two that do not fit the device together each would hold what the other one waits for until their
// bounded waits give up.  What has to fit is every XCD's share: workgroup w of a launch runs on XCD w % 8 and has a compute unit to itself, so 218 and 37
// workgroups are 255 of 256 units, but 28 + 5 of the 32 of the first XCDs.  A launch is counted as its largest share; sums of shares that fit here also fit
// where a partition of the device has fewer XCDs.  A stream's launches are ordered among themselves: it is counted with the largest of those that are not over.
#pragma once
#include <algorithm>

namespace ssd {

// A launch that may still run.  stream: whatever tells streams apart.
struct Resident { const void* stream; int wgs; };

inline bool resident_fits(const Resident* running, int n, const void* stream, int wgs, int cus) {
  constexpr int XCDS = 8;
  auto share = [](int w) { return (w + XCDS - 1) / XCDS; };
  int sum = share(wgs);
  for (int i = 0; i < n; ++i) {
    if (running[i].stream == stream) continue;
    int most = running[i].wgs;
    bool first = true;
    for (int j = 0; j < n; ++j)
      if (running[j].stream == running[i].stream) {
        first = first && j >= i;
        most = std::max(most, running[j].wgs);
      }
    if (first) sum += share(most);
  }
  return sum <= share(cus);
}

}  // namespace ssd
