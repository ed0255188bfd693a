// How the (box, angle) workgroups of a box kernel are cut into launches.
//
// HIP documents that the lanes of a launch (gridDim.x * blockDim.x) must stay
// below 2^32.  A grid over all boxes and angles of a call does not keep to that
// by itself: 41 811 boxes (a 512^3 volume) times 360 angles times 512 lanes is
// 7.7e9.  So a launch takes at most `boxes` boxes and `angles` angles, and a call
// as many launches as that needs; the box kernels add integers, so the result
// does not depend on the cut.  Plain C++: the rule is checked on the host.
#pragma once

#include <algorithm>
#include <cstdint>

namespace vam {

constexpr int kXcds = 8;  // XCDs of an MI355X: workgroup L of a launch runs on XCD L mod 8
constexpr int64_t kMaxLanes = (int64_t(1) << 32) - 1;

struct LaunchCut {
  int boxes, angles;  // the most of each in a launch, both at least 1
};

// n_boxes, na >= 1; threads: lanes of a workgroup.  Angles are cut before boxes
// (a box's segment records are shared by its angles, and almost every cut is one
// of angles), into parts that are alike.
inline LaunchCut launch_cut(int64_t n_boxes, int64_t na, int threads) {
  const int64_t most = kMaxLanes / threads / kXcds * kXcds;  // workgroups
  auto part = [](int64_t n, int64_t most_each) {
    const int64_t parts = (n + most_each - 1) / most_each;
    return (n + parts - 1) / parts;
  };
  const int64_t boxes = part(n_boxes, most);
  return {(int)boxes, (int)part(na, std::max<int64_t>(1, most / boxes))};
}

}  // namespace vam
