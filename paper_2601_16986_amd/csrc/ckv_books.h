// Host bookkeeping of deferred steps (CKV_DEFER_BOOKKEEPING): how many layers go out as one launch, and which layers'
// launches nobody on the caller's side has waited for yet.  Plain C++, no HIP, so that a host program can include it.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace ckv {

constexpr int kBookGroup = 8, kBookGroupMost = 32;

// Layers per launch of deferred bookkeeping: eight, or as many as give every compute unit a workgroup if the layers are
// small (each launch forks from the caller's stream, which costs its next layer about 10 us: 48 layers of eight units,
// captured, in groups of 32 instead of 8: 706 -> 663 us).
inline int book_group(int n_cu, int units_per_layer) { return std::max(kBookGroup, std::min(kBookGroupMost, n_cu / units_per_layer)); }

class PendingBooks {
 public:
  void reset(int layers) {
    after_.assign(layers, 0);
    any_ = false;
  }
  // A launch covers layers [first, first + count); its event is that of its first layer.
  void record(int first, int count) {
    for (int l = first; l < first + count; ++l) after_[l] = 1 + first;
    any_ = true;
  }
  // wait(first) for the launches of every layer (layer < 0) or of one, which are then no longer pending; 0, or what
  // the first failing wait returned.
  template <class Wait>
  int join(int layer, Wait wait) {
    if (!any_) return 0;
    bool left = false;
    for (int l = 0; l < (int)after_.size(); ++l) {
      if (!after_[l]) continue;
      if (layer >= 0 && l != layer) {
        left = true;
        continue;
      }
      if (int rc = wait(after_[l] - 1)) return rc;
      after_[l] = 0;
    }
    any_ = left;
    return 0;
  }

 private:
  std::vector<int16_t> after_;     // 1 + the launch's first layer (up to 256: a byte does not hold it), 0: nothing pending
  bool any_ = false;
};

}  // namespace ckv
