// Pinned host words for the row changes of contexts with a tolerance. Pinning one takes 0.2 ms, as
// long as a short run, so up to 8 words that contexts have given back are kept for the next ones (a
// context gives its word back when its stream has completed). A plain array: a word is given back
// from destructors and C entry points, where an allocation must not fail, and contexts may outlive this
// object's translation unit, so it has no destructor either.
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>

namespace kbe {

class PinnedWords {
 public:
  hipError_t take(double** p) {
    {
      std::lock_guard<std::mutex> lock(mu);
      if (n > 0) {
        *p = kept[--n];
        return hipSuccess;
      }
    }
    return hipHostMalloc((void**)p, sizeof(double), hipHostMallocMapped | hipHostMallocPortable);
  }
  void give_back(double* p) {
    if (!p) return;
    {
      std::lock_guard<std::mutex> lock(mu);
      if (n < KEPT) {
        kept[n++] = p;
        return;
      }
    }
    (void)hipHostFree(p);
  }

 private:
  static constexpr int KEPT = 8;
  std::mutex mu;
  double* kept[KEPT] = {};
  int n = 0;
};

}  // namespace kbe
