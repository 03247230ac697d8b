// Plans of recent one-shot calls (lc_copy, lc_gemm), keyed by everything a plan depends on: the layouts' contents, the element
// type, the pointers' alignment and the tuning settings in force.  Planning is pure host work, so a hit changes nothing
// but the time of the call.  Thread-safe; bounded: when full it is emptied (callers with many distinct layouts should
// hold plan handles themselves).
#pragma once
#include <unistd.h>

#include <cstring>
#include <memory>
#include <mutex>
#include <string>
#include <unordered_map>

#include "layout.hpp"

namespace lc {

// Keys are bytes: numbers as they lie in memory, sequences behind their lengths, so that no two different keys read the same.
inline void key_number(std::string* key, int64_t v) { key->append(reinterpret_cast<const char*>(&v), sizeof(v)); }
inline void key_layout(std::string* key, const Layout& L) {
  key_number(key, (int64_t)L.profile.size());
  key->append(reinterpret_cast<const char*>(L.profile.data()), L.profile.size() * sizeof(L.profile[0]));
  key_number(key, (int64_t)L.leaves.size());
  for (const Mode& m : L.leaves) {
    key_number(key, m.extent);
    key_number(key, m.stride);
  }
}

// Every tuning setting in the environment, by name and value, whoever reads it: a list of names here would miss the next one.
// One pass over the environment's names; asked for one by one the thirty settings cost a call more than the rest of its look-up.
// false: there is none, and nothing is added.
inline bool key_tuning(std::string* key) {
  bool any = false;
  for (char** e = environ; e && *e; ++e)
    if (std::strncmp(*e, "LC_TUNE_", 8) == 0) {
      any = true;
      key_number(key, (int64_t)std::strlen(*e));
      key->append(*e);
    }
  return any;
}

template <typename Plan>
class PlanCache {
 public:
  std::shared_ptr<const Plan> find(const std::string& key) {
    std::lock_guard<std::mutex> hold(lock_);
    auto it = plans_.find(key);
    return it == plans_.end() ? nullptr : it->second;
  }
  void insert(const std::string& key, std::shared_ptr<const Plan> plan) {
    std::lock_guard<std::mutex> hold(lock_);
    if (plans_.size() >= kCapacity) plans_.clear();
    plans_[key] = std::move(plan);
  }

 private:
  static constexpr size_t kCapacity = 256;
  std::mutex lock_;
  std::unordered_map<std::string, std::shared_ptr<const Plan>> plans_;
};

}  // namespace lc
