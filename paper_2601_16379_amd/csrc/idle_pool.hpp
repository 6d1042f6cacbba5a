// (The HIP runtime's declarations come from the including file, so that the host
// test compiles the pool on allocation functions of its own.)
#pragma once
#include <mutex>
#include <set>
#include <utility>
#include <vector>

namespace {

// Idle device buffers of the calls that take their workspace per call
// (isdf_hf_jk, isdf_sos_mp2, isdf_drpa), kept by their context between calls:
// allocating and freeing them cost more than the call (a device allocation of
// memory that was freed shortly before waits while it is cleared, at about 10
// GB/s: 0.1 to 0.9 s for the 2.9 GB of a Coulomb-exchange build on a 1000-k
// mesh whose kernels take 7 ms).  At most POOL_BYTES_MAX a context, and at most
// half of what is then free on the device (the caller's own allocations go on
// beside them); all pools are handed back when a device allocation of this
// library fails, before a context plans its buffers and before a fragment
// workspace grows, and a context's with it and on request (isdf_release_idle).  What is planned from the free
// memory counts every pool of the device as free: no context is refused room
// that another one keeps idle.  Buffers in a pool are not in use: a call returns
// its buffers after its stream has drained, and one that fails frees them.
constexpr size_t POOL_BYTES_MAX = (size_t)24 << 30;
class IdlePool {
 public:
  int device = 0;
  IdlePool() {
    std::lock_guard<std::mutex> lk(registry_mu());
    registry().insert(this);
  }
  ~IdlePool() {
    std::lock_guard<std::mutex> lk(registry_mu());
    registry().erase(this);
    drain();
  }
  // A buffer of at least `bytes`, or null; at most an eighth more, as what it
  // has beyond that is out of reach of the call's other allocations.
  void* take(size_t bytes, size_t* got) {
    std::lock_guard<std::mutex> lk(mu_);
    size_t best = idle_.size();
    for (size_t i = 0; i < idle_.size(); ++i)
      if (idle_[i].second >= bytes && idle_[i].second <= bytes + bytes / 8 &&
          (best == idle_.size() || idle_[i].second < idle_[best].second))
        best = i;
    if (best == idle_.size()) return nullptr;
    void* p = idle_[best].first;
    *got = idle_[best].second;
    total_ -= *got;
    idle_.erase(idle_.begin() + best);
    return p;
  }
  // Keeps a buffer (false: no room for it).  Called where a call's buffers go out
  // of scope, so nothing leaves it by an exception.
  bool give(void* p, size_t bytes) noexcept try {
    std::lock_guard<std::mutex> lk(mu_);
    if (total_ + bytes > POOL_BYTES_MAX) return false;
    size_t fr = 0, tot = 0;
    if (hipMemGetInfo(&fr, &tot) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    if (total_ + bytes > fr / 2) return false;
    idle_.emplace_back(p, bytes);
    total_ += bytes;
    return true;
  } catch (...) {
    return false;
  }
  void drain() {
    std::lock_guard<std::mutex> lk(mu_);
    for (auto& b : idle_) (void)hipFree(b.first);
    idle_.clear();
    total_ = 0;
  }
  size_t bytes() {
    std::lock_guard<std::mutex> lk(mu_);
    return total_;
  }
  // Idle bytes of every context on a device.
  static size_t bytes_on(int device) {
    std::lock_guard<std::mutex> lk(registry_mu());
    size_t n = 0;
    for (IdlePool* p : registry())
      if (p->device == device) n += p->bytes();
    return n;
  }
  // Hands back every context's idle buffers; true when there were any.
  static bool drain_all() {
    std::lock_guard<std::mutex> lk(registry_mu());
    bool any = false;
    for (IdlePool* p : registry()) {
      any = any || p->bytes() > 0;
      p->drain();
    }
    return any;
  }

 private:
  static std::mutex& registry_mu() {
    static std::mutex* m = new std::mutex();       // outlives every context
    return *m;
  }
  static std::set<IdlePool*>& registry() {
    static std::set<IdlePool*>* r = new std::set<IdlePool*>();
    return *r;
  }
  std::mutex mu_;
  std::vector<std::pair<void*, size_t>> idle_;
  size_t total_ = 0;
};

}  // namespace
