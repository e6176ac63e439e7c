// Host side of a load from host memory: gathers the bricks of a strided source
// into staging buffers, on threads of its own.
#pragma once
#include <sched.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>
#include <utility>
#include <vector>

// threads for a source of so many bytes: none below 2 MiB (a thread to start
// costs about what it copies of 256 KB), no more than a MiB each keeps busy, and
// no more than the cores this process may run on; none either for bricks (of so
// many bytes at most) below 96 KiB, which cost less to copy than to hand over
// (host loads in ms with none / with 8: 256^3 in bricks of 16^3, 23 KB each, 117
// / 148; 384^3 of 24^3, 70 KB, 135 / 169; 512^3 of 32^3, 157 KB, 183 / 170; 512^3
// of 48^3, 500 KB, 85 / 63)
inline int gather_threads(int64_t bytes, int64_t brick = INT64_MAX) {
  if (bytes < (int64_t(2) << 20) || brick < (int64_t(96) << 10)) return 0;
  cpu_set_t cores;
  const int usable = sched_getaffinity(0, sizeof cores, &cores) == 0 ? CPU_COUNT(&cores)
                                                                      : (int)std::thread::hardware_concurrency();
  return (int)std::min<int64_t>({8, bytes >> 20, std::max(usable, 1)});
}

// Threads that gather a host source's bricks into the staging buffers, each
// brick in `kParts` runs of rows.  Brick b goes to buffer b % n_buffers and is
// taken up once release() has let it.
class Gather {
 public:
  static constexpr int kParts = 16;
  struct Brick {
    const char* src;               // first element of the region
    int64_t row, plane, elem;      // byte strides of the source
    int64_t rx, ry, rz, bytes;     // region, bytes per element
  };

  Gather(std::vector<Brick> bricks, void* const* buffers, int n_buffers, int threads)
      : bricks_(std::move(bricks)), left_(bricks_.size(), kParts), buffers_(buffers, buffers + n_buffers) {
    try {
      for (int i = 0; i < threads; ++i) threads_.emplace_back([this] { work(); });
    } catch (...) {   // (as many as there are; wait() does the work where there are none)
    }
  }
  ~Gather() {
    {
      std::lock_guard<std::mutex> lock(mu_);
      stop_ = true;
    }
    cv_.notify_all();
    for (std::thread& t : threads_) t.join();
  }
  // bricks below n may be gathered
  void release(int n) {
    {
      std::lock_guard<std::mutex> lock(mu_);
      released_ = n;
    }
    cv_.notify_all();
  }
  // until brick b is in its buffer
  void wait(int b) {
    if (threads_.empty()) {
      for (int k = 0; k < kParts; ++k) part(b, k);
      return;
    }
    std::unique_lock<std::mutex> lock(mu_);
    cv_.wait(lock, [&] { return left_[b] == 0; });
  }

 private:
  void part(int b, int k) {
    const Brick& g = bricks_[b];
    const int64_t rows = g.ry * g.rz, n = g.rx * g.bytes;
    char* out = static_cast<char*>(buffers_[b % buffers_.size()]) + rows * k / kParts * n;
    for (int64_t r = rows * k / kParts; r < rows * (k + 1) / kParts; ++r, out += n) {
      const char* in = g.src + (r / g.ry) * g.plane + (r % g.ry) * g.row;
      if (g.elem == g.bytes) std::memcpy(out, in, (size_t)n);
      else
        for (int64_t x = 0; x < g.rx; ++x) std::memcpy(out + x * g.bytes, in + x * g.elem, (size_t)g.bytes);
    }
  }
  void work() {
    const int64_t total = (int64_t)bricks_.size() * kParts;
    for (;;) {
      const int64_t t = next_.fetch_add(1);
      if (t >= total) return;
      const int b = (int)(t / kParts);
      {
        std::unique_lock<std::mutex> lock(mu_);
        cv_.wait(lock, [&] { return stop_ || b < released_; });
        if (stop_) return;
      }
      part(b, (int)(t % kParts));
      std::lock_guard<std::mutex> lock(mu_);
      if (--left_[b] == 0) cv_.notify_all();
    }
  }
  std::vector<Brick> bricks_;
  std::vector<int> left_;          // parts of each brick still to do
  std::vector<void*> buffers_;
  std::vector<std::thread> threads_;
  std::mutex mu_;
  std::condition_variable cv_;
  std::atomic<int64_t> next_{0};
  int released_ = 0;
  bool stop_ = false;
};
