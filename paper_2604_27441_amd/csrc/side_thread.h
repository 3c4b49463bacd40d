// One thread beside its owner's that runs one task at a time.
#pragma once
#include <condition_variable>
#include <functional>
#include <mutex>
#include <system_error>
#include <thread>

namespace revo {

class SideThread {
 public:
  SideThread() = default;
  SideThread(const SideThread&) = delete;
  SideThread& operator=(const SideThread&) = delete;
  ~SideThread() { stop(); }

  // Starts the thread, which calls init first.  False when the system has none
  // to give: run then calls both tasks on the caller's thread.
  bool start(std::function<void()> init) {
    try {
      thread_ = std::thread([this, init] {
        init();
        loop();
      });
    } catch (const std::system_error&) {
      return false;
    }
    return true;
  }

  void stop() {
    if (!thread_.joinable()) return;
    {
      std::lock_guard<std::mutex> lk(mu_);
      stop_ = true;
    }
    cv_.notify_all();
    thread_.join();
  }

  // Calls own on the caller's thread and, at the same time, side on the other
  // one; returns when both have, with side's result or, where that is 0, own's.
  int run(const std::function<int()>& own, const std::function<int()>& side) {
    const bool two = thread_.joinable();
    if (two) {
      std::lock_guard<std::mutex> lk(mu_);
      task_ = &side;
      cv_.notify_all();
    }
    const int a = own();
    int b;
    if (two) {
      std::unique_lock<std::mutex> lk(mu_);
      cv_.wait(lk, [&] { return task_ == nullptr; });
      b = result_;
    } else {
      b = side();
    }
    return b ? b : a;
  }

 private:
  void loop() {
    std::unique_lock<std::mutex> lk(mu_);
    for (;;) {
      cv_.wait(lk, [&] { return task_ || stop_; });
      if (!task_) return;
      const std::function<int()>* t = task_;
      lk.unlock();
      const int rc = (*t)();
      lk.lock();
      result_ = rc;
      task_ = nullptr;
      cv_.notify_all();
    }
  }

  std::mutex mu_;
  std::condition_variable cv_;
  const std::function<int()>* task_ = nullptr;  // posted by run, cleared by the thread (guarded by mu_)
  int result_ = 0;
  bool stop_ = false;
  std::thread thread_;
};

}  // namespace revo
