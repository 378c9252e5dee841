// Host threads for reading a field: see CopyCrew.
#pragma once

#include <algorithm>
#include <condition_variable>
#include <cstddef>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace od {

// Host threads that copy filled staging chunks to the caller's memory while
// the device fills the next ones.  One thread copies about 14 GB/s into fresh
// pages, the link brings 57: reading 1.08 GB (512^3 fp64) took 97-109 ms with
// one thread after each chunk and takes 26-30 ms so.  What can throw is the
// constructor, ahead of the threads and of anything the device does.
class CopyCrew {
   public:
    explicit CopyCrew(size_t chunks) : done_(chunks, 0) {
        const unsigned hw = std::thread::hardware_concurrency();
        jobs_.reserve(chunks);
        threads_ = std::min<size_t>(chunks, std::min<unsigned>(hw > 0 ? hw : 1, kMost));
        crew_.reserve(threads_);
    }
    void begin() {
        try {
            while (crew_.size() < threads_) crew_.emplace_back([this] { work(); });
        } catch (...) {   // no thread, or no memory for one: fewer, or none and wait() copies itself
        }
    }
    ~CopyCrew() {
        {
            std::lock_guard<std::mutex> lk(mu_);
            closed_ = true;
        }
        filled_.notify_all();
        for (std::thread& t : crew_) t.join();
    }
    // once for each chunk
    void give(size_t chunk, char* to, const char* from, size_t bytes) {
        {
            std::lock_guard<std::mutex> lk(mu_);
            jobs_.push_back({chunk, to, from, bytes});
        }
        filled_.notify_one();
    }
    // until a chunk that was given is copied
    void wait(size_t chunk) {
        std::unique_lock<std::mutex> lk(mu_);
        while (!done_[chunk]) {
            if (crew_.empty()) {
                run(lk);
            } else {
                copied_.wait(lk);
            }
        }
    }

   private:
    static constexpr unsigned kMost = 8;
    struct Job {
        size_t chunk;
        char* to;
        const char* from;
        size_t bytes;
    };
    void run(std::unique_lock<std::mutex>& lk) {   // the oldest job, with mu_ held around it
        const Job j = jobs_[next_++];
        lk.unlock();
        std::memcpy(j.to, j.from, j.bytes);
        lk.lock();
        done_[j.chunk] = 1;
    }
    void work() {
        std::unique_lock<std::mutex> lk(mu_);
        for (;;) {
            filled_.wait(lk, [this] { return closed_ || next_ < jobs_.size(); });
            if (next_ == jobs_.size()) return;
            run(lk);
            copied_.notify_all();
        }
    }
    std::mutex mu_;
    std::condition_variable filled_, copied_;
    std::vector<Job> jobs_;   // in the order given; [next_, size) wait
    size_t next_ = 0, threads_ = 0;
    std::vector<char> done_;
    bool closed_ = false;
    std::vector<std::thread> crew_;
};

}  // namespace od
