// Scratch device memory of the SF rebuilds that split their operands first.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

#include <mutex>

namespace poseidon {

// What layers that share a launch may ask for together, and what a device's
// streams keep together (one launch's scratch may exceed it alone: operands of
// 2 GiB each take 4 GiB and a little).
constexpr size_t SCRATCH_LAUNCH_MAX = size_t{1} << 30;
constexpr size_t SCRATCH_DEVICE_MAX = size_t{4} << 30;

struct ScratchSlot;

// Scratch for the work that the holder enqueues on one stream before it lets
// go.  A stream's work runs in order, so the next holder on the same stream
// may overwrite the memory; each stream has memory of its own, and two threads
// that share a stream take turns from acquiring to releasing.  A capturing
// stream gets memory that belongs to its graph.
class Scratch {
public:
    Scratch() = default;
    Scratch(const Scratch&) = delete;
    Scratch& operator=(const Scratch&) = delete;
    ~Scratch();
    // False when the memory cannot be had (the sticky error state is clear).
    bool acquire(size_t bytes, hipStream_t stream);
    void* data() const { return data_; }

private:
    void* data_ = nullptr;
    hipStream_t stream_ = nullptr;
    bool captured_ = false;
    std::unique_lock<std::mutex> held_;
};

// Frees what the current device's streams keep (waits for the device).
void scratch_give_back();

}  // namespace poseidon
