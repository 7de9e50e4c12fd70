// Scratch memory kept per stream.  Stream-ordered allocation would need no
// bookkeeping, but on this runtime hipFreeAsync waits on the host for the
// stream's work (25-46 us a call, the launches no longer run ahead), and an
// event per call to hand one buffer from stream to stream costs 3 us of GPU
// time; a buffer that stays with its stream costs neither.
#include "scratch.h"

#include <memory>
#include <new>
#include <thread>
#include <vector>

namespace poseidon {

struct ScratchSlot {
    std::mutex use;
    int device = -1;
    hipStream_t stream = nullptr;
    std::thread::id thread;      // of hipStreamPerThread, which names another stream in every thread
    void* data = nullptr;
    size_t bytes = 0;
    uint64_t last = 0;
};

namespace {

std::mutex g_table;
std::vector<std::unique_ptr<ScratchSlot>>& table()
{
    // Never destroyed: the runtime may be gone by the time static objects are.
    static auto* t = new std::vector<std::unique_ptr<ScratchSlot>>;
    return *t;
}
uint64_t g_clock = 0;

// hipMalloc and hipFree are refused while any thread captures a stream
// globally, unless this thread says that it captures nothing itself.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// Frees a slot's memory.  hipFree waits for the device, so for any work that
// still uses it.  The slot is held.
void drop(ScratchSlot& s)
{
    if (s.data) {
        RelaxedCapture relaxed;
        (void)hipFree(s.data);
    }
    s.data = nullptr;
    s.bytes = 0;
}

}  // namespace

bool Scratch::acquire(size_t bytes, hipStream_t stream)
{
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capturing) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    stream_ = stream;
    if (capturing != hipStreamCaptureStatusNone) {
        if (hipMallocAsync(&data_, bytes, stream) != hipSuccess) {
            (void)hipGetLastError();
            data_ = nullptr;
            return false;
        }
        captured_ = true;
        return true;
    }
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const std::thread::id thread =
        stream == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id{};
    std::unique_lock<std::mutex> lock(g_table);
    ScratchSlot* slot = nullptr;
    for (auto& s : table())
        if (s->device == device && s->stream == stream && s->thread == thread)
            slot = s.get();
    if (slot && slot->bytes >= bytes) {
        slot->last = ++g_clock;
        lock.unlock();
        held_ = std::unique_lock<std::mutex>(slot->use);
        // (Another thread may have dropped it meanwhile.)
        if (slot->bytes >= bytes) {
            data_ = slot->data;
            return true;
        }
        held_.unlock();
        lock.lock();
    }
    // More memory, or the stream's first: under the table's lock, the least
    // recently used slots making room.
    if (!slot) {
        // (A slot without memory is free to change hands; the table's lock
        // keeps new holders away.)
        for (auto& s : table())
            if (!s->data && s->use.try_lock()) {
                s->use.unlock();
                slot = s.get();
                break;
            }
        if (!slot) {
            try {
                table().push_back(std::make_unique<ScratchSlot>());
            } catch (const std::bad_alloc&) {
                return false;
            }
            slot = table().back().get();
        }
        slot->device = device;
        slot->stream = stream;
        slot->thread = thread;
    }
    held_ = std::unique_lock<std::mutex>(slot->use);
    slot->last = ++g_clock;
    drop(*slot);
    for (;;) {
        size_t kept = 0;
        ScratchSlot* oldest = nullptr;
        for (auto& s : table())
            if (s->device == device && s.get() != slot && s->data) {
                kept += s->bytes;
                if (!oldest || s->last < oldest->last)
                    oldest = s.get();
            }
        if (!oldest || kept + bytes <= SCRATCH_DEVICE_MAX)
            break;
        std::lock_guard<std::mutex> other(oldest->use);
        drop(*oldest);
    }
    RelaxedCapture relaxed;
    if (hipMalloc(&slot->data, bytes) != hipSuccess) {
        (void)hipGetLastError();
        slot->data = nullptr;
        held_.unlock();
        return false;
    }
    slot->bytes = bytes;
    data_ = slot->data;
    return true;
}

Scratch::~Scratch()
{
    if (captured_)
        (void)hipFreeAsync(data_, stream_);
}

void scratch_give_back()
{
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess)
        return;
    std::lock_guard<std::mutex> lock(g_table);
    for (auto& s : table())
        if (s->device == device) {
            std::lock_guard<std::mutex> use(s->use);
            drop(*s);
        }
}

}  // namespace poseidon
