// Compute units of one device taken by launches whose workgroups wait for one another.  Two such launches that together need
// more than the device has could each hold a part of it and wait for the rest for ever: a call takes its units before its
// first such launch, waiting for calls of other threads to give theirs back, and gives them back when its stream is drained.
// Calls are served in the order in which they came: one that wants nearly the whole device is not passed for ever by smaller
// ones whose turns overlap.
#pragma once
#include <condition_variable>
#include <cstdint>
#include <mutex>

class SharedUnits {
public:
    // Waits until every call that came before has its units and `want` of the device's `all` (no more than that) are free.
    void take(int want, int all)
    {
        std::unique_lock<std::mutex> lock(mutex);
        const uint64_t mine = next++;
        changed.wait(lock, [&] { return mine == turn && taken + want <= all; });
        taken += want;
        ++turn;
        lock.unlock();
        changed.notify_all();          // the next in line may fit as well
    }
    void give(int units)
    {
        {
            std::lock_guard<std::mutex> lock(mutex);
            taken -= units;
        }
        changed.notify_all();
    }

private:
    std::mutex mutex;
    std::condition_variable changed;
    int taken = 0;
    uint64_t next = 0, turn = 0;
};
