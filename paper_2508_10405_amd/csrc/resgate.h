// Who may have resident launches on a device (host code, no HIP in it).
//
// The workgroups of a resident launch wait for each other, so the launches that
// run at one time must fit the device together: two that do not would each hold
// CUs that the other one's workgroups need.  A call takes room for its largest
// launch before its first and gives it back after its last; calls that fit side
// by side run side by side (eight contexts of one shot of 140 x 240, 30
// workgroups each, on 256 CUs), the others in the order they came.  Every device
// has a gate of its own.
#pragma once
#include <condition_variable>
#include <map>
#include <mutex>

namespace lsrtm {

// XCDs of the GPU: workgroups are dealt to them in turn, so a launch takes up
// to an eighth of its workgroups, rounded up, on each.
constexpr int RES_XCDS = 8;

class ResGate {
  public:
    // n workgroups of the room the device has (its CUs).
    void acquire(int n, int room) {
        std::unique_lock<std::mutex> lock(mu_);
        const long long mine = last_++;
        const int take = whole(n);
        cv_.wait(lock, [&] { return mine == next_ && (used_ == 0 || used_ + take <= room); });
        used_ += take;
        ++next_;
        cv_.notify_all();
    }
    void release(int n) {
        std::lock_guard<std::mutex> lock(mu_);
        used_ -= whole(n);
        cv_.notify_all();
    }

  private:
    static int whole(int n) { return (n + RES_XCDS - 1) / RES_XCDS * RES_XCDS; }
    std::mutex mu_;
    std::condition_variable cv_;
    int used_ = 0;
    long long last_ = 0, next_ = 0;    // calls that came, calls let in
};

inline ResGate& res_gate(int device) {
    static std::mutex mu;
    static std::map<int, ResGate> gates;
    std::lock_guard<std::mutex> lock(mu);
    return gates[device];              // nodes of a map stay where they are
}

// Room for the time of a scope.
class ResRoom {
  public:
    ResRoom(int device, int n, int room) : gate_(res_gate(device)), n_(n) { gate_.acquire(n, room); }
    ~ResRoom() { gate_.release(n_); }
    ResRoom(const ResRoom&) = delete;
    ResRoom& operator=(const ResRoom&) = delete;

  private:
    ResGate& gate_;
    int n_;
};

}  // namespace lsrtm
