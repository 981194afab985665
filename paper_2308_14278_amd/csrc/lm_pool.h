// lm_pool.h -- objects kept per device between calls (host only).
#pragma once
#include <mutex>

// At most N objects not in use are kept on each device, while any user of the device
// lives; they go with the last one.  take() hands an object to one call alone, so
// calls on several threads never share one; a call that finds none makes its own.
// Zero-initialised: a static pool needs no constructor and no destructor.
template <class T, int N, int DEVICES>
class DevicePool {
public:
    // A kept object of the device, or null.
    T* take(int device)
    {
        if (device < 0 || device >= DEVICES) return nullptr;
        std::lock_guard<std::mutex> lock(mu_);
        for (T*& k : dev_[device].kept)
            if (k) {
                T* t = k;
                k = nullptr;
                return t;
            }
        return nullptr;
    }
    // Keeps an object for a later call; false: it is the caller's to delete.
    bool keep(int device, T* t)
    {
        if (device < 0 || device >= DEVICES) return false;
        std::lock_guard<std::mutex> lock(mu_);
        if (dev_[device].users == 0) return false;
        for (T*& k : dev_[device].kept)
            if (!k) {
                k = t;
                return true;
            }
        return false;
    }
    void enter(int device)
    {
        if (device < 0 || device >= DEVICES) return;
        std::lock_guard<std::mutex> lock(mu_);
        ++dev_[device].users;
    }
    // The last user takes the kept objects along.
    void leave(int device)
    {
        if (device < 0 || device >= DEVICES) return;
        T* drop[N] = {};
        {
            std::lock_guard<std::mutex> lock(mu_);
            if (--dev_[device].users == 0)
                for (int k = 0; k < N; ++k) {
                    drop[k] = dev_[device].kept[k];
                    dev_[device].kept[k] = nullptr;
                }
        }
        for (T* t : drop) delete t;
    }

private:
    struct Dev {
        T* kept[N] = {};
        long long users = 0;
    };
    std::mutex mu_;
    Dev dev_[DEVICES];
};
