// Check of the per-device set-up flag: each device is set up by itself, once,
// and a device whose set-up failed is tried again.  Exit status 0 on success.
#include <stdio.h>

#include <thread>
#include <vector>

#include "device_once.hpp"

static int fail(const char *what, int a, int b)
{
    fprintf(stderr, "device_once check failed: %s (%d, %d)\n", what, a, b);
    return 1;
}

int main()
{
    pyro::DeviceOnce once;
    int calls[66] = {};
    auto set_up = [&](int dev, int status) {
        return once.run(dev, [&] {
            ++calls[dev + 1];
            return status;
        });
    };
    if (set_up(0, 7) != 7 || set_up(0, 7) != 7) return fail("a failure is returned", 0, calls[1]);
    if (calls[1] != 2) return fail("a failure is not kept", 2, calls[1]);
    for (int dev = 0; dev < 64; ++dev) {
        const int before = calls[dev + 1];
        for (int k = 0; k < 3; ++k)
            if (set_up(dev, 0) != 0) return fail("status", dev, k);
        if (calls[dev + 1] != before + 1) return fail("once per device", dev, calls[dev + 1]);
    }
    for (int dev : {-1, 64}) {  // no bit of its own: set up every time
        set_up(dev, 0);
        set_up(dev, 0);
        if (calls[dev + 1] != 2) return fail("out of range", dev, calls[dev + 1]);
    }
    pyro::DeviceOnce shared;
    std::atomic<int> runs{0};
    std::vector<std::thread> th;
    for (int t = 0; t < 4; ++t)
        th.emplace_back([&] {
            for (int k = 0; k < 1000; ++k)
                for (int dev = 0; dev < 64; ++dev)
                    shared.run(dev, [&] {
                        ++runs;
                        return 0;
                    });
        });
    for (auto &t : th) t.join();
    if (runs < 64 || runs > 4 * 64) return fail("threads", runs, 0);
    printf("device_once ok\n");
    return 0;
}
