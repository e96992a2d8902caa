// lgf_host.hpp -- host-side helpers shared by the C-ABI translation units:
// error reporting, argument checks, lattice geometry.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "lgf.h"
#include "lgf_device.hpp"

namespace lgf {

// record a message for lgf_last_error() and return st
lgf_status fail(lgf_status st, const char *fmt, ...);

bool valid_format(int f);
bool valid_dims(const int dims[4]);
Geom make_geom(const int dims[4]);
double elapsed_ms(hipEvent_t a, hipEvent_t b);

// Times of the phases of a driver on its stream without a wait per phase: the
// work between two marks goes to the second one's account (NULL: to none) when
// the stream is next waited for.  A wait costs the GPU 20-40 us of idle time, a
// tenth of a check interval on lattices up to 16^4, so a check interval has one.
struct PhaseClock {
    static constexpr int kMarks = 8;
    hipEvent_t ev[kMarks] = {};
    double *account[kMarks] = {};
    int n = 0;

    hipError_t create()
    {
        for (hipEvent_t &e : ev) {
            const hipError_t err = hipEventCreate(&e);
            if (err != hipSuccess) return err;
        }
        return hipSuccess;
    }
    void destroy()
    {
        for (hipEvent_t &e : ev)
            if (e) (void)hipEventDestroy(e);
    }
    // drop what was marked and not waited for (a call that ended early)
    void reset() { n = 0; }
    hipError_t mark(double *acc, hipStream_t s)
    {
        if (n == kMarks) {
            const hipError_t err = wait();
            if (err != hipSuccess) return err;
            // the last mark stays the start of the phase that ends here
            const hipEvent_t last = ev[kMarks - 1];
            ev[kMarks - 1] = ev[0];
            ev[0] = last;
            account[0] = nullptr;
            n = 1;
        }
        account[n] = acc;
        return hipEventRecord(ev[n++], s);
    }
    // wait for everything up to the last mark and settle the accounts
    hipError_t wait()
    {
        if (n == 0) return hipSuccess;
        const int m = n;
        n = 0;
        const hipError_t err = hipEventSynchronize(ev[m - 1]);
        if (err != hipSuccess) return err;
        for (int i = 1; i < m; ++i)
            if (account[i]) *account[i] += elapsed_ms(ev[i - 1], ev[i]);
        return hipSuccess;
    }
};

}  // namespace lgf

#define LGF_HIP(call)                                                                          \
    do {                                                                                       \
        hipError_t e_ = (call);                                                                \
        if (e_ != hipSuccess)                                                                  \
            return ::lgf::fail(LGF_EHIP, "%s failed: %s (%s:%d)", #call, hipGetErrorString(e_), \
                               __FILE__, __LINE__);                                            \
    } while (0)

#define LGF_TRY(expr)                                                                          \
    do {                                                                                       \
        lgf_status s_ = (expr);                                                                \
        if (s_ != LGF_OK) return s_;                                                           \
    } while (0)
