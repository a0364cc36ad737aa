// tlmpm_keys.h -- the short sorted key list of the slot-table pass.  Host and device code,
// so that it can be checked on the CPU.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// Up to four distinct keys, ascending, every index a compile-time constant (an array that the
// lanes of a wave index differently takes a loop over the lanes per access).  ~0 is no key: a free place, and nothing
// when added.
struct FourKeys {
    uint32_t a[4] = {~0u, ~0u, ~0u, ~0u};
    bool more = false; // there was a fifth key (the places then hold the smallest four)
    __host__ __device__ void add(uint32_t k)
    {
        const bool have = k == a[0] || k == a[1] || k == a[2] || k == a[3];
        more |= k != ~0u && !have && a[3] != ~0u;
        k = have ? ~0u : k;
#pragma unroll
        for (int i = 3; i > 0; i--) {
            const uint32_t above = a[i - 1] > k ? a[i - 1] : k; // what place i takes if k goes below it
            a[i] = a[i] < above ? a[i] : above;
        }
        a[0] = a[0] < k ? a[0] : k;
    }
    __host__ __device__ int count() const { return (a[0] != ~0u) + (a[1] != ~0u) + (a[2] != ~0u) + (a[3] != ~0u); }
};
