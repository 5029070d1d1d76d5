// Arrival counting of a grid barrier, host and device.
#pragma once

#if defined(__HIPCC__)
#define SOM_HOST_DEVICE __host__ __device__
#else
#define SOM_HOST_DEVICE
#endif

namespace som {

// Whether a counter that only grows has reached `target`, both modulo 2^32
// and less than 2^31 apart.  (A call of 2^31 - 1 steps counts more than 2^32
// arrivals: 512 workgroups reach that after 8.4 million panels.)
SOM_HOST_DEVICE inline bool arrivals_reached(unsigned arrived, unsigned target) {
    return (int)(arrived - target) >= 0;
}

}  // namespace som
