// Results of a blocking call, written by its last kernels into host memory that
// the device reaches. A copy of a few bytes into ordinary memory goes through the
// runtime's staging buffers: a kernel, the copy and the wait took 22.4 us, with
// the kernel writing here 11.9.
#pragma once

#include <hip/hip_runtime.h>

#include "solver.hpp"

namespace geo {

// One call's piece of host memory (kMaxBatch results fit), from a pool shared by
// all threads: taken at construction, given back at destruction (the pool keeps a
// few, the rest are freed). The caller synchronises its stream before it reads.
class HostBox {
public:
    static constexpr size_t kBytes = kMaxBatch * sizeof(DevScalars);
    HostBox();
    ~HostBox();
    HostBox(const HostBox &) = delete;
    HostBox &operator=(const HostBox &) = delete;
    hipError_t status() const { return status_; }
    template <typename T>
    T *as() const
    {
        return static_cast<T *>(p_);
    }

private:
    void *p_ = nullptr;
    hipError_t status_ = hipSuccess;
};

}  // namespace geo
