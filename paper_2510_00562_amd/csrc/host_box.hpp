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
// few, the rest are freed). The caller reads it after wait(). A call that ends
// before, by an error between a launch and the wait, may leave kernels on its way
// that write here: the box then waits for the stream before it is given back.
class HostBox {
public:
    static constexpr size_t kBytes = kMaxBatch * sizeof(DevScalars);
    explicit HostBox(hipStream_t st);
    ~HostBox();
    HostBox(const HostBox &) = delete;
    HostBox &operator=(const HostBox &) = delete;
    hipError_t status() const { return status_; }
    // from here on a launch may write to the box
    void use() { used_ = true; }
    // until the work on the stream has ended
    hipError_t wait();
    template <typename T>
    T *as() const
    {
        return static_cast<T *>(p_);
    }

private:
    hipStream_t st_;
    bool used_ = false;
    void *p_ = nullptr;
    hipError_t status_ = hipSuccess;
};

}  // namespace geo
