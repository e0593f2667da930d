#include "lds_limit.hpp"

#include "internal.hpp"

namespace rnn {

hipError_t allow_lds(const void* fn, size_t bytes) {
    static LdsRecord record;
    if (bytes <= 64 * 1024) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || record.covers(fn, dev, bytes)) return e;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) record.allowed(fn, dev, bytes);
    return e;
}

}  // namespace rnn
