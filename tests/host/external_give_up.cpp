// hj_join_external after a chained scan of its partition pass gave up, without a
// GPU: the library's objects linked against HIP entry points that do nothing but
// leave what such a pass leaves, partition boundaries that run backwards and the
// error word set.  Driven by tests/test_external_give_up.py.
//
// Prints the status and every host-to-device copy from outside the host arrays.
// (The arrays are reserved, not touched: the copies do nothing.)
#include <cstdio>
#include <cstdlib>

#include "../../paper_1307_1955_amd/csrc/engine.h"

namespace {
constexpr uint64_t kRows = 64 << 20;  // 2^6 partitions and more with the smallest workspace
// addresses of "device" memory are never read
char* const kDevice = reinterpret_cast<char*>(uintptr_t{1} << 40);
struct Range {
    const char* p;
    size_t n;
};
Range known[8];  // the columns, then pinned memory in the order it was taken
int nknown;

void* reserve(size_t n) {
    void* p = calloc(n, 1);
    known[nknown++] = Range{static_cast<char*>(p), n};
    return p;
}
}  // namespace

extern "C" {

void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "none"; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = reserve(n);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    free(p);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t) {
    if (kind == hipMemcpyHostToDevice) {
        bool inside = false;
        for (const Range& k : known) inside |= (const char*)src >= k.p && (const char*)src + n <= k.p + k.n;
        if (!inside) printf("copy of %zu bytes from outside\n", n);
        return hipSuccess;
    }
    // boundaries go to the last allocation: those of R's chunks (its first half) are in
    // order, in those of S the starts' second workgroup of 64 begins at 0 again
    const Range& b = known[nknown - 1];
    if ((char*)dst >= b.p && (char*)dst < b.p + b.n && n > 8) {
        const bool of_s = (char*)dst >= b.p + b.n / 2;
        for (uint32_t i = 0; i < n / 4; ++i) static_cast<uint32_t*>(dst)[i] = (of_s ? i % 64 : i) * 100;
    }
    return hipSuccess;
}
hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind) {
    if (src == kDevice && n == 8) *static_cast<uint64_t*>(dst) = 1;  // the error word
    return hipSuccess;
}

}  // extern "C"

namespace hj {
void Recorder::before(const char*) {}
void Recorder::after() { ++n; }
}  // namespace hj

int main() {
    int32_t* const col = static_cast<int32_t*>(reserve(4 * kRows));
    const hj_rel R{col, col, kRows}, S{col, col, kRows};
    const hj_out O{col, col, kRows};
    hj_params p{};
    p.algo = HJ_AUTO;
    uint64_t count = 0;
    hj_external_info info{};
    const hj_status st = hj_join_external(&p, &R, &S, &O, kDevice, size_t{64} << 20, &count, &info);
    printf("status %d fanout %u count %llu\n", (int)st, info.fanout_bits, (unsigned long long)count);
    return 0;
}
