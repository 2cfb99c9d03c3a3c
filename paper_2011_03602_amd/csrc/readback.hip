// Residuals to the host, without a copy each.
//
// Reading 8 bytes back costs far more than the kernels of a small grid: after a
// kernel, a copy to pageable memory and the synchronisation take 23 us, to
// pinned memory 15 us; a kernel that stores to pinned host memory itself, and
// the synchronisation, 13 us (11 us of them without the store). A batch's
// residuals are gathered by one kernel, which saved a run of 32 grids 0.55 ms of
// 13.7, one of 12 grids 0.22 ms of 4.4.
#include <mutex>

#include "readback.hpp"

namespace ofl {
namespace {

constexpr int kFoldThreads = 1024;
constexpr int kFoldUnroll = 8;  // loads in flight per thread

void check_launch(const char *what) { hip_check(hipGetLastError(), what); }

__global__ void publish_kernel(const double *gosa, double *slot) { *slot = *gosa; }

__global__ __launch_bounds__(256) void publish_batch_kernel(const GridView *__restrict__ views, int n, double *slots) {
    for (int b = threadIdx.x; b < n; b += 256)
        slots[b] = *views[b].gosa;
}

// One work-group: n is a sweep's waves (2 thousand at 65x65x129, 65 thousand at
// 257x257x513), a chain of loads latency bounds, so each thread has kFoldUnroll
// of them in flight.
__global__ __launch_bounds__(kFoldThreads) void fold_publish_kernel(const double *parts, long long n, double omega,
                                                                    double *gosa, double *slot) {
    __shared__ double wsum[kFoldThreads / kWave];
    double v = 0.0;
    for (long long t = threadIdx.x; t < n; t += kFoldThreads * kFoldUnroll) {
        double x[kFoldUnroll];
#pragma unroll
        for (int q = 0; q < kFoldUnroll; ++q) {
            const long long at = t + static_cast<long long>(q) * kFoldThreads;
            x[q] = at < n ? parts[at] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < kFoldUnroll; ++q)
            v += x[q];
    }
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1)
        v += __shfl_xor(v, d, kWave);
    if (threadIdx.x % kWave == 0)
        wsum[threadIdx.x / kWave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kFoldThreads / kWave; ++w)
            t += wsum[w];
        t /= omega * omega;
        *gosa = t;
        if (slot)
            *slot = t;
    }
}

}  // namespace

// One page for single grids: pinning it takes 35 us, more than the copy that a
// handle which runs once would save. 64 slots of a cache line each.
namespace {
constexpr int kSlotDoubles = 8;
std::mutex g_slot_mutex;
double *g_slot_page = nullptr;
unsigned long long g_slots_used = 0;
}  // namespace

double *host_slot_take() {
    std::lock_guard<std::mutex> lock(g_slot_mutex);
    if (g_slots_used == ~0ULL)
        return nullptr;
    if (!g_slot_page)
        g_slot_page = host_slots_alloc(64 * kSlotDoubles);
    if (!g_slot_page)
        return nullptr;
    const int n = __builtin_ctzll(~g_slots_used);
    g_slots_used |= 1ULL << n;
    return g_slot_page + n * kSlotDoubles;
}

void host_slot_return(double *slot) {
    std::lock_guard<std::mutex> lock(g_slot_mutex);
    g_slots_used &= ~(1ULL << ((slot - g_slot_page) / kSlotDoubles));
}

double *host_slots_alloc(int n) {
    void *ptr = nullptr;
    if (hipHostMalloc(&ptr, sizeof(double) * static_cast<size_t>(n), hipHostMallocPortable | hipHostMallocMapped) !=
        hipSuccess) {
        (void)hipGetLastError();  // the caller copies instead
        return nullptr;
    }
    return static_cast<double *>(ptr);
}

void host_slots_free(double *slots) { (void)hipHostFree(slots); }

void launch_publish(const double *gosa, double *slot, hipStream_t s) {
    publish_kernel<<<1, 1, 0, s>>>(gosa, slot);
    check_launch("residual readback launch");
}

void launch_publish_batch(const GridView *views, int ngrids, double *slots, hipStream_t s) {
    publish_batch_kernel<<<1, 256, 0, s>>>(views, ngrids, slots);
    check_launch("batched residual readback launch");
}

void launch_fold_publish(const double *parts, long long n, float omega, double *gosa, double *slot, hipStream_t s) {
    fold_publish_kernel<<<1, kFoldThreads, 0, s>>>(parts, n, static_cast<double>(omega), gosa, slot);
    check_launch("residual sum launch");
}

}  // namespace ofl
