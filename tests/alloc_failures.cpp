// The library's host side with the n-th memory allocation of a call failing, for n = 1, 2, ...
// until a call makes fewer: each has to return CL_ENOMEM, or CL_OK where it could do without, and
// leave neither by an exception nor by ending the process.  Built by test_host_errors.py with the
// library's host sources; what is called is the program's argument.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "compressed_layer.h"
#include "layer.hpp"
#include "team.hpp"

static std::atomic<long> g_left{-1};        // allocations until the one that fails; negative: none does

static void *allocate(std::size_t n, std::size_t align)
{
    if (g_left.load() >= 0 && g_left.fetch_sub(1) == 0) return nullptr;
    return align ? std::aligned_alloc(align, (n + align - 1) / align * align) : std::malloc(n ? n : 1);
}
static void *allocate_or_throw(std::size_t n, std::size_t align)
{
    if (void *p = allocate(n, align)) return p;
    throw std::bad_alloc();
}
void *operator new(std::size_t n) { return allocate_or_throw(n, 0); }
void *operator new[](std::size_t n) { return allocate_or_throw(n, 0); }
void *operator new(std::size_t n, std::align_val_t a) { return allocate_or_throw(n, (std::size_t)a); }
void *operator new[](std::size_t n, std::align_val_t a) { return allocate_or_throw(n, (std::size_t)a); }
void *operator new(std::size_t n, const std::nothrow_t &) noexcept { return allocate(n, 0); }
void *operator new[](std::size_t n, const std::nothrow_t &) noexcept { return allocate(n, 0); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete[](void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }
void operator delete[](void *p, std::size_t) noexcept { std::free(p); }
void operator delete(void *p, std::align_val_t) noexcept { std::free(p); }
void operator delete[](void *p, std::align_val_t) noexcept { std::free(p); }
void operator delete(void *p, std::size_t, std::align_val_t) noexcept { std::free(p); }
void operator delete[](void *p, std::size_t, std::align_val_t) noexcept { std::free(p); }

namespace cl {
void release_device(cl_layer *) {}          // (the device side is not part of this program)
}

template <class F> static int each_failure(F call)
{
    int failed = 0, passed = 0;
    for (long n = 0;; n += 1 + n / 16) {
        g_left = n;
        const int32_t rc = call();
        const bool reached = g_left.exchange(-1) < 0;
        if (rc != CL_OK && rc != CL_ENOMEM) {
            std::printf("allocation %ld failing: status %d, %s\n", n, rc, cl_last_error());
            return 1;
        }
        ++(rc == CL_OK ? passed : failed);
        if (!reached) break;
    }
    std::printf("%d calls out of memory, %d not\n", failed, passed);
    return failed > 0 ? 0 : 1;
}

int main(int, char **argv)
{
    if (!std::strcmp(argv[1], "team"))
        // a team either starts, with the threads there is memory for, and does its work once, or throws
        return each_failure([&]() -> int32_t {
            try {
                cl::Team team(64, 1);
                std::atomic<int> done{0};
                team.each(1000, [&](int64_t) { ++done; });
                return done == 1000 ? CL_OK : CL_EINVAL;
            } catch (const std::bad_alloc &) {
                return CL_ENOMEM;
            }
        });
    const int M = 1024, K = 2048;           // enough weights, records and bytes for several threads
    std::vector<float> W((size_t)M * K);
    uint32_t x = 1;
    for (float &w : W) {
        x = x * 1664525u + 1013904223u;
        w = x >> 30 ? 0.0f : (float)((x >> 8) & 0xffff) * 1e-5f - 0.3f;
    }
    const cl_layer_desc d{M, K, 5, 4, 128, 128, 0, 0};
    cl_layer *L = nullptr;
    if (cl_compress_layer(&d, W.data(), nullptr, &L) != CL_OK) return 2;
    size_t bytes = 0;
    if (cl_layer_serialize(L, nullptr, &bytes) != CL_OK) return 2;
    std::vector<char> image(bytes), again(bytes);
    if (cl_layer_serialize(L, image.data(), &bytes) != CL_OK) return 2;
    if (!std::strcmp(argv[1], "serialize"))
        return each_failure([&] {
            size_t n = bytes;
            const int32_t rc = cl_layer_serialize(L, again.data(), &n);
            return rc == CL_OK && again != image ? (int32_t)CL_ECORRUPT : rc;
        });
    if (!std::strcmp(argv[1], "deserialize"))
        return each_failure([&] {
            cl_layer *out = nullptr;
            const int32_t rc = cl_layer_deserialize(image.data(), bytes, &out);
            cl_layer_free(out);
            return rc;
        });
    if (!std::strcmp(argv[1], "compress"))
        return each_failure([&] {
            cl_layer *out = nullptr;
            const int32_t rc = cl_compress_layer(&d, W.data(), nullptr, &out);
            cl_layer_free(out);
            return rc;
        });
    const int32_t batches[3] = {1, 2, 4};
    const double ms[6] = {1, 2, 3, 1, 2, 3};
    const int64_t some[2] = {100, 100};
    return each_failure([&] {
        int32_t plan[2];
        double best;
        return cl_plan_batches(2, batches, 3, ms, some, some, some, 10000, 100, 0.0, plan, &best);
    });
}
