// Calls of the C ABI while every host allocation fails: each returns a status, no exception leaves it.
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "shflbw.h"

static bool failing = false;

void* operator new(std::size_t n)
{
    if (failing) throw std::bad_alloc();
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

static int bad = 0;

template <class F>
static void expect(const char* what, int want, F&& call)
{
    int got = 0;
    bool thrown = false;
    failing = true;
    try {
        got = call();
    } catch (...) {
        thrown = true;
    }
    failing = false;
    if (thrown || got != want) {
        std::printf("%s: %s, status %d, expected %d\n", what, thrown ? "an exception left the call" : "returned", got, want);
        ++bad;
    } else if (!shflbw_last_error()[0]) {
        std::printf("%s: no error text\n", what);
        ++bad;
    }
}

int main()
{
    const int M = 32, K = 48, V = 32;
    std::vector<unsigned short> W(M * K, 0x3c00);
    shflbw_matrix* A = nullptr;
    if (shflbw_compress(W.data(), K, nullptr, nullptr, M, K, V, SHFLBW_F16, &A) != SHFLBW_OK) return 2;
    alignas(256) static unsigned char buf[4096];
    std::vector<int> perm(M, 0);
    std::vector<unsigned char> mask(M * K);
    shflbw_matrix* B = nullptr;

    expect("compress", SHFLBW_ERR_NO_MEMORY,
           [&] { return shflbw_compress(W.data(), K, nullptr, nullptr, M, K, V, SHFLBW_F16, &B); });
    expect("compress, refused", SHFLBW_ERR_BAD_SHAPE,
           [&] { return shflbw_compress(W.data(), K, nullptr, nullptr, M + 1, K, V, SHFLBW_F16, &B); });
    expect("pattern search", SHFLBW_ERR_NO_MEMORY,
           [&] { return shflbw_pattern_search(W.data(), K, M, K, V, 0.5, -1.0, 3, SHFLBW_F16, perm.data(), mask.data()); });
    expect("decompress", SHFLBW_ERR_NULL_ARG, [&] { return shflbw_decompress(nullptr, W.data(), K); });
    expect("set_tuning", SHFLBW_ERR_BAD_OPTION, [&] { return shflbw_set_tuning(A, 9, 0); });
    expect("bind_device", SHFLBW_ERR_BAD_SHAPE, [&] { return shflbw_bind_device(A, buf + 1, nullptr); });
    expect("device_status", SHFLBW_ERR_NOT_ON_DEVICE, [&] { return shflbw_device_status(A, nullptr); });
    expect("spmm, ldx", SHFLBW_ERR_BAD_SHAPE, [&] { return shflbw_spmm(A, buf, 7, buf, 8, 8, SHFLBW_F16, nullptr); });
    expect("spmm, format", SHFLBW_ERR_BAD_DTYPE, [&] { return shflbw_spmm(A, buf, 8, buf, 8, 8, SHFLBW_BF16, nullptr); });
    expect("spmm, not bound", SHFLBW_ERR_NOT_ON_DEVICE, [&] { return shflbw_spmm(A, buf, 8, buf, 8, 8, SHFLBW_F16, nullptr); });
    expect("conv2d, K", SHFLBW_ERR_BAD_SHAPE, [&] {
        return shflbw_conv2d(A, buf, buf, 1, 3, 4, 4, 1, 1, 1, 1, 0, 0, SHFLBW_NCHW, SHFLBW_F16, nullptr);
    });
    expect("conv2d, not bound", SHFLBW_ERR_NOT_ON_DEVICE, [&] {
        return shflbw_conv2d(A, buf, buf, 1, K, 4, 4, 1, 1, 1, 1, 0, 0, SHFLBW_NCHW, SHFLBW_F16, nullptr);
    });
    expect("layernorm_transpose", SHFLBW_ERR_BAD_SHAPE, [&] {
        return shflbw_layernorm_transpose(buf, 9, nullptr, nullptr, 1e-5f, 1, buf, 8, 8, 9, SHFLBW_F16, nullptr);
    });
    shflbw_destroy(A);
    if (!bad) std::printf("every call returned a status\n");
    return bad ? 1 : 0;
}
