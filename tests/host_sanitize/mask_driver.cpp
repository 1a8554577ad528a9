// The scalar path's launch with a mask on X: forms whose kernels look at no mask are refused before anything is launched.  Built against the library
// and run without a GPU by tests/test_host_launch.py, where a launch that is not refused ends in another error than hipErrorInvalidValue.
#include <hip/hip_runtime_api.h>

#include <cstdio>

#include "common.hpp"

using namespace hcspmm;

int main()
{
    SpmmArgs good{};
    good.n_rows = good.n_cols = 100000; good.d = 64; good.ldx = good.ldy = 64;
    alignas(128) static char x[256];
    good.X = x; good.Y = reinterpret_cast<float*>(x); good.x_dtype = HCSPMM_F32;
    good.x_mask = reinterpret_cast<const uint2*>(x);
    const CsrHints few{500000, 100000, true, 1024, false, 500000};
    int bad = 0;
    auto refused = [&](const char* what, const SpmmArgs& a, const CsrHints& h, const UpdateArgs* upd, bool want) {
        const hipError_t e = launch_csr(a, 0, nullptr, nullptr, 0, nullptr, a.n_rows, nullptr, nullptr, 64, h, nullptr, upd);
        if ((e == hipErrorInvalidValue) != want) { std::fprintf(stderr, "FAILED: %s: error %d\n", what, (int)e); ++bad; }
    };
    refused("the form with a mask", good, few, nullptr, false);
    UpdateArgs upd{};
    upd.d_out = 16; upd.ldw = upd.ldy = 16;
    refused("the fused update", good, few, &upd, true);
    SpmmArgs a = good;
    a.rowend = reinterpret_cast<const int32_t*>(x);
    refused("a column panel", a, few, nullptr, true);
    a = good;
    a.n_rows = a.n_cols = 1000;
    refused("few rows", a, CsrHints{5000, 1000, true, 1024, false, 5000}, nullptr, true);
    refused("fewer waves", good, CsrHints{10000000, 100000, true, 1024, false, 10000000}, nullptr, true);
    refused("beside the matrix path", good, CsrHints{500000, 100000, true, 1024, true, 500000}, nullptr, true);
    refused("indices of 64 bits", good, CsrHints{500000, 100000, true, 1024, false, (int64_t)1 << 31}, nullptr, true);
    a = good;
    a.x_dtype = HCSPMM_BF16;
    refused("16-bit X", a, few, nullptr, true);
    a = good;
    a.d = a.ldx = 32;
    refused("narrow rows", a, few, nullptr, true);
    a = good;
    a.acc = a.Y;
    refused("rows of sums", a, few, nullptr, true);
    if (bad == 0) std::printf("mask driver: ok\n");
    return bad != 0;
}
