// Launches of the larger-batch FFN kernels (the kernel body: wide_device.h).
#include "moe_internal.h"
#include "wide_device.h"

namespace moe {

namespace {

template <bool GATEUP, bool TOK_LDS, int RB>
__global__ __launch_bounds__(wide::kThreads) void wide_kernel(StreamArgs a)
{
    wide::wide_body<GATEUP, TOK_LDS, RB>(a);
}

}  // namespace

static_assert((size_t)wide::kItemLds + (kMaxC + 1) * 16 + kWideTokCap * 2 <= (size_t)kLdsBytes,
              "any number of slots");

size_t wide_lds_bytes(int T, int k, int C)
{
    const size_t A = (size_t)T * k, n = (size_t)C + 1;
    return (size_t)wide::kItemLds + n * 16 + (A <= (size_t)wide::kTokCap ? (A * 2 + 15) / 16 * 16 : 0);
}

bool wide_tall(const StreamArgs &a, bool gateup)
{
    const long long A = (long long)a.T * a.k, slots = a.C < A ? a.C : A, G = device_cus(nullptr);
    const long long blocks = slots > 0 ? slots * ((A / slots + wide::kToks - 1) / wide::kToks) : 0;   // (routed evenly, every slot in use)
    const long long blocks_sh = (long long)a.n_shared * ((a.T + wide::kToks - 1) / wide::kToks);
    auto items = [&](int rpi) { return (a.R + rpi - 1) / rpi * blocks + (a.n_shared ? (a.R_sh + rpi - 1) / rpi * blocks_sh : 0); };
    auto rounds = [&](int rpi) { return (items(rpi) + G - 1) / (G > 0 ? G : 1); };
    const int rpi = gateup ? 32 : 64;
    // (fewer than two rounds, if so many: with slots that nobody uses there is less than one)
    return items(rpi) >= 2 * G && rounds(rpi) * 2 * 88 <= rounds(rpi / 2) * 100;
}

hipError_t launch_wide(const StreamArgs &a, bool gateup, hipStream_t s)
{
    const size_t lds = wide_lds_bytes(a.T, a.k, a.C);
    if (lds > (size_t)kLdsBytes) return hipErrorInvalidValue;
    const bool in_lds = (size_t)a.T * a.k <= (size_t)wide::kTokCap;
    const bool tall = wide_tall(a, gateup);
#define MOE_WIDE_FN(GU, L) (tall ? (const void *)wide_kernel<GU, L, 4> : (const void *)wide_kernel<GU, L, 2>)
    const void *fn = !gateup ? MOE_WIDE_FN(false, false) : in_lds ? MOE_WIDE_FN(true, true) : MOE_WIDE_FN(true, false);
#undef MOE_WIDE_FN
    hipError_t e = allow_full_lds(fn);
    if (e != hipSuccess) return e;
    const int grid = device_cus(&e);
    if (e != hipSuccess) return e;
    StreamArgs args = a;
    args.rcp_k = rcp32((unsigned)a.k);
    void *params[] = {&args};
    e = launch_timed(fn, dim3(grid), dim3(wide::kThreads), params, lds, s, gateup ? 2 : 4);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace moe
