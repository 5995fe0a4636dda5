// What the host learns of a solve while it steers it: counts and states of a hundred bytes, a dozen to fifty times a call.
//
// A copy and a wait for the stream took the stream 25 to 35 us each time: a launch of 4 us for the copy, then the runtime's way
// back to the caller and out again with the next launch.  Here one wavefront stores the words, and a number after them,
// into pinned memory that the host watches.  Likewise the times of a call's stages: an event in the stream keeps it
// busy for 6 us (and the host for 3), so the kernels that begin a stage note the device's clock instead.
// Rounds of 64 x 64 285 -> 253 us, 777 x 1501 2.21 -> 2.01 ms, 1024 x 1024 1.97 -> 1.87, 3001 x 2003 4.14 -> 3.88, 4096 x 8192
// 7.62 -> 7.28, typed 6001 x 9007 13.1 -> 12.7; from 20,000 x 20,000 on 1 %.
#include "report.h"
#include <chrono>

namespace {

__global__ __launch_bounds__(64) void report_kernel(mf_report r, unsigned long long *reported_at, unsigned *told, unsigned number)
{
    const unsigned long long now = device_time();
    const int lane = threadIdx.x;
#pragma unroll
    for (int p = 0; p < MF_REPORT_PIECES; ++p) tell(r.piece[p].from, r.piece[p].to, r.piece[p].words, lane);
    tell(&now, reported_at, 2, lane);
    tell_number(told, number, lane);
}

__global__ void note_time_kernel(unsigned long long *times, int stage) { note_time(times, stage); }

}  // namespace

int mf_send(mf_ctx *ctx, const mf_report &r, unsigned *number)
{
    *number = ++ctx->reports;
    hipLaunchKernelGGL(report_kernel, dim3(1), dim3(64), 0, ctx->stream, r, &ctx->h_told->at, &ctx->h_told->number, *number);
    MF_HIP(hipGetLastError());
    return MF_OK;
}

// Watches for a while, and leaves waits of more than a few ms, where 20 us more do not count, to the runtime.  (It also
// says what is wrong where nothing will ever be stored: a stream that is being captured, a launch that failed.)
int mf_await(mf_ctx *ctx, unsigned number)
{
    const auto told = [&]() { return (int)(__atomic_load_n(&ctx->h_told->number, __ATOMIC_ACQUIRE) - number) >= 0; };
    const auto begin = std::chrono::steady_clock::now();
    while (!told()) {
        for (int k = 0; k < 16 && !told(); ++k) __builtin_ia32_pause();
        if (std::chrono::steady_clock::now() - begin > std::chrono::milliseconds(5)) {
            MF_HIP(hipStreamSynchronize(ctx->stream));
            if (told()) break;
            ctx->hip_error = hipErrorUnknown;
            return MF_ERR_HIP;
        }
    }
    return MF_OK;
}

int mf_send_and_await(mf_ctx *ctx, const mf_report &r)
{
    unsigned number = 0;
    const int rc = mf_send(ctx, r, &number);
    return rc != MF_OK ? rc : mf_await(ctx, number);
}

void mf_note_time(mf_ctx *ctx, int stage)
{
    hipLaunchKernelGGL(note_time_kernel, dim3(1), dim3(1), 0, ctx->stream, ctx->times, stage);
}
