// What the kernels that work in steps share (kernels_slice.hip, kernels_chain4.hip, kernels_mttkrp.hip): rows gathered through buffer
// descriptors, exchange of values between the lanes of a wavefront, sums over the runs of a workgroup.
#pragma once

#include "device_common.h"

namespace sck {

typedef float sl_floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int sl_uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Rows are gathered through buffer descriptors: a read past the descriptor's end returns zero and touches no memory.  A place of a step that
// no child takes has the coordinate kNoRow, whose byte offset lies past the end of every matrix (they are smaller than 2 GiB; the offset
// is 2^32 less one row, and the lane's part of the row does not carry it over).  So it counts as 0 * 0: with some row that exists and
// a zero factor, an infinity or a NaN in that row would reach outputs that do not refer to it.
constexpr int kNoRow = -1;
constexpr uint32_t kMostBytes = 0x80000000u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t sl_rows(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);   // untyped, 32-bit
}

template <int N>
__device__ __forceinline__ auto sl_gather(__amdgpu_buffer_rsrc_t rows, uint32_t off)
{
    typedef float Vec __attribute__((ext_vector_type(N)));
    if constexpr (N == 1) return __builtin_bit_cast(Vec, __builtin_amdgcn_raw_buffer_load_b32(rows, off, 0, 0));
    else if constexpr (N == 2) return __builtin_bit_cast(Vec, __builtin_amdgcn_raw_buffer_load_b64(rows, off, 0, 0));
    else return __builtin_bit_cast(Vec, __builtin_amdgcn_raw_buffer_load_b128(rows, off, 0, 0));
}

// What the lanes of the wavefront wrote to LDS is there for its other lanes, and what they read may be overwritten.
__device__ __forceinline__ void sl_lanes_meet()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// What is left of a slice that goes on in the next run.  Runs that lie inside one slice are added up inside the workgroup first,
// in two rounds (0 to 1 and 2 to 3, then the pair 0, 1 to the last that follows it); what is left of `goes_on` afterwards goes to the slice's row atomically.
// RPB runs of WPR wavefronts per workgroup, N accumulators (of 16 bytes) of a lane; `same`: the run ends in the slice it began in, which an earlier run began.
// The staging regions are free once the first barrier is passed, and sums may lie in them until the next one after this.
template <int RPB, int WPR, int N, typename V>
__device__ __forceinline__ void sl_sum_runs(V (&acc)[N], bool &goes_on, bool same, V (*sum)[64 * N], int *state_s, int wave, int lane)
{
    const int rw = wave / WPR, sub = wave % WPR;
    if (lane == 0) state_s[wave] = (goes_on ? 1 : 0) | (goes_on && same ? 2 : 0);
    __syncthreads();
    auto state = [&](int n) { return sl_uni(state_s[n * WPR]); };
    // run n's sum goes to run n + 1
    auto pass = [&](int n) { return n + 1 < RPB && (state(n) & 1) && (state(n + 1) & 2); };
    auto send_to = [&](V *buf) {
#pragma unroll
        for (int x = 0; x < N; ++x) buf[x * 64 + lane] = acc[x];
    };
    auto add_from = [&](const V *buf) {
#pragma unroll
        for (int x = 0; x < N; ++x) acc[x] += buf[x * 64 + lane];
    };
    const bool mine = rw % 2 == 0 && pass(rw), theirs = rw % 2 == 1 && pass(rw - 1);
    if (mine) send_to(sum[wave / (2 * WPR) * WPR + sub]);
    __syncthreads();
    if (theirs) add_from(sum[wave / (2 * WPR) * WPR + sub]);
    goes_on = goes_on && !mine;
    if constexpr (RPB == 4) {
        __syncthreads();
        const bool across = pass(1);
        const int to = pass(2) ? 3 : 2;
        if (across && rw == 1) send_to(sum[0]);
        __syncthreads();
        if (across && rw == to) add_from(sum[0]);
        goes_on = goes_on && !(across && rw == 1);
    }
}

}  // namespace sck
