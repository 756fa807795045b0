// pt_readout.hip -- kernels that write results straight into pinned host memory.
//
//   gather_obs     every observable of one instance, packed in one buffer
//   gather_spins   a run of an instance's spins as int8 +-1 in [R][M][N] order
//   gather_err     the device error word
//
// The first two replace host work by one launch (MI355X, before -> now): the observables
// were sixteen copies of a few hundred bytes each, every one a runtime call and a staged
// transfer (262 -> 23 us an instance, the binding's Python included); the spins were copied
// in the device layout and transposed by one host thread (24.0 -> 0.64 ms for 64 replicas of
// 256 x 1024).  What bounds them now is the launch and the wait (observables) and the copy
// out of the pinned buffer (spins).
#include "pt_internal.h"

namespace ptq {
namespace {

constexpr int kObsThreads = 256;

// One workgroup per array: the arrays' loads do not wait for each other's.
__global__ void __launch_bounds__(kObsThreads) gather_obs_kernel(DevState st, ObsLayout o, int32_t n,
                                                                 int32_t rep_base, int32_t pair_base,
                                                                 char *out)
{
    auto copy8 = [&](int32_t at, const void *src, int64_t first, int32_t count) {
        uint64_t *d = reinterpret_cast<uint64_t *>(out + at);
        const uint64_t *s = reinterpret_cast<const uint64_t *>(src) + first;
        for (int32_t k = threadIdx.x; k < count; k += kObsThreads) d[k] = s[k];
    };
    auto copy4 = [&](int32_t at, const int32_t *src) {
        int32_t *d = reinterpret_cast<int32_t *>(out + at);
        for (int32_t k = threadIdx.x; k < o.R; k += kObsThreads) d[k] = src[rep_base + k];
    };
    switch (blockIdx.x) {
    case 0: copy8(o.E, st.E, rep_base, o.R); break;
    case 1: copy8(o.C, st.C, rep_base, o.R); break;
    case 2: copy8(o.rt, st.rt, rep_base, o.R); break;
    case 3: copy8(o.sumE, st.sumE, rep_base, o.R); break;
    case 4: copy8(o.sumC, st.sumC, rep_base, o.R); break;
    case 5: copy8(o.sumE2, st.sumE2, rep_base, o.R); break;
    case 6: copy8(o.sumC2, st.sumC2, rep_base, o.R); break;
    case 7: copy8(o.nup, st.nup, rep_base, o.R); break;
    case 8: copy8(o.ndown, st.ndown, rep_base, o.R); break;
    case 9: copy8(o.acc, st.acc, pair_base, o.R - 1); break;
    case 10: copy8(o.att, st.att, pair_base, o.R - 1); break;
    case 11: copy8(o.sumCt, st.sumCt, (int64_t)rep_base * kTauLags, o.R * kTauLags); break;
    case 12: copy4(o.rung, st.rung_of); break;
    case 13: copy4(o.repof, st.replica_of); break;
    case 14: copy4(o.label, st.label); break;
    default:
        copy8(o.ctr, st.ctr + n, 0, (int32_t)(sizeof(Counters) / 8));
        if (threadIdx.x == 0) *reinterpret_cast<uint32_t *>(out + o.err) = *st.err;
        break;
    }
}

constexpr int kSpinThreads = 256;

// Bytes [first, first + bytes) of an instance's spins in [R][M][N] order.  A thread forms 16
// consecutive bytes (one 16-byte store: a wave writes 1 KiB of host memory at a time); its
// sixteen reads run down a column of the device layout and come from L2.  bytes past the
// last whole sixteen are stored one by one.
template <bool PACKED>
__global__ void __launch_bounds__(kSpinThreads) gather_spins_kernel(DevState st, int32_t n, int64_t first,
                                                                    int32_t bytes, char *out, uint32_t *err_out)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *err_out = *st.err;
    const InstDesc d = st.inst[n];
    const int32_t at = (int32_t)(blockIdx.x * kSpinThreads + threadIdx.x) * 16;
    if (at >= bytes) return;
    const int32_t per_rep = d.N * d.M;
    int32_t c = (int32_t)((first + at) / per_rep);
    int32_t rest = (int32_t)((first + at) - (int64_t)c * per_rep);
    int32_t k = rest / d.N, i = rest - k * d.N;
    const int32_t here = bytes - at < 16 ? bytes - at : 16;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int b = 0; b < 16; ++b) {
        if (b < here) {
            const int32_t p = d.M >= 2 ? (k & 1) : 0, m = d.M >= 2 ? (k >> 1) : 0;
            uint32_t x;
            if constexpr (PACKED) {
                const uint32_t *words = reinterpret_cast<const uint32_t *>(st.spins + d.spin_base);
                const int64_t pos = (((int64_t)(c >> 5) * d.parities + p) * d.N + i) * d.bp_row + m;
                x = (words[pos] >> (c & 31)) & 1u;
            } else {
                const uint8_t *rep = st.spins + d.spin_base + (int64_t)c * d.rep_bytes;
                x = rep[((int64_t)p * d.N + i) * d.Mh + m];
            }
            w[b >> 2] |= ((2u * x - 1u) & 0xFFu) << (8 * (b & 3));
            if (++i == d.N) {
                i = 0;
                if (++k == d.M) {
                    k = 0;
                    ++c;
                }
            }
        }
    }
    if (here == 16) {
        *reinterpret_cast<uint4 *>(out + at) = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
        for (int b = 0; b < here; ++b) out[at + b] = (char)(w[b >> 2] >> (8 * (b & 3)));
    }
}

__global__ void gather_err_kernel(DevState st, uint32_t *out) { *out = *st.err; }

}  // namespace

hipError_t launch_gather_err(const DevState &st, uint32_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(gather_err_kernel, dim3(1), dim3(1), 0, s, st, out);
    return hipGetLastError();
}

hipError_t launch_gather_obs(const DevState &st, const ObsLayout &o, int32_t n, int32_t rep_base,
                             int32_t pair_base, void *out, hipStream_t s)
{
    hipLaunchKernelGGL(gather_obs_kernel, dim3(16), dim3(kObsThreads), 0, s, st, o, n, rep_base, pair_base,
                       (char *)out);
    return hipGetLastError();
}

hipError_t launch_gather_spins(const DevState &st, bool packed, int32_t n, int64_t first, int32_t bytes,
                               void *out, uint32_t *err_out, hipStream_t s)
{
    if (bytes <= 0) return hipSuccess;
    const dim3 grid((bytes + 16 * kSpinThreads - 1) / (16 * kSpinThreads));
    if (packed)
        hipLaunchKernelGGL(gather_spins_kernel<true>, grid, dim3(kSpinThreads), 0, s, st, n, first, bytes,
                           (char *)out, err_out);
    else
        hipLaunchKernelGGL(gather_spins_kernel<false>, grid, dim3(kSpinThreads), 0, s, st, n, first, bytes,
                           (char *)out, err_out);
    return hipGetLastError();
}

}  // namespace ptq
