// Device-side update of the sorted allocation table (the per-context list of
// Sec. 2 / Fig. 2, kept sorted by base for interval lookups).  A new table
// version is the merge of the previous version, minus the bases freed since,
// plus the allocations made since; the result goes to another buffer of the
// version ring, so checks still in flight keep reading their own version.
//
//   k_merge        one lane per old entry: its index in the new table is its
//                  old index, less the frees below it, plus the inserts below
//                  it, and the entries that fall on every 2^shift-th index
//                  also go to the levels above; the version's DevState
//                  is written by the first block
//   k_state        the DevState and the lower levels (a version uploaded whole)
//
// Every freed base is in the old table, so "frees below" is a search in the
// sorted frees and no scan over the old entries is needed.  Bound by latency
// for tables of up to 100,000 entries (one launch, about 4 us), by the copy of
// the table (48 B per entry) above.  A change of a few allocations, the usual
// one when a server applies one event at a time, travels in the launch's own
// arguments: a version then takes one launch, where two uploads from host
// memory and four merge kernels took a chain of about 20 us and the host
// waited for the staging buffer of the version before (20,000 requests with
// 2,000 such events over 100,000 allocations: 145 -> 92 ms).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "xc_internal.h"

namespace xc {
namespace {

constexpr int kB = 256;

// number of entries of a[0..n) that are < x / <= x (a sorted ascending)
template <typename P>
__device__ __forceinline__ uint64_t lower_bound(P a, uint64_t n, uint64_t x)
{
    uint64_t lo = 0, hi = n;
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

template <typename P>
__device__ __forceinline__ uint64_t upper_bound(P a, uint64_t n, uint64_t x)
{
    uint64_t lo = 0, hi = n;
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (a[mid] <= x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ void put(const MergeArgs &m, uint64_t pos, uint64_t base, uint64_t end, uint64_t off)
{
    m.new_base[pos] = base;
    m.new_end[pos] = end;
    m.new_off[pos] = off;
    if ((pos & ((1ull << m.top_shift) - 1ull)) == 0) m.new_top[pos >> m.top_shift] = base;
    if (m.mid_shift && (pos & ((1ull << m.mid_shift) - 1ull)) == 0) m.new_mid[pos >> m.mid_shift] = base;
    if ((pos & ((1u << kFineShift) - 1u)) == 0) m.new_fine[pos >> kFineShift] = base;
}

__device__ __forceinline__ void put_state(const DevState &st, DevState *out)
{
    if (out && blockIdx.x == 0 && threadIdx.x == 0) *out = st;
}

// INLINE: the change is words[0, n_del + 3 n_ins) of the arguments; the old
// entry at or after an insert places it (the lane past the last entry places
// those after all), so no lane searches the old table.  Otherwise the change
// lies in device memory and one lane per insert searches the old table.
template <bool INLINE>
__global__ void __launch_bounds__(kB) k_merge(MergeArgs m)
{
    __shared__ uint64_t sw[INLINE ? kMergeInline : 1];
    put_state(m.state, m.state_out);
    const uint64_t i = (uint64_t)blockIdx.x * kB + threadIdx.x;
    if constexpr (INLINE) {
        for (uint32_t k = threadIdx.x; k < m.n_del + 3 * m.n_ins; k += kB) sw[k] = m.words[k];
        __syncthreads();
        if (i > m.n_old) return;
        const uint64_t *del = sw, *ins = sw + m.n_del;
        const uint64_t nd = m.n_del, ni = m.n_ins;
        const uint64_t b = i < m.n_old ? m.old_base[i] : ~0ull;
        // the inserts above the previous old entry, up to this one (all that are left, past the last)
        uint64_t j = i ? upper_bound(ins, ni, m.old_base[i - 1]) : 0;
        const uint64_t j1 = i < m.n_old ? upper_bound(ins, ni, b) : ni;
        for (; j < j1; ++j) {
            const uint64_t x = ins[j];
            put(m, j + i - lower_bound(del, nd, x), x, ins[ni + j], ins[2 * ni + j]);
        }
        if (i >= m.n_old) return;
        const uint64_t k = lower_bound(del, nd, b);
        if (k < nd && del[k] == b) return;   // freed
        put(m, i - k + lower_bound(ins, ni, b), b, m.old_end[i], m.old_off[i]);
    } else {
        if (i < m.n_old) {
            const uint64_t b = m.old_base[i];
            const uint64_t k = lower_bound(m.del, m.n_del, b);
            if (k < m.n_del && m.del[k] == b) return;   // freed
            put(m, i - k + lower_bound(m.ins_base, m.n_ins, b), b, m.old_end[i], m.old_off[i]);
        } else if (i < m.n_old + m.n_ins) {
            const uint64_t j = i - m.n_old;
            const uint64_t x = m.ins_base[j];
            put(m, j + lower_bound(m.old_base, m.n_old, x) - lower_bound(m.del, m.n_del, x), x, m.ins_end[j],
                m.ins_off[j]);
        }
    }
}

__global__ void __launch_bounds__(kB) k_state(DevState st, DevState *out, uint64_t *mid, uint64_t *fine)
{
    put_state(st, out);
    const uint64_t k = (uint64_t)blockIdx.x * kB + threadIdx.x;
    if ((k << kFineShift) < st.table.n) fine[k] = st.table.base[k << kFineShift];
    if (mid && k < st.table.nmid) mid[k] = st.table.base[k << st.table.mid_shift];
}

}  // namespace

hipError_t launch_merge(const MergeArgs &m, hipStream_t s)
{
    if (m.in_words) {
        const uint64_t blocks = (m.n_old + 1 + kB - 1) / kB;
        hipLaunchKernelGGL((k_merge<true>), dim3((uint32_t)blocks), dim3(kB), 0, s, m);
    } else {
        const uint64_t tot = std::max<uint64_t>(m.n_old + m.n_ins, 1);
        hipLaunchKernelGGL((k_merge<false>), dim3((uint32_t)((tot + kB - 1) / kB)), dim3(kB), 0, s, m);
    }
    return hipGetLastError();
}

hipError_t launch_state(const DevState &st, DevState *out, uint64_t *mid, uint64_t *fine, hipStream_t s)
{
    const uint64_t k = std::max<uint64_t>(std::max<uint64_t>(mid ? st.table.nmid : 1, (st.table.n >> kFineShift) + 1), 1);
    hipLaunchKernelGGL(k_state, dim3((uint32_t)((k + kB - 1) / kB)), dim3(kB), 0, s, st, out, mid, fine);
    return hipGetLastError();
}

hipError_t launch_merge_warm(hipStream_t s)
{
    MergeArgs m{};
    m.in_words = 1;
    return launch_merge(m, s);   // nothing to merge, no state: loads the code only
}

}  // namespace xc
