// Stable LSD radix sort of (u64 key, u32 value) pairs, 8-bit digits.  The
// key bits that differ between keys are gathered first (each key-building
// block ORs key ^ first key); a pass over a byte that is the same in every
// key is skipped on the device, and each kernel finds its input buffer from
// that mask.  One kernel counts every live byte's digits over all keys; a pass
// is then one kernel: inside a 4,096-key tile each wave ranks its keys with 8
// ballots per key, the tile learns where its digits go by looking back over
// the tiles before it, is sorted locally through LDS and written out as
// contiguous runs per digit.  With count, scan and scatter as three kernels a
// pass, a join of 1M records whose passes all skip took 253 us, now 222, and
// one of 5,000 154 us, now 108.
#include <hip/hip_runtime.h>

#include "sort.h"

namespace xc {
namespace {

constexpr int kT = 256;                          // threads per block
constexpr int kWaves = kT / 64;
constexpr int kSortTile = 4096;                  // keys per sort tile
constexpr int kWaveItems = kSortTile / kWaves;   // contiguous keys per wave
constexpr int kRounds = kWaveItems / 64;
constexpr uint32_t kSortHist = 8 * 256 + 8;      // digit counts of 8 bytes, then a ticket counter per pass
constexpr uint32_t kHistGrid = 512;              // blocks of the digit count, at most
static_assert(kT == kSortKeyBlock, "one part per block of the key kernels");

// the key bits that differ anywhere: OR of the per-block partials
constexpr int kMaskT = 1024;
__global__ __launch_bounds__(kMaskT) void k_sort_mask(const uint64_t *parts, uint32_t nparts, uint64_t *mask,
                                                      uint32_t *hist)
{
    __shared__ uint64_t part[kMaskT / 64];
    // the digit counts and tickets of the sort that follows start at 0
    for (uint32_t j = threadIdx.x; j < kSortHist; j += kMaskT) hist[j] = 0;
    uint64_t x = 0;
    for (uint32_t j = threadIdx.x; j < nparts; j += kMaskT) x |= parts[j];
    for (int d = 32; d >= 1; d >>= 1) x |= __shfl_xor(x, d);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t y = 0;
        for (int w = 0; w < kMaskT / 64; ++w) y |= part[w];
        *mask = y;
    }
}

// ---- radix sort ----------------------------------------------------------


// keys to sort: mcap, or the count held in device memory when there is one
// (never above mcap)
__device__ __forceinline__ uint64_t sort_count_of(uint64_t mcap, const uint64_t *mdev)
{
    if (!mdev) return mcap;
    const uint64_t m = *mdev;
    return m < mcap ? m : mcap;
}

// exclusive sum over the block's threads; *total receives the block sum
__device__ uint32_t block_excl_sum(uint32_t x, uint32_t *total)
{
    __shared__ uint32_t wsum[kWaves];
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t inc = x;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d);
        if (l >= d) inc += y;
    }
    if (l == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
    for (int j = 0; j < kWaves; ++j) {
        if (j < w) off += wsum[j];
        tot += wsum[j];
    }
    __syncthreads();
    *total = tot;
    return off + inc - x;
}

// Digit counts of every live byte over all keys, and the look-back words of
// each tile cleared.  A byte that is the same in the whole wave, as the high
// bytes of addresses mostly are, is counted once for it.
__global__ __launch_bounds__(kT) void k_sort_hist(const uint64_t *keys, uint64_t mcap, const uint64_t *mdev,
                                                  const uint64_t *maskp, int bytes, uint32_t *hist, uint64_t *look)
{
    const uint64_t mask = *maskp;
    if (mask == 0) return;
    const uint64_t m = sort_count_of(mcap, mdev);
    __shared__ uint32_t h[8][256];
    for (int j = threadIdx.x; j < 8 * 256; j += kT) (&h[0][0])[j] = 0;
    __syncthreads();
    const uint32_t tiles = (uint32_t)((m + kSortTile - 1) / kSortTile);
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        look[(uint64_t)tile * 256 + threadIdx.x] = 0;
        const uint64_t base = (uint64_t)tile * kSortTile + threadIdx.x;
        uint64_t k[kSortTile / kT];
#pragma unroll
        for (int i = 0; i < kSortTile / kT; ++i) {
            const uint64_t idx = base + (uint64_t)i * kT;
            k[i] = idx < m ? keys[idx] : 0ull;
        }
#pragma unroll
        for (int i = 0; i < kSortTile / kT; ++i) {
            if (base + (uint64_t)i * kT >= m) continue;
            for (int p = 0; p < bytes; ++p) {
                if (!sort_pass_live(mask, p)) continue;
                const uint32_t d = (uint32_t)(k[i] >> (8 * p)) & 0xFFu;
                const uint64_t here = __ballot(true), same = __ballot(d == __builtin_amdgcn_readfirstlane(d));
                if (same != here) atomicAdd(&h[p][d], 1u);
                else if ((here & lanes_below()) == 0) atomicAdd(&h[p][d], (uint32_t)__popcll(here));
            }
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < 8 * 256; j += kT)
        if ((&h[0][0])[j]) atomicAdd(&hist[j], (&h[0][0])[j]);
}

// A tile's look-back word for a digit: its keys of that digit (kOwn), or those
// of it and all tiles before it (kUpTo), in the low half, and in the high half
// which of the two, of which pass (0: cleared, and older passes read as not
// there yet).
__device__ __forceinline__ uint64_t look_word(int pass, bool upto, uint32_t n)
{
    return (uint64_t)(2 * pass + (upto ? 2 : 1)) << 32 | n;
}

__device__ __forceinline__ void look_put(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Keys of digit t in the tiles before `tile`.  Every wait ends: tiles are
// numbered by a ticket in the order in which their blocks began, and a block
// writes its own counts before it waits for those of earlier ones.  Tiles that
// begin together walk back over each other's own counts, a memory latency a
// step: with kLook words read a step the 12 passes of a join of 1M records take
// 206 us, with one word 242.
constexpr int kLook = 8;
__device__ __forceinline__ uint32_t look_back(const uint64_t *look, uint32_t tile, int pass, int t)
{
    uint32_t sum = 0;
    while (tile > 0) {
        uint64_t v[kLook];
#pragma unroll
        for (int j = 0; j < kLook; ++j) {
            const uint32_t q = tile > (uint32_t)j ? tile - 1 - j : 0;
            v[j] = __hip_atomic_load(look + (uint64_t)q * 256 + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        bool there = true;
#pragma unroll
        for (int j = 0; j < kLook; ++j) {
            const uint32_t state = (uint32_t)(v[j] >> 32);
            there = there && tile > 0 && state >= (uint32_t)(2 * pass + 1);
            if (there) {
                sum += (uint32_t)v[j];
                tile = state == (uint32_t)(2 * pass + 2) ? 0 : tile - 1;   // 0: nothing before it is missing
            }
        }
        if (!there && tile > 0) __builtin_amdgcn_s_sleep(1);
    }
    return sum;
}

// one pass: stable scatter of a tile by one digit
__global__ __launch_bounds__(kT) void k_sort_pass(uint64_t *ka, uint64_t *kb, uint32_t *va, uint32_t *vb,
                                                  uint64_t mcap, const uint64_t *mdev, const uint64_t *maskp, int pass,
                                                  uint32_t *hist, uint64_t *look)
{
    const uint64_t mask = *maskp;
    if (!sort_pass_live(mask, pass)) return;
    const uint64_t m = sort_count_of(mcap, mdev);
    __shared__ uint32_t ticket;
    if (threadIdx.x == 0) ticket = atomicAdd(&hist[8 * 256 + pass], 1u);
    __syncthreads();
    const uint32_t tile = ticket;
    if ((uint64_t)tile * kSortTile >= m) return;   // a tile past the keys (the whole block leaves)
    const int par = sort_parity(mask, pass);
    const uint64_t *kin = par ? kb : ka;
    const uint32_t *vin = par ? vb : va;
    uint64_t *kout = par ? ka : kb;
    uint32_t *vout = par ? va : vb;
    const int shift = 8 * pass;

    __shared__ uint64_t skey[kSortTile];
    __shared__ uint32_t sval[kSortTile];
    __shared__ uint32_t wrun[kWaves][256];   // per wave: running count, then exclusive prefix across waves
    __shared__ uint32_t dstart[256];         // first tile-local position of each digit
    __shared__ uint32_t gbase[256];          // global position of this tile's first key of each digit

    for (int j = threadIdx.x; j < kWaves * 256; j += kT) (&wrun[0][0])[j] = 0;
    __syncthreads();
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const uint64_t base = (uint64_t)tile * kSortTile + (uint64_t)w * kWaveItems + l;
    uint64_t k[kRounds];
    uint32_t v[kRounds], pk[kRounds];
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
        const uint64_t idx = base + (uint64_t)i * 64;
        k[i] = idx < m ? kin[idx] : 0ull;
        v[i] = idx < m ? vin[idx] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
        const bool valid = base + (uint64_t)i * 64 < m;
        const uint32_t d = (uint32_t)(k[i] >> shift) & 0xFFu;
        const uint64_t peers = match8(d, valid);
        const uint32_t rank = (uint32_t)__popcll(peers & lanes_below());
        uint32_t run = 0;
        if (valid) run = wrun[w][d];
        if (valid && rank == 0) wrun[w][d] = run + (uint32_t)__popcll(peers);
        pk[i] = valid ? (d << 16) | (run + rank) : 0xFFFFFFFFu;
    }
    __syncthreads();
    const int t = threadIdx.x;
    uint32_t acc = 0;
    for (int j = 0; j < kWaves; ++j) {
        const uint32_t c = wrun[j][t];
        wrun[j][t] = acc;
        acc += c;
    }
    uint64_t *mine = look + (uint64_t)tile * 256 + t;
    look_put(mine, look_word(pass, tile == 0, acc));
    uint32_t unused;
    dstart[t] = block_excl_sum(acc, &unused);
    const uint32_t first = block_excl_sum(hist[pass * 256 + t], &unused);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
        if (pk[i] != 0xFFFFFFFFu) {
            const uint32_t d = pk[i] >> 16;
            const uint32_t pos = dstart[d] + wrun[w][d] + (pk[i] & 0xFFFFu);
            skey[pos] = k[i];
            sval[pos] = v[i];
        }
    }
    const uint32_t before = look_back(look, tile, pass, t);
    if (tile > 0) look_put(mine, look_word(pass, true, before + acc));
    gbase[t] = first + before;
    __syncthreads();
    const uint64_t left = m - (uint64_t)tile * kSortTile;
    const uint32_t nvalid = left < (uint64_t)kSortTile ? (uint32_t)left : (uint32_t)kSortTile;
    for (uint32_t j = t; j < nvalid; j += kT) {
        const uint64_t key = skey[j];
        const uint32_t d = (uint32_t)(key >> shift) & 0xFFu;
        const uint64_t g = (uint64_t)gbase[d] + (j - dstart[d]);
        if (g < m) {
            kout[g] = key;
            vout[g] = sval[j];
        }
    }
}


uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

}  // namespace

hipError_t sort_reserve(SortWs &w, uint64_t n)
{
    if (n <= w.cap) return hipSuccess;
    sort_release(w);
    const uint64_t tiles = ceil_div(n, kSortTile);
    hipError_t e = hipSuccess;
    auto get = [&](void **p, uint64_t bytes) {
        if (e == hipSuccess) e = hipMalloc(p, bytes ? bytes : 8);
    };
    for (int i = 0; i < 2; ++i) {
        get((void **)&w.keys[i], n * sizeof(uint64_t));
        get((void **)&w.vals[i], n * sizeof(uint32_t));
    }
    get((void **)&w.look, 256 * tiles * sizeof(uint64_t));
    get((void **)&w.hist, kSortHist * sizeof(uint32_t));
    get((void **)&w.parts, ceil_div(n, kT) * sizeof(uint64_t));
    get((void **)&w.mask, sizeof(uint64_t));
    if (e != hipSuccess) {
        sort_release(w);
        return e;
    }
    w.cap = n;
    return hipSuccess;
}

void sort_release(SortWs &w)
{
    void *ps[] = {w.keys[0], w.keys[1], w.vals[0], w.vals[1], w.look, w.hist, w.parts, w.mask};
    for (void *p : ps)
        if (p) (void)hipFree(p);
    w = SortWs{};
}

hipError_t sort_mask_only(SortWs &w, uint64_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_sort_mask, dim3(1), dim3(kMaskT), 0, s, w.parts, (uint32_t)ceil_div(n, kT), w.mask,
                       w.hist);
    return hipGetLastError();
}

hipError_t sort_pairs(SortWs &w, uint64_t n, hipStream_t s, const uint64_t *n_dev, int bytes)
{
    if (n == 0) return hipSuccess;
    if (bytes < 1 || bytes > 8) return hipErrorInvalidValue;
    const uint32_t tiles = (uint32_t)ceil_div(n, kSortTile);
    hipLaunchKernelGGL(k_sort_mask, dim3(1), dim3(kMaskT), 0, s, w.parts, (uint32_t)ceil_div(n, kT), w.mask,
                       w.hist);
    hipLaunchKernelGGL(k_sort_hist, dim3(tiles < kHistGrid ? tiles : kHistGrid), dim3(kT), 0, s, w.keys[0], n, n_dev,
                       w.mask, bytes, w.hist, w.look);
    for (int pass = 0; pass < bytes; ++pass)
        hipLaunchKernelGGL(k_sort_pass, dim3(tiles), dim3(kT), 0, s, w.keys[0], w.keys[1], w.vals[0], w.vals[1], n,
                           n_dev, w.mask, pass, w.hist, w.look);
    return hipGetLastError();
}

}  // namespace xc
