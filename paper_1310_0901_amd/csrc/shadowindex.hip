// Indexes of the faulty shadow chunks for large check-only batches (gfx950).
//
// A batch worked as segments reads the same shadow bytes many times (each
// host byte about 160 times, each device byte about 15 times on the
// 1M-record configuration).  A record checked without propagation needs few
// facts about the bytes it reads: for its valid source bytes, how many are
// undefined (V != 0 where A = 1), the first undefined one and the first
// unaddressable one (A = 0, host sources only); for the valid bytes of a host
// destination, the first unaddressable one.  The ranges themselves were
// judged by k_classify's lookups.  Here the parts of each shadow space the
// batch reads (its granules of 256 chunks, 4 KiB of V, that some record reads)
// are read once into two sorted lists: the chunks holding an undefined byte,
// with its mask and the undefined bytes of all chunks before it, and the
// chunks holding an unaddressable byte, with its mask.  A record's facts then
// come from two binary searches per list and the masks of its edge chunks: its
// range lies inside listed granules, so the entries between its searches are
// all of its faulty chunks.  The spaces are the host region (V and A bits) and
// the shadow pool (V only; addressability there is the allocation table's).
// An index is built when reading the listed granules costs less than the scan
// it saves (worth), and is valid when both lists fit their capacity; a record
// whose spaces all have a valid index is answered and leaves the scan, any
// other is scanned as before.  The facts are exact, so verdicts do not depend
// on the choice.  Each kernel works both spaces in one launch.
//
//   (k_classify adds the batch's valid bytes per space to state[0], and
//   marks the granules that its records read)
//   k_sidx_mark_count, k_sidx_mark_list
//                  the marked granules as an ascending list (marks cleared)
//   k_sidx_count   block b over its contiguous slice of the listed granules of
//                  the host region, then of the pool: list entries and
//                  undefined bytes; every block stops once the lists overflow
//   k_sidx_scan    a block per space: the blocks' offsets, the totals, validity
//   k_sidx_fill    block b writes its entries in chunk order (a block with
//                  none returns at once)
//   k_sidx_query   one lane per record: answers the records of a check
//                  without propagation whose spaces are indexed, takes their
//                  units out of the scan, and redoes the scan's block-local
//                  prefix
//   k_sidx_rows    one wave per pitched 2D record whose rows follow row 0:
//                  the same, with the list entries of its span mapped onto
//                  its rows
#include <hip/hip_runtime.h>

#include "xc_internal.h"

namespace xc {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4u __attribute__((aligned(4)));
template <typename T> using gcptr = const __attribute__((address_space(1))) T *;

constexpr int kT = 256;
constexpr uint32_t kPer = 16;                          // granules worked side by side
constexpr uint64_t kGran = 1ull << (kIdxGranShift - 4);   // chunks per granule
static_assert(kGran == kT, "a chunk of a granule per thread");
constexpr uint32_t kMarkT = 1024;                      // threads of the marking kernels
constexpr uint32_t kMarkPer = 4;                       // steps per thread of them
constexpr uint64_t kMarkBlock = (uint64_t)kMarkPer * kMarkT;   // steps per block
constexpr uint32_t kPerStep = 1u << (kIdxStepShift - kIdxGranShift);   // granules per step
static_assert(kPerStep == 16, "a step's granules are 16 bits");

// one bit per non-zero byte of w (SWAR: no carry crosses a byte)
__device__ __forceinline__ uint32_t nz4(uint32_t w)
{
    const uint32_t t = (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u;
    return ((t >> 7) | (t >> 14) | (t >> 21) | (t >> 28)) & 0xFu;
}

__device__ __forceinline__ uint32_t nz16(u32x4 v)
{
    return nz4(v.x) | (nz4(v.y) << 4) | (nz4(v.z) << 8) | (nz4(v.w) << 12);
}

// one shadow space as the kernels read it: V bytes (16-byte aligned), A bits
// as 16-bit words (none for the pool), length in bytes
struct Space {
    const uint8_t *v;
    const uint16_t *a16;
    uint64_t len;
};

__device__ __forceinline__ Space space_of(uint32_t space, const DevState *st)
{
    if (space == 0) return Space{st->region.v, st->region.a16, st->region.hl};
    return Space{reinterpret_cast<const uint8_t *>(st->pool), nullptr, st->pool_len};
}

__device__ __forceinline__ uint64_t space_chunks(const Space &S) { return (S.len + 15) >> 4; }

__device__ __forceinline__ uint64_t space_steps(const Space &S) { return (S.len + (1ull << kIdxStepShift) - 1) >> kIdxStepShift; }
__device__ __forceinline__ uint64_t space_grans(const Space &S) { return (S.len + (1ull << kIdxGranShift) - 1) >> kIdxGranShift; }

// The index is built for this batch: a space whose steps fit the marks, and
// less to read than the scan would.  The counting pass streams its granules at
// 6.5-7 TB/s; the scan works a batch's bytes at 4-5 TB/s, most of it short of
// that; and the pass, its lists and the query cost about 25 us more, the scan
// of about 96 MiB (2,000 requests, 354 MB in 187 MB of granules: 151 us
// scanned, 135 us indexed).
__device__ __forceinline__ bool worth(const ShadowIndex &x, const Space &S, uint64_t grans)
{
    if (S.len == 0 || space_steps(S) > x.steps_cap || grans == 0) return false;
    return x.always || x.state[0] >= (grans << kIdxGranShift) / 4 * 3 + (96ull << 20);
}

// positions [p0, p1) of the granule list that block b works, whole groups of kPer
__device__ __forceinline__ void block_slice(const ShadowIndex &x, uint32_t b, uint64_t *p0, uint64_t *p1)
{
    const uint64_t m = x.state[kIdxSteps];
    const uint64_t per = ((m + x.grid - 1) / x.grid + kPer - 1) / kPer * kPer;
    *p0 = (uint64_t)b * per < m ? (uint64_t)b * per : m;
    *p1 = *p0 + per < m ? *p0 + per : m;
}

// undefined (V != 0, A = 1) and unaddressable (A = 0) bytes of chunk c < the
// space's chunks; bits of bytes past the space's end are clear
__device__ __forceinline__ void chunk_faults(const Space &S, uint64_t c, uint32_t *und, uint32_t *un)
{
    const u32x4 v = *reinterpret_cast<const u32x4 *>(S.v + 16 * c);
    const uint32_t a = S.a16 ? (uint32_t)S.a16[c] : 0xFFFFu;
    const uint64_t left = S.len - 16 * c;
    const uint32_t live = left < 16 ? (1u << left) - 1u : 0xFFFFu;
    *und = nz16(v) & a & live;
    *un = ~a & live;
}

// block-wide exclusive scan of three values; tot receives the block's sums
__device__ void block_scan3(uint64_t x[3], uint64_t ex[3], uint64_t tot[3])
{
    __shared__ uint64_t ws[kT / 64][3];
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    uint64_t inc[3] = {x[0], x[1], x[2]};
    for (uint32_t d = 1; d < 64u; d <<= 1) {
        uint64_t y[3];
        for (int k = 0; k < 3; ++k) y[k] = __shfl_up(inc[k], d);
        if (lane >= d)
            for (int k = 0; k < 3; ++k) inc[k] += y[k];
    }
    if (lane == 63u)
        for (int k = 0; k < 3; ++k) ws[w][k] = inc[k];
    __syncthreads();
    for (int k = 0; k < 3; ++k) {
        uint64_t off = 0, all = 0;
        for (uint32_t q = 0; q < kT / 64; ++q) {
            if (q < w) off += ws[q][k];
            all += ws[q][k];
        }
        ex[k] = off + inc[k] - x[k];
        tot[k] = all;
    }
    __syncthreads();   // ws is reused by the next call
}

__device__ __forceinline__ uint64_t block_sum(uint64_t v)
{
    __shared__ uint64_t ws[kMarkT / 64];
    for (int k = 32; k >= 1; k >>= 1) v += __shfl_xor(v, k);
    if ((threadIdx.x & 63u) == 0) ws[threadIdx.x >> 6] = v;
    __syncthreads();
    uint64_t all = 0;
    for (uint32_t q = 0; q < kMarkT / 64; ++q) all += ws[q];
    __syncthreads();   // ws is reused by the next call
    return all;
}

// The marked granules of steps s0 .. s0 + 3, 16 bits each, of a space of
// `grans` granules (every one of them when the batch asked for all).
__device__ __forceinline__ uint64_t marked(const ShadowIndex &x, uint64_t s0, uint64_t grans, bool all)
{
    const uint32_t whole = *reinterpret_cast<const uint32_t *>(x.smark + s0);
    const u32x4 *f = reinterpret_cast<const u32x4 *>(x.fmark + s0 * kPerStep);
    u32x4 fine[kMarkPer];
#pragma unroll
    for (uint32_t j = 0; j < kMarkPer; ++j) fine[j] = f[j];
    uint64_t bits = 0;
#pragma unroll
    for (uint32_t j = 0; j < kMarkPer; ++j)
        bits |= (uint64_t)(all || ((whole >> (8 * j)) & 0xFFu) ? 0xFFFFu : nz16(fine[j])) << (16 * j);
    const uint64_t g0 = s0 * kPerStep;
    if (g0 >= grans) return 0;
    return grans - g0 >= 64 ? bits : bits & ((1ull << (grans - g0)) - 1ull);
}

// marked granules among block b's kMarkBlock steps
__global__ void __launch_bounds__(kMarkT) k_sidx_mark_count(ShadowIndex h, ShadowIndex p, const DevState *stp)
{
    const ShadowIndex &x = blockIdx.y ? p : h;
    if (blockIdx.x >= x.mark_grid) return;
    const uint64_t grans = space_grans(space_of(blockIdx.y, stp));
    const uint64_t s0 = (uint64_t)blockIdx.x * kMarkBlock + kMarkPer * threadIdx.x;
    const uint64_t n = block_sum(s0 * kPerStep < grans ? (uint64_t)__popcll(marked(x, s0, grans, x.state[kIdxAll] != 0)) : 0);
    if (threadIdx.x == 0) x.mcnt[blockIdx.x] = n;
}

// Block b lists its marked granules after those of the blocks before it, when
// the index is worth its cost, and clears its marks; block 0 writes the list's
// length (0: not built).  Each block adds the bytes the counting pass will
// read for its granules.
__global__ void __launch_bounds__(kMarkT) k_sidx_mark_list(ShadowIndex h, ShadowIndex p, const DevState *stp)
{
    __shared__ uint64_t ws[kMarkT / 64];
    const ShadowIndex &x = blockIdx.y ? p : h;
    if (blockIdx.x >= x.mark_grid) return;
    const Space S = space_of(blockIdx.y, stp);
    const uint64_t grans = space_grans(S);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
    const uint64_t s0 = (uint64_t)blockIdx.x * kMarkBlock + kMarkPer * tid;
    if (blockIdx.x > 0 && (uint64_t)blockIdx.x * kMarkBlock * kPerStep >= grans) return;   // past the space: no marks
    uint64_t before = 0, total = 0;
    for (uint32_t k = tid; k < x.mark_grid; k += kMarkT) {
        const uint64_t c = x.mcnt[k];
        total += c;
        before += k < blockIdx.x ? c : 0;
    }
    before = block_sum(before);
    total = block_sum(total);
    const bool build = worth(x, S, total);
    const uint64_t bits = s0 * kPerStep < grans ? marked(x, s0, grans, x.state[kIdxAll] != 0) : 0;
    if (bits) {   // (marks of granules past the space's end there are none)
        *reinterpret_cast<uint32_t *>(x.smark + s0) = 0;
#pragma unroll
        for (uint32_t j = 0; j < kMarkPer; ++j)
            *reinterpret_cast<u32x4 *>(x.fmark + (s0 + j) * kPerStep) = u32x4{0u, 0u, 0u, 0u};
    }
    if (blockIdx.x == 0 && tid == 0) {
        x.state[kIdxSteps] = build ? total : 0;
        x.state[kIdxMarked] = total;
    }
    if (!build) return;
    // block exclusive scan of the threads' marked granules
    const uint64_t n = (uint64_t)__popcll(bits);
    uint64_t inc = n;
    for (uint32_t d = 1; d < 64u; d <<= 1) {
        const uint64_t y = __shfl_up(inc, d);
        if (lane >= d) inc += y;
    }
    if (lane == 63u) ws[w] = inc;
    __syncthreads();
    uint64_t off = before;
    for (uint32_t q = 0; q < w; ++q) off += ws[q];
    off += inc - n;
    // the chunks the counting pass reads for them (the space's last granule may be short)
    const uint64_t nch = space_chunks(S);
    uint64_t chunks = n * kGran;
    if (bits) {
        const uint64_t end = (s0 * kPerStep + 64u - (uint64_t)__builtin_clzll(bits)) * kGran;   // past the last one
        if (end > nch) chunks -= end - nch;
    }
    for (uint32_t j = 0; j < kMarkPer; ++j) {
        uint32_t b = (uint32_t)(bits >> (16 * j)) & 0xFFFFu;
        const uint32_t g = (uint32_t)(s0 + j) * kPerStep;
        if (b == 0xFFFFu) {   // a whole step: four 16-byte stores
#pragma unroll
            for (uint32_t q = 0; q < 16; q += 4)
                *reinterpret_cast<u32x4u *>(x.slist + off + q) = u32x4{g + q, g + q + 1, g + q + 2, g + q + 3};
            off += 16;
            continue;
        }
        for (; b; b &= b - 1u) x.slist[off++] = g + (uint32_t)__builtin_ctz(b);
    }
    chunks = block_sum(chunks);
    if (tid == 0 && chunks)
        atomicAdd((unsigned long long *)x.read, (unsigned long long)(chunks * (x.space == 0 ? 18u : 16u)));
}

// The counting pass of one index over block b's slice of its listed granules
// (nothing when the index is not built).  16 granules at a time, a chunk of
// each per thread, are loaded back to back (non-temporal: each byte is read
// once), then examined; each wave notes in which of the 16 it met a faulty
// chunk, so that the fill reads only those.  The granules of the slice are
// read from the list 64 at a time, one per lane.  A block that met list entries
// adds them to the index's running count and stops when the entries of both
// kinds together pass the room of both lists, so that a space dense with faults
// costs a few per cent of its bytes before the scan takes over.  Bound by HBM: 48.8 GB at 6.8-7.0 TB/s, where a plain read
// of the same shape reaches 0.87-0.89 of 8 TB/s.
__device__ __forceinline__ void count_slice(const ShadowIndex &x, const Space &S)
{
    const bool has_a = S.a16 != nullptr;   // the host region's A bits
    uint64_t p0, p1;
    block_slice(x, blockIdx.x, &p0, &p1);
    const uint64_t nch = space_chunks(S);
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const gcptr<u32x4> vp = reinterpret_cast<gcptr<u32x4>>(reinterpret_cast<uint64_t>(S.v));
    const gcptr<uint16_t> ap = reinterpret_cast<gcptr<uint16_t>>(reinterpret_cast<uint64_t>(S.a16));
    const uint64_t full = S.len >> 4;   // chunks wholly inside the space
    uint64_t c3[3] = {0, 0, 0};
    for (uint64_t g = p0; g < p1; g += 64) {
        const uint32_t mine = x.slist[g + lane < p1 ? g + lane : p1 - 1];
        const uint32_t ng = p1 - g < 64 ? (uint32_t)(p1 - g) : 64u;
        uint32_t found = 0;
        for (uint32_t k = 0; k < ng; k += kPer) {
            // the group's granules, in scalar registers; its last may be short
            // of kPer granules, or hold the space's end
            const uint32_t nk = ng - k < kPer ? ng - k : kPer;
            const uint64_t top = (uint64_t)__builtin_amdgcn_readlane((int)mine, (int)(k + nk - 1)) * kGran + kGran;
            u32x4 v[kPer];
            uint32_t a[kPer];
            const bool inside = nk == kPer && top <= full;
            if (inside) {
#pragma unroll
                for (uint32_t j = 0; j < kPer; ++j) {
                    const uint64_t c = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)mine, (int)(k + j)) * kGran;
                    v[j] = __builtin_nontemporal_load(vp + c + threadIdx.x);
                }
#pragma unroll
                for (uint32_t j = 0; j < kPer; ++j) {
                    const uint64_t c = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)mine, (int)(k + j)) * kGran;
                    a[j] = has_a ? (uint32_t)ap[c + threadIdx.x] : 0xFFFFu;
                }
            } else {
#pragma unroll
                for (uint32_t j = 0; j < kPer; ++j) {
                    v[j] = u32x4{0u, 0u, 0u, 0u};
                    a[j] = 0xFFFFu;
                    if (j < nk) {
                        const uint64_t c = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)mine, (int)(k + j)) * kGran +
                                           threadIdx.x;
                        if (c < nch) {
                            v[j] = __builtin_nontemporal_load(vp + c);
                            if (has_a) a[j] = ap[c];
                        }
                    }
                }
            }
            // almost every chunk is clean (V all 0, A all 1): the lane's chunks
            // are examined one by one only when they are not
            uint32_t orv = 0, anda = 0xFFFFu;
#pragma unroll
            for (uint32_t j = 0; j < kPer; ++j) {
                orv |= v[j].x | v[j].y | v[j].z | v[j].w;
                anda &= a[j];
            }
            uint32_t any = 0;   // granules of the group where this lane met an entry
            if (orv != 0u || anda != 0xFFFFu) {
#pragma unroll
                for (uint32_t j = 0; j < kPer; ++j) {
                    uint32_t live = 0xFFFFu;
                    if (!inside) {   // bytes past the space's end are clear
                        const uint64_t c = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)mine, (int)((k + j) & 63u)) * kGran +
                                           threadIdx.x;
                        const uint64_t left = j < nk && c < nch ? S.len - 16 * c : 0;
                        live = left < 16 ? (1u << left) - 1u : 0xFFFFu;
                    }
                    const uint32_t und = nz16(v[j]) & a[j] & live, un = ~a[j] & live;
                    c3[0] += und ? 1u : 0u;
                    c3[1] += un ? 1u : 0u;
                    c3[2] += (uint32_t)__builtin_popcount(und);
                    found += (und ? 1u : 0u) + (un ? 1u : 0u);
                    any |= (und | un) ? 1u << j : 0u;
                }
            }
            uint32_t seen = 0;
            if (__ballot(any != 0)) {
#pragma unroll
                for (uint32_t j = 0; j < kPer; ++j) seen |= __ballot((any >> j) & 1u) ? 1u << j : 0u;
            }
            if (lane == 0) x.sflag[4 * ((g + k) / kPer) + wave] = (uint16_t)seen;
        }
        // entries met since the last look, and whether the lists are past full
        // (waves of one block may leave at different granules: nothing below
        // depends on the work skipped, since the index is then not valid)
        if (__ballot(found != 0)) {
            for (int d = 32; d >= 1; d >>= 1) found += (uint32_t)__shfl_xor((int)found, d);
            uint64_t now = 0;
            if (lane == 0) now = atomicAdd((unsigned long long *)&x.state[kIdxSeen], (unsigned long long)found) + found;
            now = ((uint64_t)(uint32_t)__shfl((int)(now >> 32), 0) << 32) | (uint32_t)__shfl((int)(uint32_t)now, 0);
            if (now > x.cap_u + x.cap_n) break;
        }
    }
    uint64_t ex[3], tot[3];
    block_scan3(c3, ex, tot);
    if (threadIdx.x == 0)
        for (int k = 0; k < 3; ++k) x.bcnt[3 * blockIdx.x + k] = tot[k];
}

// Both indexes' counting passes in one launch: each block counts its slice of
// the host region's listed granules, then its slice of the pool's, so that the
// shorter pass leaves no tail of its own (both indexes have the same grid).
__global__ void __launch_bounds__(kT) k_sidx_count(ShadowIndex h, ShadowIndex p, const DevState *stp)
{
#pragma nounroll
    for (uint32_t k = 0; k < 2; ++k) {
        const ShadowIndex &x = k ? p : h;
        if (x.state[kIdxSteps]) count_slice(x, space_of(k, stp));
    }
}

// offsets of the blocks' entries into [3 grid, 6 grid) of bcnt
__global__ void __launch_bounds__(1024) k_sidx_scan(ShadowIndex h, ShadowIndex p)
{
    __shared__ uint64_t ws[16][3];
    const ShadowIndex &x = blockIdx.x ? p : h;
    if (x.state[kIdxSteps] == 0 || x.state[kIdxSeen] > x.cap_u + x.cap_n) {   // not built, or stopped half way
        if (threadIdx.x == 0) x.state[1] = 0;
        return;
    }
    const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
    const uint32_t per = (x.grid + 1023) / 1024;
    const uint32_t b0 = tid * per < x.grid ? tid * per : x.grid, b1 = b0 + per < x.grid ? b0 + per : x.grid;
    uint64_t s[3] = {0, 0, 0};
    for (uint32_t b = b0; b < b1; ++b)
        for (int k = 0; k < 3; ++k) s[k] += x.bcnt[3 * b + k];
    uint64_t inc[3] = {s[0], s[1], s[2]};
    for (uint32_t d = 1; d < 64u; d <<= 1) {
        uint64_t y[3];
        for (int k = 0; k < 3; ++k) y[k] = __shfl_up(inc[k], d);
        if (lane >= d)
            for (int k = 0; k < 3; ++k) inc[k] += y[k];
    }
    if (lane == 63u)
        for (int k = 0; k < 3; ++k) ws[w][k] = inc[k];
    __syncthreads();
    uint64_t run[3];
    for (int k = 0; k < 3; ++k) {
        uint64_t off = 0;
        for (uint32_t q = 0; q < w; ++q) off += ws[q][k];
        run[k] = off + inc[k] - s[k];
    }
    for (uint32_t b = b0; b < b1; ++b)
        for (int k = 0; k < 3; ++k) {
            x.bcnt[3 * (x.grid + b) + k] = run[k];
            run[k] += x.bcnt[3 * b + k];
        }
    if (tid == 0) {
        uint64_t tot[3];
        for (int k = 0; k < 3; ++k) {
            uint64_t all = 0;
            for (uint32_t q = 0; q < 16; ++q) all += ws[q][k];
            tot[k] = all;
        }
        const bool valid = tot[0] <= x.cap_u && tot[1] <= x.cap_n;
        x.state[1] = valid ? 1u : 0u;
        x.state[2] = tot[0];
        x.state[3] = tot[1];
        if (valid) {
            x.uchunk[tot[0]] = ~0ull;
            x.ucum[tot[0]] = tot[2];
        }
    }
}

// The entries of one granule, a chunk per thread, in chunk order at the
// running offsets ou / on / op.
__device__ __forceinline__ void fill_granule(const ShadowIndex &x, const Space &S, uint64_t base, uint64_t nch,
                                             uint64_t &ou, uint64_t &on, uint64_t &op)
{
    const uint64_t c = base + threadIdx.x;
    uint32_t und = 0, un = 0;
    if (c < nch) chunk_faults(S, c, &und, &un);
    uint64_t v[3] = {und ? 1u : 0u, un ? 1u : 0u, (uint64_t)__builtin_popcount(und)};
    uint64_t ex[3], tot[3];
    block_scan3(v, ex, tot);
    if (und) {
        const uint64_t i = ou + ex[0];
        x.uchunk[i] = c;
        x.umask[i] = und;
        x.ucum[i] = op + ex[2];
    }
    if (un) {
        const uint64_t i = on + ex[1];
        x.nchunk[i] = c;
        x.nmask[i] = un;
    }
    ou += tot[0];
    on += tot[1];
    op += tot[2];
}

// The block reads its slice's flags 256 groups of granules at a time, one
// group per thread, lists the flagged granules in order, and fills only those.
__global__ void __launch_bounds__(kT) k_sidx_fill(ShadowIndex h, ShadowIndex p, const DevState *stp)
{
    __shared__ uint32_t list[kT * kPer];
    const ShadowIndex &x = blockIdx.y ? p : h;
    if (!x.state[1]) return;
    const Space S = space_of(blockIdx.y, stp);
    const uint32_t b = blockIdx.x;
    if (x.bcnt[3 * b] == 0 && x.bcnt[3 * b + 1] == 0) return;
    uint64_t p0, p1;
    block_slice(x, b, &p0, &p1);
    const uint64_t nch = space_chunks(S);
    uint64_t ou = x.bcnt[3 * (x.grid + b)], on = x.bcnt[3 * (x.grid + b) + 1], op = x.bcnt[3 * (x.grid + b) + 2];
    for (uint64_t g0 = p0; g0 < p1; g0 += kT * kPer) {
        const uint64_t g = g0 + kPer * threadIdx.x;
        uint32_t f = 0;
        if (g < p1) {
            const uint64_t q = *reinterpret_cast<const uint64_t *>(x.sflag + 4 * (g / kPer));
            f = (uint32_t)(q | (q >> 16) | (q >> 32) | (q >> 48)) & 0xFFFFu;
        }
        uint64_t v[3] = {(uint64_t)__builtin_popcount(f), 0, 0};
        uint64_t ex[3], tot[3];
        block_scan3(v, ex, tot);
        for (uint32_t i = (uint32_t)ex[0]; f; f &= f - 1u) list[i++] = kPer * threadIdx.x + (uint32_t)__builtin_ctz(f);
        __syncthreads();
        const uint32_t n = (uint32_t)tot[0];
        for (uint32_t k = 0; k < n; ++k) fill_granule(x, S, (uint64_t)x.slist[g0 + list[k]] * kGran, nch, ou, on, op);
        __syncthreads();   // list is rewritten next
    }
}

// first i in [0, n) with key[i] >= k (n if none)
__device__ __forceinline__ uint64_t lower_bound(const uint64_t *key, uint64_t n, uint64_t k)
{
    uint64_t lo = 0, hi = n;
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (key[mid] < k) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Facts about space offsets [ra, rb) (ra < rb): bytes [ra, rb) of chunk c
// are the bits of range_mask(c).
struct Range {
    uint64_t ca, cb;
    uint32_t lo_bit, hi_bit;
    __device__ Range(uint64_t ra, uint64_t rb)
        : ca(ra >> 4), cb((rb - 1) >> 4), lo_bit((uint32_t)(ra & 15u)), hi_bit((uint32_t)((rb - 1) & 15u)) {}
    __device__ uint32_t mask(uint64_t c) const
    {
        uint32_t m = 0xFFFFu;
        if (c == ca) m &= (0xFFFFu << lo_bit) & 0xFFFFu;
        if (c == cb) m &= (2u << hi_bit) - 1u;
        return m;
    }
};

// first faulty byte of the range among list entries [i0, i1) (space offset,
// or ~0): only the first two entries can hold it, since every entry's mask
// is non-zero and only the edge chunks are cut
__device__ __forceinline__ uint64_t first_in(const uint64_t *chunk, const uint32_t *mask, uint64_t i0, uint64_t i1,
                                             const Range &g)
{
    for (uint64_t i = i0; i < i1 && i < i0 + 2; ++i) {
        const uint32_t bits = mask[i] & g.mask(chunk[i]);
        if (bits) return 16 * chunk[i] + (uint64_t)__builtin_ctz(bits);
    }
    return ~0ull;
}

// undefined bytes of the range and the first one (space offset, or ~0)
// A list's chunk indices with every stride-th of them (samples) in LDS, for a
// two-level search: the samples first, then at most stride - 1 entries in
// global memory.
constexpr uint32_t kSamp = 256;   // samples per list

struct Sampled {
    const uint64_t *chunk;
    uint64_t n, stride, ns;
    const uint64_t *s;   // LDS: chunk[i * stride], i < ns
};

// the block fills s (kSamp entries) for a list of n entries (none when the
// index is not valid); every thread of the block calls it
__device__ __forceinline__ Sampled sample_list(uint64_t *s, const uint64_t *chunk, uint64_t n, bool valid)
{
    if (!valid) n = 0;
    const uint64_t st = n <= kSamp ? 1 : (n + kSamp - 1) / kSamp;
    const uint64_t m = (n + st - 1) / st;
    for (uint64_t i = threadIdx.x; i < m; i += kT) s[i] = chunk[i * st];
    return Sampled{chunk, n, st, m, s};
}

// lower_bound over the sampled list
__device__ __forceinline__ uint64_t lower_bound(const Sampled &x, uint64_t k)
{
    uint64_t lo = 0, hi = x.ns;   // the first sample >= k
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (x.s[mid] < k) lo = mid + 1; else hi = mid;
    }
    // the entries after sample lo - 1 (< k) up to sample lo (>= k), or the list's end
    const uint64_t a = lo == 0 ? 0 : (lo - 1) * x.stride + 1, b = lo < x.ns ? lo * x.stride : x.n;
    return a + lower_bound(x.chunk + a, b - a, k);
}

__device__ __forceinline__ uint64_t undef_in(const ShadowIndex &x, const Sampled &su, const Range &g, uint64_t *first)
{
    const uint64_t i0 = lower_bound(su, g.ca), i1 = lower_bound(su, g.cb + 1);
    uint64_t n = x.ucum[i1] - x.ucum[i0];
    if (i1 > i0) {
        // the edge chunks' bytes outside the range
        if (x.uchunk[i0] == g.ca) n -= (uint64_t)__builtin_popcount(x.umask[i0] & ~(0xFFFFu << g.lo_bit) & 0xFFFFu);
        if (x.uchunk[i1 - 1] == g.cb) n -= (uint64_t)__builtin_popcount(x.umask[i1 - 1] & ~((2u << g.hi_bit) - 1u));
    }
    *first = first_in(x.uchunk, x.umask, i0, i1, g);
    return n;
}

// the first unaddressable byte of the range (space offset, or ~0)
__device__ __forceinline__ uint64_t unaddr_in(const ShadowIndex &x, const Sampled &sn, const Range &g)
{
    const uint64_t j0 = lower_bound(sn, g.ca), j1 = lower_bound(sn, g.cb + 1);
    return first_in(x.nchunk, x.nmask, j0, j1, g);
}

__device__ __forceinline__ void take_first(uint64_t *first, uint64_t off, int64_t off0)
{
    const uint64_t i = (uint64_t)((int64_t)off - off0);   // record byte index of space offset off
    *first = i < *first ? i : *first;
}

// With `pitch`, the positions are pitched 2D records: only those worked as
// one transfer (kRowsContig, whose descriptor is that transfer's) are
// answered, and their units per row go to 0.
__global__ void __launch_bounds__(kT) k_sidx_query(BatchArgs a, ShadowIndex h, ShadowIndex p, Pitch *pitch)
{
    __shared__ uint64_t samp[3][kSamp];
    // the lists' samples: the host region's undefined and unaddressable
    // chunks, the pool's undefined chunks
    const Sampled hu = sample_list(samp[0], h.uchunk, h.state[2], h.state[1] != 0);
    const Sampled hn = sample_list(samp[1], h.nchunk, h.state[3], h.state[1] != 0);
    const Sampled pu = sample_list(samp[2], p.uchunk, p.state[2], p.state[1] != 0);
    __syncthreads();
    const uint64_t t = (uint64_t)blockIdx.x * kT + threadIdx.x;
    const bool none = h.state[1] == 0 && p.state[1] == 0;   // no index: nothing changes but the units to scan
    if (pitch && none) return;
    uint64_t units = !pitch && t < a.count ? a.weight[t] : 0;   // left to scan
    if (!none && a.out && t < a.count && (!pitch || pitch[t].uniform == kRowsContig)) {
        const Desc d = a.desc[t];
        const bool src_host = (d.ctl & CTL_SRC_HOST) != 0;
        const bool has_src = d.v_hi > d.v_lo;
        const bool dsta = (d.ctl & CTL_DST_A) != 0 && d.d_hi > d.d_lo;
        // a check without propagation whose spaces have a valid index
        const bool ok = (d.ctl & CTL_CHECK) && !(d.ctl & CTL_PROP) && d.units > 0 &&
                        (!has_src || (src_host ? h.state[1] : p.state[1])) && (!dsta || h.state[1]);
        if (ok) {
            cg_verdict v = a.out[t];
            uint64_t first = v.first_bad;
            if (has_src) {
                // space offset of the record's byte 0: host region offset, or pool offset
                const int64_t off0 = src_host ? d.a_src + (int64_t)desc_o(d)
                                              : (int64_t)(d.src_sh + desc_o(d) - a.st->pool);
                const Range g((uint64_t)(off0 + d.v_lo), (uint64_t)(off0 + d.v_hi));
                uint64_t fu;
                const uint64_t undef = src_host ? undef_in(h, hu, g, &fu) : undef_in(p, pu, g, &fu);
                if (undef) {
                    v.flags |= CG_SRC_UNDEF;
                    take_first(&first, fu, off0);
                }
                v.undef_bytes += undef;
                if (src_host) {
                    const uint64_t fn = unaddr_in(h, hn, g);
                    if (fn != ~0ull) {
                        v.flags |= CG_SRC_UNADDR;
                        take_first(&first, fn, off0);
                    }
                }
            }
            if (dsta) {
                const int64_t off0 = d.a_dst + (int64_t)desc_o(d);   // host region offset of the destination's byte 0
                const Range g((uint64_t)(off0 + d.d_lo), (uint64_t)(off0 + d.d_hi));
                const uint64_t fn = unaddr_in(h, hn, g);
                if (fn != ~0ull) {
                    v.flags |= CG_DST_UNADDR;
                    take_first(&first, fn, off0);
                }
            }
            v.first_bad = first;
            a.out[t] = v;
            a.desc[t].units = 0;
            a.weight[t] = 0;
            if (pitch) pitch[t].upr = 0;
            units = 0;
        }
    }
    if (pitch) return;   // (k_reweigh follows, after the rows)
    // the block's prefix and sum of the weights max(units, 1), as k_classify
    // makes them, and whether a unit is left
    if (__syncthreads_or(units != 0) && threadIdx.x == 0) atomicOr((unsigned long long *)&h.state[kIdxLeft], 1ull);
    if (none) return;   // (k_classify's stand)
    uint64_t v[3] = {t < a.count ? (units ? units : 1) : 0, 0, 0}, ex[3], tot[3];
    block_scan3(v, ex, tot);
    if (t < a.count) a.local[t] = ex[0];
    if (threadIdx.x == 0) a.bsum[blockIdx.x] = tot[0];
}

// One side of a pitched record in a shadow space: byte c of row r (r < R,
// c < w) is space offset S + r q + c and byte r w + c of the record (its
// bytes are numbered row by row).  Rows may overlap (q < w), even coincide
// (q = 0): a byte then belongs to several rows.
struct RowSide {
    uint64_t S, R, q, w;
};

// the rows holding the byte at offset o = space offset - S: how many, and the
// record byte index of its first one (CG_NONE if none)
__device__ __forceinline__ void byte_rows(const RowSide &x, uint64_t o, uint64_t *n, uint64_t *first)
{
    uint64_t lo, hi;
    if (x.q == 0) {
        if (o >= x.w) return;
        lo = 0;
        hi = x.R - 1;
    } else {
        hi = o / x.q;
        if (hi > x.R - 1) hi = x.R - 1;
        lo = o < x.w ? 0 : (o - x.w) / x.q + 1;   // the first row whose end passes o
    }
    if (lo > hi) return;
    *n += hi - lo + 1;
    const uint64_t i = lo * x.w + (o - lo * x.q);
    *first = i < *first ? i : *first;
}

// bits [lo, hi) of a 16-bit mask (0 <= lo, both clamped to 16)
__device__ __forceinline__ uint32_t bit_range(uint64_t lo, uint64_t hi)
{
    if (hi > 16) hi = 16;
    if (lo >= hi) return 0;
    return ((1u << (uint32_t)hi) - 1u) & ~((1u << (uint32_t)lo) - 1u);
}

// The bytes of chunk c marked in `sel` that lie in rows of side x: how many
// (a byte counted once per row holding it) and the first one's record byte
// index.  Chunks meet at most two rows, and a byte at most one, when
// q >= max(w, 16): one division per chunk; otherwise byte by byte.
__device__ __forceinline__ void chunk_rows(const RowSide &x, uint64_t c, uint32_t sel, uint64_t *n, uint64_t *first)
{
    const uint64_t b0 = 16 * c;
    const uint32_t k0 = b0 < x.S ? (uint32_t)(x.S - b0) : 0u;   // bytes below the first row are in none
    sel &= (0xFFFFu << k0) & 0xFFFFu;
    if (!sel) return;
    const uint64_t o0 = b0 + k0 - x.S;   // offset of byte k0
    if (x.q >= 16 && x.q >= x.w) {
        const uint64_t r = o0 / x.q, m = o0 - r * x.q;
        // bytes k0 + j: row r for m + j < q, row r + 1 after
        uint32_t in = 0;
        if (r < x.R && m < x.w) in |= bit_range(k0, k0 + (x.w - m));
        if (r + 1 < x.R && x.q - m < 16) in |= bit_range(k0 + (x.q - m), k0 + (x.q - m) + x.w);
        const uint32_t hit = sel & in;
        if (!hit) return;
        *n += (uint64_t)__builtin_popcount(hit);
        const uint64_t j = (uint64_t)__builtin_ctz(hit) - k0;
        const uint64_t i = m + j < x.q ? r * x.w + m + j : (r + 1) * x.w + (m + j - x.q);
        *first = i < *first ? i : *first;
        return;
    }
    for (uint32_t bits = sel; bits; bits &= bits - 1u) byte_rows(x, o0 + ((uint64_t)__builtin_ctz(bits) - k0), n, first);
}

// the list entries [i0, i1) against side x, one lane per entry
__device__ __forceinline__ void walk_rows(const uint64_t *chunk, const uint32_t *mask, uint64_t i0, uint64_t i1,
                                          const RowSide &x, uint32_t lane, uint64_t *n, uint64_t *first)
{
    for (uint64_t i = i0 + lane; i < i1; i += 64) chunk_rows(x, chunk[i], mask[i], n, first);
}

__device__ __forceinline__ uint64_t wave_sum(uint64_t v)
{
    for (int k = 32; k >= 1; k >>= 1) v += __shfl_xor(v, k);
    return v;
}

__device__ __forceinline__ uint64_t wave_min(uint64_t v)
{
    for (int k = 32; k >= 1; k >>= 1) {
        const uint64_t o = __shfl_xor(v, k);
        v = o < v ? o : v;
    }
    return v;
}

// Pitched positions whose rows follow row 0 (kRowsUniform: every
// row whole inside row 0's allocation or the host region) in a check without
// propagation, one wave per position.  The list entries between the first
// row's start and the last row's end are mapped onto the rows: undefined
// bytes counted once per row holding them, the first faulty byte by the
// record's row-by-row numbering.  A position whose spaces lack a valid index,
// or whose span holds more entries than a scan of its rows would read
// chunks (and more than 4,096), is left to the scan.
__global__ void __launch_bounds__(kT) k_sidx_rows(BatchArgs a, ShadowIndex h, ShadowIndex p, Pitch *pitch)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t t = (uint64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
    if (!a.out || t >= a.count) return;
    const Pitch P = pitch[t];
    if (P.uniform != kRowsUniform) return;
    const Desc d = a.desc[t];
    const bool src_host = (d.ctl & CTL_SRC_HOST) != 0;
    const bool dsta = (d.ctl & CTL_DST_A) != 0 && d.d_hi > d.d_lo;
    const int64_t w = (int64_t)P.width;
    // row 0 is valid whole on both sides (its verdict has no flags)
    const bool ok = (d.ctl & CTL_CHECK) && !(d.ctl & CTL_PROP) && d.units > 0 && P.rows > 0 && d.v_lo == 0 &&
                    d.v_hi == w && (!dsta || (d.d_lo == 0 && d.d_hi == w)) &&
                    (src_host ? h.state[1] : p.state[1]) && (!dsta || h.state[1]);
    if (!ok) return;
    const ShadowIndex &xs = src_host ? h : p;
    const uint32_t o = desc_o(d);
    const RowSide rs{src_host ? (uint64_t)(d.a_src + (int64_t)o) : d.src_sh + o - a.st->pool, P.rows, P.spitch,
                     P.width};
    const RowSide rd{(uint64_t)(d.a_dst + (int64_t)o), P.rows, P.dpitch, P.width};
    // the chunks of each side's span, first row to last
    const uint64_t sa = rs.S >> 4, sb = (rs.S + (rs.R - 1) * rs.q + rs.w - 1) >> 4;
    const uint64_t da = rd.S >> 4, db = (rd.S + (rd.R - 1) * rd.q + rd.w - 1) >> 4;
    // the six list bounds, one lane each: undefined entries of the source span,
    // unaddressable ones of the host source's and of the host destination's
    uint64_t bound = 0;
    if (lane < 2) bound = lower_bound(xs.uchunk, xs.state[2], lane == 0 ? sa : sb + 1);
    else if (lane < 4 && src_host) bound = lower_bound(h.nchunk, h.state[3], lane == 2 ? sa : sb + 1);
    else if (lane >= 4 && lane < 6 && dsta) bound = lower_bound(h.nchunk, h.state[3], lane == 4 ? da : db + 1);
    const uint64_t i0 = __shfl(bound, 0), i1 = __shfl(bound, 1), j0 = __shfl(bound, 2), j1 = __shfl(bound, 3),
                   k0 = __shfl(bound, 4), k1 = __shfl(bound, 5);
    const uint64_t entries = (i1 - i0) + (j1 - j0) + (k1 - k0);
    const uint64_t chunks = P.rows * ((P.width + 15) >> 4) * (dsta ? 2 : 1);
    if (entries > 4096 && entries > chunks) return;
    uint64_t undef = 0, fu = CG_NONE, fs = CG_NONE, fd = CG_NONE, unused = 0;
    walk_rows(xs.uchunk, xs.umask, i0, i1, rs, lane, &undef, &fu);
    walk_rows(h.nchunk, h.nmask, j0, j1, rs, lane, &unused, &fs);
    walk_rows(h.nchunk, h.nmask, k0, k1, rd, lane, &unused, &fd);
    undef = wave_sum(undef);
    fu = wave_min(fu);
    fs = wave_min(fs);
    fd = wave_min(fd);
    if (lane == 0) {
        cg_verdict v = a.out[t];
        if (undef) v.flags |= CG_SRC_UNDEF;
        if (fs != CG_NONE) v.flags |= CG_SRC_UNADDR;
        if (fd != CG_NONE) v.flags |= CG_DST_UNADDR;
        v.undef_bytes += undef;
        uint64_t first = v.first_bad;
        first = fu < first ? fu : first;
        first = fs < first ? fs : first;
        first = fd < first ? fd : first;
        v.first_bad = first;
        a.out[t] = v;
        a.desc[t].units = 0;
        a.weight[t] = 0;
        pitch[t].upr = 0;
    }
}

}  // namespace

hipError_t launch_sidx_count(const ShadowIndex &h, const ShadowIndex &p, const DevState *st, hipStream_t s)
{
    hipLaunchKernelGGL(k_sidx_count, dim3(h.grid), dim3(kT), 0, s, h, p, st);
    return hipGetLastError();
}

hipError_t launch_sidx_finish(const ShadowIndex &h, const ShadowIndex &p, const DevState *st, hipStream_t s)
{
    hipLaunchKernelGGL(k_sidx_scan, dim3(2), dim3(1024), 0, s, h, p);
    hipLaunchKernelGGL(k_sidx_fill, dim3(h.grid, 2), dim3(kT), 0, s, h, p, st);
    return hipGetLastError();
}

hipError_t launch_sidx_marks(const ShadowIndex &h, const ShadowIndex &p, const DevState *st, hipStream_t s)
{
    const dim3 grid(h.mark_grid > p.mark_grid ? h.mark_grid : p.mark_grid, 2);
    hipLaunchKernelGGL(k_sidx_mark_count, grid, dim3(kMarkT), 0, s, h, p, st);
    hipLaunchKernelGGL(k_sidx_mark_list, grid, dim3(kMarkT), 0, s, h, p, st);
    return hipGetLastError();
}

hipError_t launch_sidx_build(const ShadowIndex &h, const ShadowIndex &p, const DevState *st, hipStream_t s)
{
    hipError_t e = launch_sidx_marks(h, p, st, s);
    if (e == hipSuccess) e = launch_sidx_count(h, p, st, s);
    return e != hipSuccess ? e : launch_sidx_finish(h, p, st, s);
}

hipError_t launch_sidx_query(const BatchArgs &ar, const ShadowIndex &h, const ShadowIndex &p, hipStream_t s,
                             Pitch *pitch)
{
    const uint64_t blocks = (ar.count + kT - 1) / kT;
    hipLaunchKernelGGL(k_sidx_query, dim3((uint32_t)blocks), dim3(kT), 0, s, ar, h, p, pitch);
    if (pitch) {
        const uint64_t wblocks = (ar.count + kT / 64 - 1) / (kT / 64);
        hipLaunchKernelGGL(k_sidx_rows, dim3((uint32_t)wblocks), dim3(kT), 0, s, ar, h, p, pitch);
    }
    return hipGetLastError();
}

}  // namespace xc
