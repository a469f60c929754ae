// HIP kernels of the transfer checker, written for gfx950 (CDNA4, wave64).
//
// The method (Cudagrind, arXiv 1310.0901): every copy is cross-checked
// against the context's list of live device allocations (Sec. 2, Fig. 2
// caption); host source bytes must be addressable and defined, tracked with
// bitwise shadow precision (Sec. 1.1); the report gives the bytes the copy
// needs against the bytes the allocation holds (Sec. 4.5); definedness is
// carried through host/device, device/host and device/device copies (Sec. 5).
//
// Pipeline of one batched check (all integer, bit-exact):
//   k_classify     one lane per record: decode, interval lookup in the
//                  sorted allocation table (top level staged in LDS),
//                  range-derived verdict fields, scan descriptor, work weight,
//                  block-local exclusive scan of the weights; for a check the
//                  shadow indexes may answer, the valid bytes per shadow space
//                  and the marks of the 4 KiB shadow granules they fall in;
//   (shadowindex.hip) large check-only batches: indexes of the faulty chunks
//                  of those steps, which answer the records whose spaces they
//                  cover (their units leave the scan);
//   (segment.hip)  large batches only: every record's units cut at blocks of
//                  source memory, the pieces sorted by block and laid out as
//                  the batch's positions (descriptors, weights, block-local
//                  scan), so that work reading the same bytes runs together;
//                  the kernels below work by position and send findings to
//                  each position's record;
//   k_scan_sums    one block: exclusive scan of the per-block sums, tile size;
//   k_prefix_tiles global prefix; k_tile_starts first record of every tile
//                  (k_plan_tiles: these three in one, up to 262,144 records);
//   k_batched      persistent kernel: tiles of the flattened 16-byte unit space
//                  (one tile per wave when the batch is small), for a
//                  segmented batch one contiguous chunk per XCD, taken from
//                  per-chunk device counters; 16-byte V windows at any
//                  alignment and their A bits, SWAR non-zero masks, popcount /
//                  ctz for the undefined count and first fault, DPP wave
//                  reductions, rare global atomics; optional non-temporal V
//                  store to the destination shadow.
// The plain path runs k_classify once, then k_plain once per record.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "xc_internal.h"

namespace xc {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4u __attribute__((aligned(1)));   // at any byte address
typedef uint32_t u32u __attribute__((aligned(1)));

constexpr uint64_t NONE = CG_NONE;

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------

// Bits j of a 16-byte chunk with lo <= j < hi (offsets relative to the chunk).
__device__ __forceinline__ uint32_t rmask(int64_t lo, int64_t hi)
{
    int64_t l = lo < 0 ? 0 : (lo > 16 ? 16 : lo);
    int64_t h = hi < 0 ? 0 : (hi > 16 ? 16 : hi);
    return h > l ? ((1u << (uint32_t)h) - (1u << (uint32_t)l)) : 0u;
}

// One bit per byte of w: set where the byte is non-zero (SWAR, no carries
// cross byte lanes because every byte sum stays below 0x100).
__device__ __forceinline__ uint32_t nz4(uint32_t w)
{
    uint32_t t = (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u;
    return ((t >> 7) | (t >> 14) | (t >> 21) | (t >> 28)) & 0xFu;
}

__device__ __forceinline__ uint32_t nz16(u32x4 v)
{
    return nz4(v.x) | (nz4(v.y) << 4) | (nz4(v.z) << 8) | (nz4(v.w) << 12);
}

// At the head of a branch that is rarely taken: keeps it a branch.  Worked
// without one, the masks and sums of all of an unrolled loop's windows live in
// registers at once, and half the waves fit.
__device__ __forceinline__ void stay_branched() { asm volatile(""); }

// 4-bit mask -> byte mask (0x00 / 0xFF per byte); the shifted copies of m do
// not overlap, so the multiply has no carries.
__device__ __forceinline__ uint32_t expand4(uint32_t m)
{
    return ((m * 0x00204081u) & 0x01010101u) * 0xFFu;
}

// Value a source chunk contributes to propagation: its V byte where the
// source byte is valid, 0xFF where it is not.
__device__ __forceinline__ u32x4 prop_val(u32x4 v, uint32_t ok)
{
    if (ok == 0xFFFFu) return v;
    stay_branched();
    u32x4 r;
    r.x = v.x | ~expand4(ok & 0xFu);
    r.y = v.y | ~expand4((ok >> 4) & 0xFu);
    r.z = v.z | ~expand4((ok >> 8) & 0xFu);
    r.w = v.w | ~expand4((ok >> 12) & 0xFu);
    return r;
}

// Global (address space 1) views of device addresses, so that the compiler
// emits global_load / global_store rather than flat accesses.
template <typename T> using gptr = __attribute__((address_space(1))) T *;
template <typename T> using gcptr = const __attribute__((address_space(1))) T *;

__device__ __forceinline__ void store_word_masked(uint64_t p, uint32_t w, uint32_t m)
{
    if (m == 0xFu) { *reinterpret_cast<gptr<u32u>>(p) = w; return; }
    gptr<uint8_t> b = reinterpret_cast<gptr<uint8_t>>(p);
    if (m & 1u) b[0] = (uint8_t)w;
    if (m & 2u) b[1] = (uint8_t)(w >> 8);
    if (m & 4u) b[2] = (uint8_t)(w >> 16);
    if (m & 8u) b[3] = (uint8_t)(w >> 24);
}

// Store the bytes of v selected by m at p (any alignment).
__device__ __forceinline__ void store_masked(uint64_t p, u32x4 v, uint32_t m)
{
    if (m == 0xFFFFu) { __builtin_nontemporal_store(v, reinterpret_cast<gptr<u32x4u>>(p)); return; }
    stay_branched();
    if (m & 0x000Fu) store_word_masked(p, v.x, m & 0xFu);
    if (m & 0x00F0u) store_word_masked(p + 4, v.y, (m >> 4) & 0xFu);
    if (m & 0x0F00u) store_word_masked(p + 8, v.z, (m >> 8) & 0xFu);
    if (m & 0xF000u) store_word_masked(p + 12, v.w, (m >> 12) & 0xFu);
}

__device__ __forceinline__ int32_t clamp32(int64_t x)
{
    return x < -(1ll << 30) ? -(1 << 30) : (x > (1ll << 30) ? (1 << 30) : (int32_t)x);
}

// rmask for offsets already clamped to 32 bits
__device__ __forceinline__ uint32_t rmask32(int32_t lo, int32_t hi)
{
    const int32_t l = lo < 0 ? 0 : (lo > 16 ? 16 : lo);
    const int32_t h = hi < 0 ? 0 : (hi > 16 ? 16 : hi);
    return h > l ? ((1u << h) - (1u << l)) : 0u;
}

__device__ __forceinline__ uint32_t ufl32(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ uint64_t ufl64(uint64_t x)
{
    return ((uint64_t)ufl32((uint32_t)(x >> 32)) << 32) | ufl32((uint32_t)x);
}

// *p through scalar loads: p is the same for the whole wave, and the kernel
// does not write what it points at.
template <typename T>
__device__ __forceinline__ T ld_uniform(const T *p)
{
    static_assert(sizeof(T) % 4 == 0, "whole words");
    using cword = const __attribute__((address_space(4))) uint32_t;
    cword *q = reinterpret_cast<cword *>(ufl64(reinterpret_cast<uint64_t>(p)));
    uint32_t w[sizeof(T) / 4];
#pragma unroll
    for (uint32_t k = 0; k < sizeof(T) / 4; ++k) w[k] = q[k];
    T x;
    __builtin_memcpy(&x, w, sizeof(T));
    return x;
}

// ---- DPP wave reductions (every lane of the wave must be active) --------
template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t x)
{
    uint32_t lo = dpp32<CTRL>((uint32_t)x), hi = dpp32<CTRL>((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t readlane64(uint64_t x, int l)
{
    uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
    uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}
// quad_perm [1,0,3,2] = 0xB1, quad_perm [2,3,0,1] = 0x4E, row_half_mirror =
// 0x141, row_mirror = 0x140: after the four steps every lane holds its
// 16-lane row's total; the four rows are combined from lanes 0/16/32/48.
__device__ __forceinline__ uint64_t wave_min64(uint64_t x)
{
    uint64_t y;
    y = dpp64<0xB1>(x); x = y < x ? y : x;
    y = dpp64<0x4E>(x); x = y < x ? y : x;
    y = dpp64<0x141>(x); x = y < x ? y : x;
    y = dpp64<0x140>(x); x = y < x ? y : x;
    uint64_t a = readlane64(x, 0), b = readlane64(x, 16), c = readlane64(x, 32), d = readlane64(x, 48);
    a = b < a ? b : a;
    c = d < c ? d : c;
    return c < a ? c : a;
}
__device__ __forceinline__ uint64_t wave_sum64(uint64_t x)
{
    x += dpp64<0xB1>(x);
    x += dpp64<0x4E>(x);
    x += dpp64<0x141>(x);
    x += dpp64<0x140>(x);
    return readlane64(x, 0) + readlane64(x, 16) + readlane64(x, 32) + readlane64(x, 48);
}
__device__ __forceinline__ uint32_t wave_or32(uint32_t x)
{
    x |= dpp32<0xB1>(x);
    x |= dpp32<0x4E>(x);
    x |= dpp32<0x141>(x);
    x |= dpp32<0x140>(x);
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 0) | (uint32_t)__builtin_amdgcn_readlane((int)x, 16) |
           (uint32_t)__builtin_amdgcn_readlane((int)x, 32) | (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
}

__device__ __forceinline__ uint64_t wave_or64(uint64_t x)
{
    return (uint64_t)wave_or32((uint32_t)x) | ((uint64_t)wave_or32((uint32_t)(x >> 32)) << 32);
}

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// Loads and stores of a window of 16 V bytes at any byte address.  Unaligned 16-byte accesses run at 0.93-1.0 of the aligned rate on gfx950
// (64 MiB and 2 GiB copies at source and destination offsets of 0, 1, 4, 8 and
// 13 bytes), so both sides of a record are read and written in the same
// windows and nothing is realigned in registers.

template <bool NT>
__device__ __forceinline__ u32x4 ld16(uint64_t addr)
{
    gcptr<u32x4u> p = reinterpret_cast<gcptr<u32x4u>>(addr);
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

// The destination shadow is written once and not read again by the batch:
// non-temporal stores keep it out of the caches' way (2 GiB copied with
// non-temporal loads: 889 us with cached stores, 750-800 without).
__device__ __forceinline__ void st16(uint64_t addr, u32x4 v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<gptr<u32x4u>>(addr));
}

__device__ __forceinline__ uint32_t ld_half(uint64_t addr) { return *reinterpret_cast<gcptr<uint16_t>>(addr); }

// A bits [bit, bit + 16) of the bitmap, from one unaligned word inside its nab
// bytes; bits outside it come out as any value.
__device__ __forceinline__ uint32_t ld_a16(uint64_t a16, int64_t nab, int64_t bit)
{
    int64_t b = bit >> 3;
    b = b < 0 ? 0 : (b > nab - 4 ? nab - 4 : b);
    const uint32_t w = *reinterpret_cast<gcptr<u32u>>(a16 + (uint64_t)b);
    const int64_t s = bit - 8 * b;   // -15 .. 31 for bits that matter
    return (s >= 0 ? (s < 32 ? w >> (uint32_t)s : 0u) : w << (uint32_t)(-s & 31)) & 0xFFFFu;
}

__device__ __forceinline__ int64_t a_bytes(const Region &R) { return (int64_t)(((R.hl + 63) >> 6) << 3); }

// The same for windows from bit `bit` on, 16 bits apart, with 32-bit offsets.
struct AWords {
    uint64_t base;         // address of the word of window 0 (which may lie outside the bitmap)
    int32_t lo, hi, s;     // first and last byte offset from there inside the bitmap, first bit in the word
    __device__ __forceinline__ AWords(const Region &R, int64_t bit)
    {
        const int64_t b = bit >> 3;
        base = (uint64_t)R.a16 + (uint64_t)b;
        lo = clamp32(-b);
        hi = clamp32(a_bytes(R) - 4 - b);
        s = (int32_t)(bit & 7);
    }
    // the window 16 w bits on
    __device__ __forceinline__ uint32_t at(int32_t w) const { return word(2 * w, s); }
    // the window n bits on (n >= 0)
    __device__ __forceinline__ uint32_t bits(int32_t n) const { return word((s + n) >> 3, (s + n) & 7); }

private:
    __device__ __forceinline__ uint32_t word(int32_t p, int32_t bit) const
    {
        const int32_t q = p < lo ? lo : (p > hi ? hi : p);
        const uint32_t x = *reinterpret_cast<gcptr<u32u>>(base + (uint64_t)(int64_t)q);
        const int32_t k = bit + 8 * (p - q);   // -16 < k < 32 where any bit matters
        return (k >= 0 ? x >> (uint32_t)(k & 31) : x << (uint32_t)(-k & 31)) & 0xFFFFu;
    }
};

// The 16 bytes s bytes after those of v (before, for s < 0; |s| < 16), with
// zeros where v has none.
__device__ __forceinline__ u32x4 byte_shift(u32x4 v, int32_t s)
{
    uint64_t lo = ((uint64_t)v.y << 32) | v.x, hi = ((uint64_t)v.w << 32) | v.z;
    if (s > 0) {
        if (s >= 8) { lo = hi; hi = 0; s -= 8; }
        if (s) { lo = (lo >> (8 * s)) | (hi << (64 - 8 * s)); hi >>= 8 * s; }
    } else if (s < 0) {
        s = -s;
        if (s >= 8) { hi = lo; lo = 0; s -= 8; }
        if (s) { hi = (hi << (8 * s)) | (lo >> (64 - 8 * s)); lo <<= 8 * s; }
    }
    return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

// ---------------------------------------------------------------------------
// descriptor in registers
// ---------------------------------------------------------------------------
struct DV {
    uint64_t src_sh, dst_sh;
    int64_t v_lo, v_hi, d_lo, d_hi, a_src, a_dst;
    uint64_t e0, units;
    uint32_t ctl, o;
};

__device__ __forceinline__ DV make_dv(const Desc &x)
{
    DV d;
    d.src_sh = x.src_sh; d.dst_sh = x.dst_sh;
    d.v_lo = x.v_lo; d.v_hi = x.v_hi; d.d_lo = x.d_lo; d.d_hi = x.d_hi;
    d.a_src = x.a_src; d.a_dst = x.a_dst; d.e0 = x.e0; d.units = x.units;
    d.ctl = x.ctl;
    d.o = desc_o(x);
    return d;
}

// Per-lane descriptor (lanes may work on different records).
__device__ __forceinline__ DV load_desc(const Desc *D, uint64_t t) { return make_dv(D[t]); }

// Wave-uniform descriptor, in scalar registers.
__device__ __forceinline__ DV load_desc_uniform(const Desc *D, uint64_t t) { return make_dv(ld_uniform(D + t)); }

// The first and the last 16-aligned chunk holding a valid source byte.  A
// window that is only partly valid may reach outside the shadow; it is loaded
// from its address clamped to these two, where every byte is inside the
// allocation's slot or the region's padded V bytes, and shifted into place
// (every valid byte of the window lies in the clamped load).
__device__ __forceinline__ uint64_t src_first(const DV &d) { return (d.src_sh + d.o + (uint64_t)d.v_lo) & ~15ull; }
__device__ __forceinline__ uint64_t src_last(const DV &d) { return (d.src_sh + d.o + (uint64_t)d.v_hi - 1u) & ~15ull; }

// Window e of one lane: V bytes, valid-byte mask, and (host source) the
// in-range bytes whose A bit is 0.  AL: the source's windows are aligned
// chunks, as those of a check without propagation are, pitched rows apart
// (classify_rec); a chunk with a valid byte lies whole in the shadow, and its
// A bits are a half word of their own.
template <bool NT, bool AL>
__device__ __forceinline__ void src_window(const DV &d, const Region &R, int64_t e, u32x4 &v, uint32_t &ok,
                                           uint32_t &unaddr)
{
    const int64_t i0 = 16 * e - (int64_t)d.o;
    const uint32_t m = rmask(d.v_lo - i0, d.v_hi - i0);
    v = u32x4{0u, 0u, 0u, 0u};
    ok = 0u;
    unaddr = 0u;
    if (m) {
        const uint64_t p = d.src_sh + (uint64_t)(16 * e);
        if constexpr (AL) {
            v = ld16<NT>(p);
        } else {
            const uint64_t lo = src_first(d), hi = src_last(d);
            const uint64_t q = p < lo ? lo : (p > hi ? hi : p);
            v = ld16<NT>(q);
            if (p != q) v = byte_shift(v, (int32_t)(int64_t)(p - q));
        }
        if (d.ctl & CTL_SRC_HOST) {
            const uint32_t a = AL ? ld_half((uint64_t)R.a16 + (uint64_t)((d.a_src + 16 * e) >> 3))
                                  : ld_a16((uint64_t)R.a16, a_bytes(R), d.a_src + 16 * e);
            ok = m & a;
            unaddr = m & ~a;
        } else {
            ok = m;
        }
    }
}

struct Acc {
    uint64_t first, undef;
    uint32_t flags;
};

__device__ __forceinline__ void acc_reset(Acc &a) { a.first = NONE; a.undef = 0; a.flags = 0; }

__device__ __forceinline__ void acc_min(Acc &a, int64_t i) { a.first = (uint64_t)i < a.first ? (uint64_t)i : a.first; }

// one 0x80 per non-zero byte of w
__device__ __forceinline__ uint32_t nz80(uint32_t w) { return (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u; }

// Findings of a window whose byte 0 is the record's byte i0 (checking only).
// A lane's windows ascend, so once it has a first fault below i0 only the
// count is left to take (dense shadow: 4 words of 4 operations).
__device__ __forceinline__ void src_findings(Acc &a, int64_t i0, u32x4 v, uint32_t ok, uint32_t unaddr)
{
    if (unaddr) {
        stay_branched();
        a.flags |= CG_SRC_UNADDR;
        acc_min(a, i0 + __builtin_ctz(unaddr));
    }
    if (v.x | v.y | v.z | v.w) {
        stay_branched();
        if (ok == 0xFFFFu && i0 >= 0 && a.first < (uint64_t)i0) {
            a.flags |= CG_SRC_UNDEF;
            a.undef += (uint64_t)(uint32_t)(__builtin_popcount(nz80(v.x)) + __builtin_popcount(nz80(v.y)) +
                                            __builtin_popcount(nz80(v.z)) + __builtin_popcount(nz80(v.w)));
            return;
        }
        const uint32_t und = nz16(v) & ok;
        if (und) {
            a.flags |= CG_SRC_UNDEF;
            a.undef += (uint64_t)__builtin_popcount(und);
            acc_min(a, i0 + __builtin_ctz(und));
        }
    }
}

__device__ __forceinline__ void dst_findings(Acc &a, int64_t i0, uint32_t unaddr)
{
    if (unaddr) {
        stay_branched();
        a.flags |= CG_DST_UNADDR;
        acc_min(a, i0 + __builtin_ctz(unaddr));
    }
}

// Wave-wide flush of uniform-mode accumulators for record t (all lanes active).
__device__ __forceinline__ void flush_wave(Acc &a, cg_verdict *out, uint64_t t)
{
    if (__ballot(a.flags != 0u)) {
        const uint64_t first = wave_min64(a.first);
        const uint64_t und = wave_sum64(a.undef);
        const uint32_t fl = wave_or32(a.flags);
        if (lane_id() == 0) {
            atomicOr(&out[t].flags, fl);
            if (first != NONE) atomicMin((unsigned long long *)&out[t].first_bad, (unsigned long long)first);
            if (und) atomicAdd((unsigned long long *)&out[t].undef_bytes, (unsigned long long)und);
        }
    }
    acc_reset(a);
}

// ---------------------------------------------------------------------------
// uniform mode: the whole wave works on units [k_begin, k_end) of one record
// ---------------------------------------------------------------------------

// Windows 64 j + lane (j < U) of an interior iteration: V from vbase, A words
// of the source (SA) and of the destination (DA) at byte 2 * window of abase /
// dbase, their bits starting at bit ss / ds of the word.
template <int U, bool NT, bool SA, bool DA>
struct Interior {
    u32x4 v[U];
    uint32_t a[U], da[U];
    __device__ __forceinline__ Interior(uint64_t vbase, uint64_t abase, uint32_t ss, uint64_t dbase, uint32_t ds)
    {
        const uint32_t lane = lane_id();
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint32_t w = 64u * j + lane;
            v[j] = ld16<NT>(vbase + 16u * w);
            if constexpr (SA) a[j] = *reinterpret_cast<gcptr<u32u>>(abase + 2u * w);
            if constexpr (DA) da[j] = *reinterpret_cast<gcptr<u32u>>(dbase + 2u * w);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            a[j] = SA ? (a[j] >> ss) & 0xFFFFu : 0xFFFFu;
            da[j] = DA ? (da[j] >> ds) & 0xFFFFu : 0xFFFFu;
        }
    }
    // findings: none when every V byte of the wave's windows is 0 and every A
    // bit 1, which one test over all windows tells
    __device__ __forceinline__ void check(int64_t i0, Acc &acc) const
    {
        uint32_t bad = 0;
#pragma unroll
        for (int j = 0; j < U; ++j) bad |= v[j].x | v[j].y | v[j].z | v[j].w | (a[j] ^ 0xFFFFu) | (da[j] ^ 0xFFFFu);
        if (__ballot(bad != 0u) == 0) return;
        const uint32_t lane = lane_id();
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint32_t w = 64u * j + lane;
            src_findings(acc, i0 + 16 * w, v[j], a[j], a[j] ^ 0xFFFFu);
            if constexpr (DA) dst_findings(acc, i0 + 16 * w, da[j] ^ 0xFFFFu);
        }
    }
    // findings and stores, window 0's first byte being record byte i0 and
    // going to address dst
    __device__ __forceinline__ void carry(bool check, int64_t i0, uint64_t dst, Acc &acc) const
    {
        const uint32_t lane = lane_id();
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint32_t w = 64u * j + lane;
            if (check) {
                src_findings(acc, i0 + 16 * w, v[j], a[j], a[j] ^ 0xFFFFu);
                if constexpr (DA) dst_findings(acc, i0 + 16 * w, da[j] ^ 0xFFFFu);
            }
            const u32x4 x = SA ? prop_val(v[j], a[j]) : v[j];
            if (!DA || da[j] == 0xFFFFu) st16(dst + 16u * w, x);
            else store_masked(dst + 16u * w, x, da[j]);
        }
    }
};

// Units [kb, kb + 64 G) of a record below k_end, by the whole wave, at its
// edges: windows that are only partly valid, or not at all, are masked, and
// loaded from clamped addresses (lanes without a valid byte read some valid
// chunk and ignore it), so that all G loads go out back to back.
template <int G, bool NT, bool PROP>
__device__ __forceinline__ void run_edge(const DV &d, const Region &R, uint64_t kb, uint64_t k_end, Acc &acc)
{
    const int32_t lane = (int32_t)lane_id();
    const bool check = (d.ctl & CTL_CHECK) != 0;
    const bool prop = PROP && (d.ctl & CTL_PROP) != 0;
    const bool dsta = (d.ctl & CTL_DST_A) != 0;
    const bool src_host = (d.ctl & CTL_SRC_HOST) != 0;
    const bool dst_host = (d.ctl & CTL_DST_HOST) != 0;
    constexpr int32_t W = 16 * 64 * G;   // bytes worked
    const int64_t eb = (int64_t)(d.e0 + kb);
    const int64_t i0b = 16 * eb - (int64_t)d.o;
    const int32_t vlo = clamp32(d.v_lo - i0b), vhi = clamp32(d.v_hi - i0b);
    const int32_t dlo = clamp32(d.d_lo - i0b), dhi = clamp32(d.d_hi - i0b);
    const int32_t kend = clamp32((int64_t)(k_end - kb));
    u32x4 v[G];
    uint32_t ok[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
        v[j] = u32x4{0u, 0u, 0u, 0u};
        ok[j] = 0u;
    }
    if (vlo < W && vhi > 0 && vhi > vlo) {   // some window holds a valid byte
        const uint64_t vbase = d.src_sh + (uint64_t)(16 * eb);
        const int32_t lo = clamp32((int64_t)(src_first(d) - vbase)), hi = clamp32((int64_t)(src_last(d) - vbase));
        bool moved = false;
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int32_t p = 16 * (64 * j + lane);
            const int32_t q = p < lo ? lo : (p > hi ? hi : p);
            v[j] = ld16<NT>(vbase - 16u + (uint32_t)(q + 16));   // q >= -15
            moved |= p != q;
        }
        if (src_host) {
            const AWords A(R, d.a_src + 16 * eb);
#pragma unroll
            for (int j = 0; j < G; ++j) ok[j] = A.at(64 * j + lane);
        } else {
#pragma unroll
            for (int j = 0; j < G; ++j) ok[j] = 0xFFFFu;
        }
        if (__ballot(moved)) {
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const int32_t p = 16 * (64 * j + lane);
                const int32_t q = p < lo ? lo : (p > hi ? hi : p);
                if (p != q && p - q < 16 && q - p < 16) v[j] = byte_shift(v[j], p - q);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < G; ++j) {
        const int32_t cr = 64 * j + lane;
        const uint32_t m = cr < kend ? rmask32(vlo - 16 * cr, vhi - 16 * cr) : 0u;
        const uint32_t un = m & ~ok[j];
        ok[j] &= m;
        if (check) src_findings(acc, i0b + 16 * cr, v[j], ok[j], un);
    }
    if ((dsta || prop) && dlo < W && dhi > 0) {
        const uint64_t dbase = d.dst_sh + (uint64_t)(16 * eb);
        const AWords A(R, d.a_dst + 16 * eb);
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int32_t cr = 64 * j + lane;
            const uint32_t md = cr < kend ? rmask32(dlo - 16 * cr, dhi - 16 * cr) : 0u;
            uint32_t wm = md;
            if (dst_host) {
                wm = md & A.at(cr);
                if (check) dst_findings(acc, i0b + 16 * cr, md & ~wm);
            }
            if (prop && wm) store_masked(dbase + (uint64_t)(uint32_t)(16 * cr), prop_val(v[j], ok[j]), wm);
        }
    }
}

// The wave's iterations start at k_begin and are `step` units apart.  Lane l
// of sub-iteration j handles unit kb + 64 j + l: window e = e0 + kb + 64 j + l
// of both sides.  Per iteration all offsets are taken relative to the first
// unit, in 32 bits.
template <int U, bool NT, bool PROP>
__device__ __forceinline__ void run_uniform(const DV &d, const Region &R, uint64_t k_begin, uint64_t k_end,
                                            Acc &acc, uint64_t step = 64u * U)
{
    const bool check = (d.ctl & CTL_CHECK) != 0;
    const bool prop = PROP && (d.ctl & CTL_PROP) != 0;
    const bool dsta = (d.ctl & CTL_DST_A) != 0;
    const bool src_host = (d.ctl & CTL_SRC_HOST) != 0;
    const bool dst_host = (d.ctl & CTL_DST_HOST) != 0;
    const uint64_t a16b = (uint64_t)R.a16;
    const int64_t nab = a_bytes(R);
    constexpr int32_t W = 16 * 64 * U;   // bytes per iteration
    constexpr int G = U < 2 ? 1 : 2;
    k_begin = ufl64(k_begin);   // (in scalar registers, so that all the offsets below are)
    k_end = ufl64(k_end);
    step = ufl64(step);

    for (uint64_t kb = k_begin; kb < k_end; kb += step) {
        const int64_t eb = (int64_t)(d.e0 + kb);
        const int64_t i0b = 16 * eb - (int64_t)d.o;
        // Interior iteration: every window lies wholly inside the valid source
        // range and, where the destination is worked, inside its valid range
        // (and the A words inside the bitmap), so no byte mask or clamp is
        // needed.
        const int64_t sbit = d.a_src + 16 * eb, dbit = d.a_dst + 16 * eb;
        bool in = d.v_lo <= i0b && d.v_hi >= i0b + W && k_end - kb >= 64u * U;
        if (src_host) in &= sbit >= 0 && ((sbit + W) >> 3) + 4 <= nab;
        if (dsta || prop) in &= d.d_lo <= i0b && d.d_hi >= i0b + W;
        if (dst_host && (dsta || prop)) in &= dbit >= 0 && ((dbit + W) >> 3) + 4 <= nab;
        if (in && (PROP ? prop : check)) {
            // (a host destination has a device source, a host source a device destination)
            const uint64_t vbase = d.src_sh + (uint64_t)(16 * eb), dbase = d.dst_sh + (uint64_t)(16 * eb);
            const uint64_t sab = a16b + (uint64_t)(sbit >> 3), dab = a16b + (uint64_t)(dbit >> 3);
            const uint32_t ss = (uint32_t)sbit & 7u, ds = (uint32_t)dbit & 7u;
            if constexpr (PROP) {
                if (src_host) Interior<U, NT, true, false>(vbase, sab, ss, 0, 0).carry(check, i0b, dbase, acc);
                else if (dst_host) Interior<U, NT, false, true>(vbase, 0, 0, dab, ds).carry(check, i0b, dbase, acc);
                else Interior<U, NT, false, false>(vbase, 0, 0, 0, 0).carry(check, i0b, dbase, acc);
            } else {
                if (dsta) Interior<U, NT, false, true>(vbase, 0, 0, dab, ds).check(i0b, acc);
                else if (src_host) Interior<U, NT, true, false>(vbase, sab, ss, 0, 0).check(i0b, acc);
                else Interior<U, NT, false, false>(vbase, 0, 0, 0, 0).check(i0b, acc);
            }
            continue;
        }
        // (two windows per lane at a time: four would cost the registers that
        // let twice the waves run)
#pragma nounroll
        for (uint64_t k = kb; k < kb + 64u * U && k < k_end; k += 64u * G)
            run_edge<G, NT, PROP>(d, R, k, k_end < kb + 64u * U ? k_end : kb + 64u * U, acc);
    }
}

// run_edge for a check whose source windows are aligned chunks: the chunks of
// lanes without a valid byte are loaded at the nearest that has one, the A
// bits with them, and nothing is shifted, so that four windows fit a lane.
template <int G, bool NT>
__device__ __forceinline__ void check_edge(const DV &d, const Region &R, uint64_t kb, uint64_t k_end, Acc &acc)
{
    const int32_t lane = (int32_t)lane_id();
    const bool src_host = (d.ctl & CTL_SRC_HOST) != 0;
    constexpr int32_t W = 16 * 64 * G;   // bytes worked
    const int64_t eb = (int64_t)(d.e0 + kb);
    const int64_t i0b = 16 * eb - (int64_t)d.o;
    const int32_t vlo = clamp32(d.v_lo - i0b), vhi = clamp32(d.v_hi - i0b);
    const int32_t kend = clamp32((int64_t)(k_end - kb));
    u32x4 v[G];
    uint32_t ok[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
        v[j] = u32x4{0u, 0u, 0u, 0u};
        ok[j] = 0xFFFFu;
    }
    const int32_t clo = (vlo >> 4) > 0 ? (vlo >> 4) : 0;
    const int32_t chi = ((vhi + 15) >> 4) < 64 * G ? ((vhi + 15) >> 4) : 64 * G;
    // (a record without a valid source byte has no source chunk to load)
    if (vhi > vlo && chi > clo) {   // some chunk holds a valid byte
        const uint64_t vbase = d.src_sh + (uint64_t)(16 * eb);
        const uint64_t abase = (uint64_t)R.a16 + (uint64_t)((d.a_src + 16 * eb) >> 3);
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int32_t c = 64 * j + lane;
            const int32_t cc = c < clo ? clo : (c >= chi ? chi - 1 : c);
            v[j] = ld16<NT>(vbase + (uint32_t)(16 * cc));
            if (src_host) ok[j] = ld_half(abase + (uint32_t)(2 * cc));
        }
    }
#pragma unroll
    for (int j = 0; j < G; ++j) {
        const int32_t cr = 64 * j + lane;
        const uint32_t m = cr < kend ? rmask32(vlo - 16 * cr, vhi - 16 * cr) : 0u;
        src_findings(acc, i0b + 16 * cr, v[j], m & ok[j], m & ~ok[j]);
    }
    if (d.ctl & CTL_DST_A) {
        const int32_t dlo = clamp32(d.d_lo - i0b), dhi = clamp32(d.d_hi - i0b);
        if (dlo < W && dhi > 0) {
            const AWords A(R, d.a_dst + 16 * eb);
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const int32_t cr = 64 * j + lane;
                const uint32_t md = cr < kend ? rmask32(dlo - 16 * cr, dhi - 16 * cr) : 0u;
                dst_findings(acc, i0b + 16 * cr, md & ~A.at(cr));
            }
        }
    }
}

// The wave's windows 64 j + lane (j < U) of an interior iteration of a check:
// V from vbase; the A bits of a host source are half words from abase on, those
// of a host destination start at bit ds of the words there (a host destination
// has a device source, a host source a device destination).
template <int U, bool NT>
__device__ __forceinline__ void check_interior(uint64_t vbase, uint64_t abase, bool src_host, bool dsta, uint32_t ds,
                                               int64_t i0, Acc &acc)
{
    // (one address for all windows: 1,024 V bytes further is the instruction's own offset)
    const uint32_t lane = lane_id();
    vbase += 16u * lane;
    abase += 2u * lane;
    i0 += 16 * (int64_t)lane;
    u32x4 v[U];
    uint32_t a[U];
#pragma unroll
    for (int j = 0; j < U; ++j) v[j] = ld16<NT>(vbase + 1024u * j);
#pragma unroll
    for (int j = 0; j < U; ++j) a[j] = 0xFFFFu;
    if (src_host) {
#pragma unroll
        for (int j = 0; j < U; ++j) a[j] = ld_half(abase + 128u * j);
    } else if (dsta) {
#pragma unroll
        for (int j = 0; j < U; ++j) a[j] = (*reinterpret_cast<gcptr<u32u>>(abase + 128u * j) >> ds) & 0xFFFFu;
    }
    // no finding when every V byte is 0 and every A bit 1, which one test over
    // all windows tells
    uint32_t bad = 0;
#pragma unroll
    for (int j = 0; j < U; ++j) bad |= v[j].x | v[j].y | v[j].z | v[j].w | (a[j] ^ 0xFFFFu);
    if (__ballot(bad != 0u) == 0) return;
#pragma unroll
    for (int j = 0; j < U; ++j) {
        if (dsta) dst_findings(acc, i0 + 1024 * j, a[j] ^ 0xFFFFu);
        src_findings(acc, i0 + 1024 * j, v[j], src_host ? a[j] : 0xFFFFu, src_host ? a[j] ^ 0xFFFFu : 0u);
    }
}

// run_uniform for the checks of check_transfers; G windows a lane at a
// record's edges.  A batch whose records read
// the same bytes again and again takes them from the caches at 20 TB/s, where
// the waves' instructions count: the interior iterations follow each other, so
// their range is found once per call, and an iteration is its loads, one test
// and one address (with the ranges tested per iteration, by the code that
// serves any alignment, about 100 instructions and 40 more registers).  1M mixed
// records without an index, in segments, 64 KiB tiles, cached loads: 69.2 ms with
// that code, 55.5 so; with the host's segments in LDS 64.2 and 52.7, and in 1 MiB
// tiles with non-temporal loads 69.5 and 64.3.  4,096 records of 64 KiB in one
// launch 67 and 55 us.
template <int U, bool NT, int G = (U > 4 ? 4 : U)>
__device__ __forceinline__ void run_check(const DV &d, const Region &R, uint64_t k_begin, uint64_t k_end, Acc &acc,
                                          uint64_t step = 64u * U)
{
    const bool dsta = (d.ctl & CTL_DST_A) != 0;
    const bool src_host = (d.ctl & CTL_SRC_HOST) != 0;
    const uint64_t a16b = (uint64_t)R.a16;
    constexpr uint64_t N = 64u * U;   // units per iteration
    k_begin = ufl64(k_begin);
    k_end = ufl64(k_end);
    step = ufl64(step);
    // units [in_lo, in_hi) have interior windows
    const int64_t o = (int64_t)d.o;
    int64_t lo = d.v_lo, hi = d.v_hi;
    if (dsta) {
        const int64_t last = 8 * (a_bytes(R) - 4) - d.a_dst - o;   // the A words lie inside the bitmap up to here
        lo = lo > d.d_lo ? lo : d.d_lo;
        hi = hi < d.d_hi ? hi : d.d_hi;
        hi = hi < last ? hi : last;
    }
    const int64_t in_lo = ((lo + o + 15) >> 4) - (int64_t)d.e0;
    int64_t in_hi = ((hi + o) >> 4) - (int64_t)d.e0;
    in_hi = in_hi < (int64_t)k_end ? in_hi : (int64_t)k_end;
    uint64_t kb = k_begin;
    while (kb < k_end) {
        if ((int64_t)kb >= in_lo && (int64_t)(kb + N) <= in_hi) {
            for (; (int64_t)(kb + N) <= in_hi; kb += step) {
                const int64_t e = (int64_t)(d.e0 + kb), bit = (src_host ? d.a_src : d.a_dst) + 16 * e;
                check_interior<U, NT>(d.src_sh + (uint64_t)(16 * e), a16b + (uint64_t)(bit >> 3), src_host, dsta,
                                      (uint32_t)bit & 7u, 16 * e - o, acc);
            }
            continue;
        }
        const uint64_t ke = k_end < kb + N ? k_end : kb + N;
#pragma nounroll
        for (uint64_t k = kb; k < ke; k += 64u * G) check_edge<G, NT>(d, R, k, ke, acc);
        kb += step;
    }
}

// a record that is no pitched row
template <int U, bool NT, bool PROP>
__device__ __forceinline__ void run_units(const DV &d, const Region &R, uint64_t k_begin, uint64_t k_end, Acc &acc,
                                          uint64_t step = 64u * U)
{
    if constexpr (PROP) run_uniform<U, NT, true>(d, R, k_begin, k_end, acc, step);
    else run_check<U, NT>(d, R, k_begin, k_end, acc, step);
}

// ---------------------------------------------------------------------------
// one unit handled by one lane (small records, tile boundaries)
// ---------------------------------------------------------------------------
template <bool NT, bool PROP, bool AL>
__device__ __forceinline__ void run_unit(const DV &d, const Region &R, uint64_t k, Acc &acc)
{
    const bool check = (d.ctl & CTL_CHECK) != 0;
    const int64_t e = (int64_t)(d.e0 + k);
    const int64_t i0 = 16 * e - (int64_t)d.o;
    u32x4 v;
    uint32_t ok, un;
    src_window<NT, AL>(d, R, e, v, ok, un);
    if (check) src_findings(acc, i0, v, ok, un);
    if (d.ctl & (CTL_DST_A | CTL_PROP)) {
        const uint32_t md = rmask(d.d_lo - i0, d.d_hi - i0);
        uint32_t wm = md;
        if ((d.ctl & CTL_DST_HOST) && md) {
            wm = md & ld_a16((uint64_t)R.a16, a_bytes(R), d.a_dst + 16 * e);
            if (check) dst_findings(acc, i0, md & ~wm);
        }
        if (PROP && (d.ctl & CTL_PROP) && wm) store_masked(d.dst_sh + (uint64_t)(16 * e), prop_val(v, ok), wm);
    }
}

// Segmented flush: lanes hold findings for records `rec` (contiguous runs of
// equal values; inactive lanes carry rec = ~0).  Only called when some lane
// found something.
__device__ __forceinline__ void flush_segmented(Acc &a, uint64_t rec, cg_verdict *out)
{
    const uint32_t lane = lane_id();
    const uint64_t prev = __shfl_up(rec, 1);
    const bool head = lane == 0u || prev != rec;
    const uint64_t heads = __ballot(head);
    const uint64_t below = heads & (lane == 63u ? ~0ull : ((2ull << lane) - 1ull));
    const uint32_t start = 63u - (uint32_t)__builtin_clzll(below);
    for (uint32_t dd = 1; dd < 64u; dd <<= 1) {
        const uint64_t of = __shfl_up(a.first, dd);
        const uint64_t ou = __shfl_up(a.undef, dd);
        const uint32_t ofl = __shfl_up(a.flags, dd);
        if (lane >= dd && lane - dd >= start) {
            a.first = of < a.first ? of : a.first;
            a.undef += ou;
            a.flags |= ofl;
        }
    }
    const uint64_t next = __shfl_down(rec, 1);
    const bool tail = lane == 63u || next != rec;
    if (tail && rec != ~0ull && a.flags) {
        atomicOr(&out[rec].flags, a.flags);
        if (a.first != NONE) atomicMin((unsigned long long *)&out[rec].first_bad, (unsigned long long)a.first);
        if (a.undef) atomicAdd((unsigned long long *)&out[rec].undef_bytes, (unsigned long long)a.undef);
    }
    acc_reset(a);
}

// ---------------------------------------------------------------------------
// k_classify
// ---------------------------------------------------------------------------

// Largest index j with base[j] <= p among live allocations, if p < end[j].
__device__ __forceinline__ int64_t table_lookup(const TableView &tb, const uint64_t *top, uint64_t p)
{
    if (tb.n == 0 || top[0] > p) return -1;
    uint32_t lo = 0, hi = tb.ntop - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (top[mid] <= p) lo = mid; else hi = mid - 1;
    }
    uint64_t a = (uint64_t)lo << tb.top_shift;
    uint64_t b = a + (1ull << tb.top_shift);
    b = (b < tb.n ? b : tb.n) - 1;
    while (a < b) {
        const uint64_t mid = (a + b + 1) >> 1;
        if (tb.base[mid] <= p) a = mid; else b = mid - 1;
    }
    return p < tb.end[a] ? (int64_t)a : -1;
}

// wave-wide sum of a 32-bit value (every lane active)
__device__ __forceinline__ uint32_t wave_add32(uint32_t x)
{
    for (int d = 32; d >= 1; d >>= 1) x += (uint32_t)__shfl_xor((int)x, d);
    return x;
}

// The table search of table_lookup done by one wave (every lane active): the
// top level, then the segment of 2^top_shift entries it picks, are each
// compared 64 entries at a time, so two rounds of independent loads take the
// place of a chain of dependent ones.  Entries are sorted by base, so the
// number of them at or below p is one past the last of them.
__device__ __forceinline__ int64_t table_lookup_wave(const TableView &tb, uint64_t p)
{
    if (tb.n == 0) return -1;
    const uint32_t lane = lane_id();
    uint32_t c = 0;
    for (uint32_t k = lane; k < tb.ntop; k += 64) c += tb.top[k] <= p ? 1u : 0u;
    c = wave_add32(c);
    if (c == 0) return -1;
    const uint64_t a0 = (uint64_t)(c - 1) << tb.top_shift;
    const uint64_t a1 = a0 + (1ull << tb.top_shift) < tb.n ? a0 + (1ull << tb.top_shift) : tb.n;
    uint32_t c2 = 0;
    for (uint64_t k = a0 + lane; k < a1; k += 64) c2 += tb.base[k] <= p ? 1u : 0u;
    c2 = wave_add32(c2);
    const uint64_t j = a0 + c2 - 1;   // base[a0] is top[c - 1] <= p, so c2 >= 1
    return p < tb.end[j] ? (int64_t)j : -1;
}

// Byte indices i in [0, n) with hb <= p + i < hb + hl, as [lo, hi) (empty: 0, 0).
__device__ __forceinline__ void region_clip(uint64_t p, uint64_t n, uint64_t hb, uint64_t hl,
                                            uint64_t &lo, uint64_t &hi)
{
    lo = hi = 0;
    if (hl == 0) return;
    if (p >= hb) {
        const uint64_t off = p - hb;
        if (off >= hl) return;
        lo = 0;
        hi = (n < hl - off) ? n : hl - off;
    } else {
        const uint64_t gap = hb - p;
        if (gap >= n) return;
        lo = gap;
        hi = (n - gap > hl) ? gap + hl : n;
    }
}

__device__ __forceinline__ uint64_t clamp_scan(uint64_t x) { return x < kScanLimit ? x : kScanLimit; }

// does the record have a device source / destination to look up?
__device__ __forceinline__ bool dev_src(const cg_transfer &r) { return r.kind <= CG_D2D && r.n && r.kind != CG_H2D; }
__device__ __forceinline__ bool dev_dst(const cg_transfer &r) { return r.kind <= CG_D2D && r.n && r.kind != CG_D2H; }

// Decode record r, given the table entries holding its device source and
// destination pointers (js, jd: -1 when none, or when the side is on the
// host): its descriptor, its verdict's range-derived fields, and its number
// of units (returned).  With `row`, the record is a row that others follow at
// any pitch: its windows start at its first byte (o = 0).
__device__ __forceinline__ uint64_t classify_rec(const cg_transfer &r, uint32_t mode, const DevState &st, int64_t js, int64_t jd,
                                 Desc &ds, cg_verdict &v, bool row = false)
{
    const uint64_t n = r.n;
    ds = Desc{};
    uint32_t flags = 0;
    uint64_t first = NONE, avail = 0;
    const bool check = (mode & CG_CHECK) != 0;
    uint64_t units = 0;

    if (r.kind > CG_D2D) {
        flags = CG_BAD_KIND;
    } else if (n != 0) {
        const bool src_host = r.kind == CG_H2D;
        const bool dst_host = r.kind == CG_D2H;
        const Region &R = st.region;
        uint64_t vlo = 0, vhi = 0, dlo = 0, dhi = 0, avail_s = 0, avail_d = 0;
        uint64_t src0 = 0, dst0 = 0;   // shadow address of byte 0 (when valid)
        bool src_ok = false, dst_ok = false;
        if (src_host) {
            region_clip(r.src, n, R.hb, R.hl, vlo, vhi);
            if (vhi <= vlo || vlo > 0) { flags |= CG_SRC_UNADDR; first = 0; }
            else if (vhi < n) { flags |= CG_SRC_UNADDR; first = first < vhi ? first : vhi; }
            src_ok = vhi > vlo;
            src0 = (uint64_t)R.v + (r.src - R.hb);
            ds.a_src = (int64_t)(r.src - R.hb);
        } else {
            const int64_t j = js;
            if (j < 0) { flags |= CG_SRC_UNALLOC; first = 0; }
            else {
                avail_s = st.table.end[j] - r.src;
                if (n > avail_s) { flags |= CG_SRC_OVERRUN; first = first < avail_s ? first : avail_s; }
                vlo = 0;
                vhi = n < avail_s ? n : avail_s;
                src0 = st.pool + st.table.off[j] + (r.src - st.table.base[j]);
                src_ok = true;
            }
        }
        if (dst_host) {
            region_clip(r.dst, n, R.hb, R.hl, dlo, dhi);
            if (dhi <= dlo || dlo > 0) { flags |= CG_DST_UNADDR; first = 0; }
            else if (dhi < n) { flags |= CG_DST_UNADDR; first = first < dhi ? first : dhi; }
            dst_ok = dhi > dlo;
            dst0 = (uint64_t)R.v + (r.dst - R.hb);
            ds.a_dst = (int64_t)(r.dst - R.hb);
        } else {
            const int64_t j = jd;
            if (j < 0) { flags |= CG_DST_UNALLOC; first = 0; }
            else {
                avail_d = st.table.end[j] - r.dst;
                if (n > avail_d) { flags |= CG_DST_OVERRUN; first = first < avail_d ? first : avail_d; }
                dlo = 0;
                dhi = n < avail_d ? n : avail_d;
                dst0 = st.pool + st.table.off[j] + (r.dst - st.table.base[j]);
                dst_ok = true;
            }
        }
        bool overlap = false;
        if (r.kind == CG_D2D) {
            overlap = (r.src < r.dst) ? (r.dst - r.src < n) : (r.src - r.dst < n);
            if (overlap) flags |= CG_OVERLAP;
        }
        avail = src_host ? avail_d : (dst_host ? avail_s : (avail_s < avail_d ? avail_s : avail_d));

        const bool prop = (mode & CG_PROPAGATE) && !overlap;
        const bool dsta = check && dst_host;
        const bool dstwork = (prop || dsta) && dst_ok;
        vlo = clamp_scan(vlo); vhi = clamp_scan(vhi);
        dlo = clamp_scan(dlo); dhi = clamp_scan(dhi);
        // the windows align the destination when it is written, else the source
        const uint32_t o = row ? 0u : (uint32_t)((prop && dst_ok) || !src_ok ? dst0 : src0) & 15u;
        // windows of the source's and of the destination's valid bytes
        uint64_t e_lo = ~0ull, e_hi = 0;
        if (src_ok && vhi > vlo) {
            e_lo = (vlo + o) >> 4;
            e_hi = ((vhi - 1 + o) >> 4) + 1;
            // propagation needs every destination window, including those whose
            // bytes come only from invalid source bytes (written as 0xFF)
        }
        if (dstwork && dhi > dlo) {
            const uint64_t f_lo = (dlo + o) >> 4, f_hi = ((dhi - 1 + o) >> 4) + 1;
            e_lo = f_lo < e_lo ? f_lo : e_lo;
            e_hi = f_hi > e_hi ? f_hi : e_hi;
        }
        if (e_hi > e_lo) units = e_hi - e_lo; else e_lo = 0;
        ds.src_sh = src0 - o;
        ds.dst_sh = dst0 - o;
        ds.a_src -= (int64_t)o;
        ds.a_dst -= (int64_t)o;
        ds.v_lo = (int64_t)vlo; ds.v_hi = (int64_t)vhi;
        ds.d_lo = (int64_t)dlo; ds.d_hi = (int64_t)dhi;
        ds.e0 = e_lo;
        ds.units = units;
        ds.ctl = (src_host ? CTL_SRC_HOST : 0u) | (dst_host ? CTL_DST_HOST : 0u) | (check ? CTL_CHECK : 0u) |
                 (prop && dst_ok ? CTL_PROP : 0u) | (dsta && dst_ok ? CTL_DST_A : 0u) | (o << CTL_O_SHIFT);
        if (!src_ok) { ds.v_lo = 0; ds.v_hi = 0; }
    }
    v.flags = flags;
    v.reserved = 0;
    v.first_bad = first;
    v.undef_bytes = 0;
    v.avail = avail;
    return units;
}

// Marks the granules (2^12 bytes of V) of shadow space k that hold its bytes
// [lo, hi), for that index's counting pass: a byte per granule of the steps
// (2^16 bytes) at the range's ends, a byte for every step it covers whole, 16
// per store.  Plain byte-masked stores merge in memory whichever XCD's L2 they
// leave from; granule bits set by atomics, which all meet in one place, took
// 310 us for 1M records.
__device__ __forceinline__ void mark_steps(const BatchArgs &a, int k, uint64_t lo, uint64_t hi)
{
    uint8_t *m = a.index_mark[k];
    if (!m || hi <= lo) return;
    constexpr uint32_t sh = kIdxStepShift - kIdxGranShift;
    const uint64_t g0 = lo >> kIdxGranShift, g1 = ((hi - 1) >> kIdxGranShift) + 1;   // granules [g0, g1)
    uint64_t s = g0 >> sh, e = g1 >> sh;                                             // steps [s, e) start to end
    // granules [x, x + n) of one step, n < 16, by at most two stores
    auto part = [&](uint64_t x, uint32_t n) {
        if (n == 0 || (x >> sh) >= a.mark_cap[k]) return;
        uint8_t *f = a.index_fine[k] + x;
        typedef uint64_t u64u __attribute__((aligned(1)));
        typedef uint16_t u16u __attribute__((aligned(1)));
        if (n >= 8) {
            *reinterpret_cast<u64u *>(f) = *reinterpret_cast<u64u *>(f + n - 8) = 0x0101010101010101ull;
        } else if (n >= 4) {
            *reinterpret_cast<u32u *>(f) = *reinterpret_cast<u32u *>(f + n - 4) = 0x01010101u;
        } else if (n >= 2) {
            *reinterpret_cast<u16u *>(f) = *reinterpret_cast<u16u *>(f + n - 2) = (uint16_t)0x0101u;
        } else {
            f[0] = 1;
        }
    };
    if (s == e) {
        part(g0, (uint32_t)(g1 - g0));
        return;
    }
    if (g0 & 15u) {
        part(g0, 16u - (uint32_t)(g0 & 15u));
        ++s;
    }
    part(g1 & ~15ull, (uint32_t)(g1 & 15u));
    if (e > a.mark_cap[k]) e = a.mark_cap[k];
    for (; s < e && (s & 15u); ++s) m[s] = 1;
    for (; s + 16 <= e; s += 16) *reinterpret_cast<uint4 *>(m + s) = make_uint4(0x01010101u, 0x01010101u, 0x01010101u, 0x01010101u);
    for (; s < e; ++s) m[s] = 1;
}

// space offsets of a descriptor's byte 0: of its source (host region or pool)
// and of a host destination
__device__ __forceinline__ uint64_t src_space_off(const Desc &ds, const DevState &st)
{
    return (ds.ctl & CTL_SRC_HOST) ? (uint64_t)(ds.a_src + (int64_t)desc_o(ds)) : ds.src_sh + desc_o(ds) - st.pool;
}

__device__ __forceinline__ uint64_t dst_space_off(const Desc &ds) { return (uint64_t)(ds.a_dst + (int64_t)desc_o(ds)); }

// the steps a transfer's index answer reads: its valid source bytes, and a
// host destination's valid bytes
__device__ __forceinline__ void mark_desc(const BatchArgs &a, const DevState &st, const Desc &ds)
{
    if (ds.v_hi > ds.v_lo) {
        const uint64_t o = src_space_off(ds, st);
        mark_steps(a, (ds.ctl & CTL_SRC_HOST) ? 0 : 1, o + (uint64_t)ds.v_lo, o + (uint64_t)ds.v_hi);
    }
    if ((ds.ctl & CTL_DST_A) && ds.d_hi > ds.d_lo) {
        const uint64_t o = dst_space_off(ds);
        mark_steps(a, 0, o + (uint64_t)ds.d_lo, o + (uint64_t)ds.d_hi);
    }
}

// Record t of a batch: its descriptor and work weight, and its verdict's
// range-derived fields; returns its number of units (and in sp[0], sp[1] its
// valid bytes in the host region and in the shadow pool, when sp is given).
__device__ uint64_t classify_one(const BatchArgs &a, const DevState &st, uint64_t t, const uint64_t *top,
                                 uint64_t *sp = nullptr)
{
    const cg_transfer r = a.recs[t];
    const int64_t js = dev_src(r) ? table_lookup(st.table, top, r.src) : -1;
    const int64_t jd = dev_dst(r) ? table_lookup(st.table, top, r.dst) : -1;
    Desc ds;
    cg_verdict v;
    const uint64_t units = classify_rec(r, a.mode, st, js, jd, ds, v);
    if (sp) {
        const uint64_t src = ds.v_hi > ds.v_lo ? (uint64_t)(ds.v_hi - ds.v_lo) : 0;
        const uint64_t dst = (ds.ctl & CTL_DST_A) && ds.d_hi > ds.d_lo ? (uint64_t)(ds.d_hi - ds.d_lo) : 0;
        sp[0] = ((ds.ctl & CTL_SRC_HOST) ? src : 0) + dst;
        sp[1] = (ds.ctl & CTL_SRC_HOST) ? 0 : src;
        mark_desc(a, st, ds);
    }
    a.desc[t] = ds;
    a.weight[t] = units;
    if (a.out && (a.mode & CG_CHECK)) a.out[t] = v;
    return units;
}

__device__ __forceinline__ void clear_left(const BatchArgs &a, uint32_t tid)
{
    if (a.index_bytes[0] && blockIdx.x == 0 && tid == 0) a.index_bytes[0][kIdxLeft] = 0;
}

__global__ void __launch_bounds__(kClassifyBlock) k_classify(BatchArgs a)
{
    __shared__ uint64_t top[kMaxTop];
    __shared__ uint64_t wsum[kClassifyBlock / 64];
    __shared__ uint64_t isum[2][kClassifyBlock / 64];
    const uint32_t tid = threadIdx.x;
    clear_left(a, tid);
    const DevState st = *a.st;
    for (uint32_t k = tid; k < st.table.ntop; k += kClassifyBlock) top[k] = st.table.top[k];
    __syncthreads();
    const uint64_t t = (uint64_t)blockIdx.x * kClassifyBlock + tid;
    uint64_t w = 0, sp[2] = {0, 0};
    if (t < a.count) {
        const uint64_t u = classify_one(a, st, t, top, sp);
        w = u ? u : 1;
    }
    const uint32_t lane = lane_id(), wid = tid >> 6;
    if (a.index_bytes[0]) {
        // the batch's valid bytes per shadow space (the shadow indexes' cost
        // test): wave sums here, one atomic per block below
        for (int k = 0; k < 2; ++k) {
            uint64_t x = sp[k];
            for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d);
            if (lane == 0) isum[k][wid] = x;
        }
    }
    // block exclusive scan of w
    uint64_t x = w;
    for (uint32_t d = 1; d < 64u; d <<= 1) {
        const uint64_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63u) wsum[wid] = x;
    __syncthreads();
    uint64_t off = 0;
    for (uint32_t k = 0; k < wid; ++k) off += wsum[k];
    if (t < a.count) a.local[t] = off + x - w;
    if (tid == kClassifyBlock - 1) a.bsum[blockIdx.x] = off + x;
    if (a.index_bytes[0] && tid == 0)
        for (int k = 0; k < 2; ++k) {
            uint64_t b = 0;
            for (uint32_t q = 0; q < kClassifyBlock / 64; ++q) b += isum[k][q];
            if (b) atomicAdd((unsigned long long *)a.index_bytes[k], (unsigned long long)b);
        }
}

// After the shadow indexes have answered pitched positions (their weight set
// to 0): each position's weight max(units, 1) again, with the block-local
// prefix and block sums that k_classify leaves, and the units left to scan.
__global__ void __launch_bounds__(kClassifyBlock) k_reweigh(BatchArgs a)
{
    __shared__ uint64_t wsum[kClassifyBlock / 64];
    const uint32_t tid = threadIdx.x;
    const uint64_t t = (uint64_t)blockIdx.x * kClassifyBlock + tid;
    uint64_t w = 0, u = 0;
    if (t < a.count) {
        u = a.weight[t];
        w = u ? u : 1;
    }
    if (__syncthreads_or(u != 0) && tid == 0) atomicOr((unsigned long long *)&a.index_bytes[0][kIdxLeft], 1ull);
    const uint32_t lane = lane_id(), wid = tid >> 6;
    uint64_t x = w;
    for (uint32_t d = 1; d < 64u; d <<= 1) {
        const uint64_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63u) wsum[wid] = x;
    __syncthreads();
    uint64_t off = 0;
    for (uint32_t k = 0; k < wid; ++k) off += wsum[k];
    if (t < a.count) a.local[t] = off + x - w;
    if (tid == kClassifyBlock - 1) a.bsum[blockIdx.x] = off + x;
}

// ---------------------------------------------------------------------------
// pitched 2D records (check_transfers_2d) as positions of their own
// ---------------------------------------------------------------------------


// rows of a 2D record that are worked: every row below index 2^32 that
// starts below byte 2^62 of the record (its bytes are numbered row by row)
__device__ __forceinline__ uint64_t rows_worked(const cg_transfer2d &r)
{
    if (r.width == 0 || r.rows == 0) return 0;
    const uint64_t lim = r.width >= kScanLimit ? 1 : (kScanLimit + r.width - 1) / r.width;
    uint64_t n = r.rows < lim ? r.rows : lim;
    return n < (1ull << 32) ? n : (1ull << 32);
}

// A bound of the bytes from any row's start to the end of that row's valid
// source and destination parts, for a record whose rows do not follow row 0:
// a device side ends within its allocation (none is larger than
// st.size_bound); a host side ends within the region, at most `gap + hl`
// bytes from a row that starts `gap` bytes below it.  The host side's rows
// start no lower than row 0 unless their addresses wrap past 2^64.
__device__ __forceinline__ uint64_t row_extent_bound(const Pitch &P, uint64_t rows, const DevState &st)
{
    uint64_t e = st.size_bound;
    if (P.kind == CG_H2D || P.kind == CG_D2H) {
        const Region &R = st.region;
        const uint64_t p = P.kind == CG_H2D ? P.src : P.dst, q = P.kind == CG_H2D ? P.spitch : P.dpitch;
        const bool wraps = q != 0 && rows > 1 && rows - 1 > (~0ull - p) / q;
        const uint64_t gap = wraps ? R.hb : (p < R.hb ? R.hb - p : 0);
        const uint64_t h = gap + R.hl;
        e = e > h ? e : h;
    }
    return e;
}

// do rows 0 .. n-1 of one side, starting at p with pitch q and `w` bytes
// long, all lie in [lo, hi)?  (p >= lo is known)
__device__ __forceinline__ bool rows_inside(uint64_t p, uint64_t q, uint64_t w, uint64_t n, uint64_t lo, uint64_t hi)
{
    (void)lo;
    if (p >= hi || w > hi - p) return false;
    if (n <= 1 || q == 0) return true;
    return n - 1 <= (hi - p - w) / q;   // p + (n-1) q + w <= hi
}

// the transfer record of row r
__device__ __forceinline__ cg_transfer row_record(const Pitch &P, uint64_t r)
{
    return cg_transfer{P.src + r * P.spitch, P.dst + r * P.dpitch, P.width, P.kind, 0u};
}

// The steps the index answer of a record whose rows follow row 0 reads: on
// each side, the span from the first row's start to the last row's end when
// it is at most 4 times the rows' bytes (plus 4 steps); a sparser side asks
// for every step of its space instead, so that marking stays within a
// fraction of the bytes the rows hold.
__device__ __forceinline__ void mark_rows(const BatchArgs &a, const DevState &st, const Desc &ds, const Pitch &P)
{
    auto side = [&](int k, uint64_t o, uint64_t q) {
        const uint64_t span = (P.rows - 1) * q + P.width;
        if (span / 4 <= P.rows * P.width + (4ull << kIdxStepShift)) mark_steps(a, k, o, o + span);
        else a.index_bytes[k][kIdxAll] = 1;
    };
    if (ds.v_hi > ds.v_lo) side((ds.ctl & CTL_SRC_HOST) ? 0 : 1, src_space_off(ds, st), P.spitch);
    if ((ds.ctl & CTL_DST_A) && ds.d_hi > ds.d_lo) side(0, dst_space_off(ds), P.dpitch);
}

// Whether the windows of a pitched record's rows that follow row 0 are aligned
// chunks of their sources, each row at its own phase: in a check without
// propagation, where nothing is written at the windows' places.  A host
// source's A bits are then half words as well and no window is shifted.  Rows
// of up to 16 bytes whose pitch does not keep row 0's phase stay one window
// from their start each instead of two chunks.  Without an index, windows from
// the rows' starts and aligned chunks: 4,096 copies of 1,280 rows of 4,032 bytes
// at 4,096, 6.84 and 3.62 ms; 20,480 rows of 240 at 256, 7.00 and 3.72; 1,000
// copies of 1,237 rows of 4,000 at 4,041, 1.70 and 0.84, to the host 1.92 and
// 1.36; 50,000 of 17 at 33, 616 and 306 us; 100,000 of 16 at 17, to the host, 656
// and 791.
__device__ __forceinline__ bool rows_aligned(uint32_t mode, const Pitch &P)
{
    return !(mode & CG_PROPAGATE) && ((P.spitch & 15u) == 0 || P.width > 16);
}

// One lane per pitched 2D record: row 0 looked up and classified (its
// descriptor is the position's), whether every row follows from it, the
// units (rows * upr) and the verdict before any row is worked: row 0's when
// the rows are uniform, else {0, NONE, 0, row 0's avail} (the rows bring
// their own flags), with ROWS_LIMIT when not every row is worked.  A record
// with no rows or width 0 gives {0, NONE, 0, 0}, one with rows and a bad
// kind {BAD_KIND, NONE, 0, 0}; both weigh 1 and have no units.  upr bounds
// the units of every row: a uniform row's follow from the width, any other
// row's from the extent of its valid parts (so a bogus width costs no more
// than the memory its rows can reach).
__global__ void __launch_bounds__(kClassifyBlock) k_classify_2d(BatchArgs a, const cg_transfer2d *recs2d, Pitch *pitch)
{
    __shared__ uint64_t top[kMaxTop];
    __shared__ uint64_t wsum[kClassifyBlock / 64];
    __shared__ uint64_t isum[2][kClassifyBlock / 64];
    uint64_t ib[2] = {0, 0};   // this record's valid bytes per shadow space (the indexes' cost test)
    const uint32_t tid = threadIdx.x;
    clear_left(a, tid);
    const DevState st = *a.st;
    for (uint32_t k = tid; k < st.table.ntop; k += kClassifyBlock) top[k] = st.table.top[k];
    __syncthreads();
    const uint64_t t = (uint64_t)blockIdx.x * kClassifyBlock + tid;
    uint64_t w = 0;
    if (t < a.count) {
        const cg_transfer2d R2 = recs2d[t];
        Pitch P{R2.src, R2.dst, R2.width, R2.rows, R2.spitch, R2.dpitch, 0, R2.kind, 0};
        Desc ds = {};
        cg_verdict v{0u, 0u, NONE, 0, 0};
        uint64_t units = 0;
        const uint64_t rows = rows_worked(R2);
        if (rows == 0) {
            // nothing to check
        } else if (R2.kind > CG_D2D) {
            v.flags = CG_BAD_KIND;
        } else {
            const cg_transfer r0 = row_record(P, 0);
            const int64_t js = dev_src(r0) ? table_lookup(st.table, top, r0.src) : -1;
            const int64_t jd = dev_dst(r0) ? table_lookup(st.table, top, r0.dst) : -1;
            cg_verdict v0;
            classify_rec(r0, a.mode, st, js, jd, ds, v0, !rows_aligned(a.mode, P));
            const Region &R = st.region;
            auto side_ok = [&](bool host, int64_t j, uint64_t p, uint64_t q) {
                if (host) return R.hl > 0 && p >= R.hb && rows_inside(p, q, P.width, rows, R.hb, R.hb + R.hl);
                return j >= 0 && rows_inside(p, q, P.width, rows, st.table.base[j], st.table.end[j]);
            };
            const bool uniform = (v0.flags & ~CG_OVERLAP) == 0 && (R2.kind != CG_D2D || R2.spitch == R2.dpitch) &&
                                 side_ok(R2.kind == CG_H2D, js, P.src, P.spitch) &&
                                 side_ok(R2.kind == CG_D2H, jd, P.dst, P.dpitch);
            P.rows = rows;
            uint64_t ext = P.width < kScanLimit ? P.width : kScanLimit;
            if (!uniform) {
                const uint64_t b = row_extent_bound(P, rows, st);
                ext = b < ext ? b : ext;
            }
            // rows that follow row 0 all have its units, or, in aligned chunks that
            // each row's own phase gives, at most (width + 14) / 16 + 1; any other
            // row at most (ext + 14) / 16 + 2, the most any alignment gives
            P.upr = !uniform ? (ext + 14) / 16 + 2
                    : rows_aligned(a.mode, P) && (P.spitch & 15u) ? (P.width + 14) / 16 + 1 : ds.units;
            P.uniform = uniform ? kRowsUniform : 0u;
            // rows back to back on every side the check reads: one transfer
            // (in the rows' allocations, so its lookups are row 0's)
            if (uniform && !(a.mode & CG_PROPAGATE) && R2.spitch == R2.width &&
                (R2.kind != CG_D2H || R2.dpitch == R2.width)) {
                const cg_transfer rc{P.src, P.dst, rows * P.width, P.kind, 0u};
                cg_verdict vc;
                P.upr = classify_rec(rc, a.mode, st, js, jd, ds, vc);
                P.uniform = kRowsContig;
            }
            units = P.uniform == kRowsContig ? P.upr : rows * P.upr;
            if (P.uniform && a.index_bytes[0]) {
                // the valid bytes read per shadow space, for the indexes' cost
                // test: one transfer's, or row 0's times the rows
                const uint64_t nr = P.uniform == kRowsContig ? 1 : rows;
                const uint64_t src = ds.v_hi > ds.v_lo ? nr * (uint64_t)(ds.v_hi - ds.v_lo) : 0;
                const uint64_t dst = (ds.ctl & CTL_DST_A) && ds.d_hi > ds.d_lo ? nr * (uint64_t)(ds.d_hi - ds.d_lo) : 0;
                ib[0] = ((ds.ctl & CTL_SRC_HOST) ? src : 0) + dst;
                ib[1] = (ds.ctl & CTL_SRC_HOST) ? 0 : src;
                if (P.uniform == kRowsContig) mark_desc(a, st, ds);
                else mark_rows(a, st, ds, P);
            }
            v = uniform ? v0 : cg_verdict{0u, 0u, NONE, 0, v0.avail};
            if (rows < R2.rows) v.flags |= CG_ROWS_LIMIT;
        }
        pitch[t] = P;
        a.desc[t] = ds;
        a.weight[t] = units;
        if (a.out && (a.mode & CG_CHECK)) a.out[t] = v;
        w = units ? units : 1;
    }
    const uint32_t lane = lane_id(), wid = tid >> 6;
    if (a.index_bytes[0])
        for (int k = 0; k < 2; ++k) {
            uint64_t y = ib[k];
            for (int d = 32; d >= 1; d >>= 1) y += __shfl_xor(y, d);
            if (lane == 0) isum[k][wid] = y;
        }
    uint64_t x = w;
    for (uint32_t d = 1; d < 64u; d <<= 1) {
        const uint64_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63u) wsum[wid] = x;
    __syncthreads();
    uint64_t off = 0;
    for (uint32_t k = 0; k < wid; ++k) off += wsum[k];
    if (t < a.count) a.local[t] = off + x - w;
    if (tid == kClassifyBlock - 1) a.bsum[blockIdx.x] = off + x;
    // one atomic per block and space for the cost test
    if (a.index_bytes[0] && tid == 0)
        for (int k = 0; k < 2; ++k) {
            uint64_t b = 0;
            for (uint32_t q = 0; q < kClassifyBlock / 64; ++q) b += isum[k][q];
            if (b) atomicAdd((unsigned long long *)a.index_bytes[k], (unsigned long long)b);
        }
}

// Row r's descriptor when the rows are uniform: row 0's moved by the pitches.
__device__ __forceinline__ Desc row_desc(const Desc &d0, const Pitch &P, uint64_t r)
{
    Desc x = d0;
    x.src_sh += r * P.spitch;
    x.dst_sh += r * P.dpitch;
    x.a_src += (int64_t)(r * P.spitch);
    x.a_dst += (int64_t)(r * P.dpitch);
    return x;
}

// every field of a wave-uniform descriptor in scalar registers
__device__ __forceinline__ DV dv_uniform(const Desc &x)
{
    Desc u;
    u.src_sh = ufl64(x.src_sh); u.dst_sh = ufl64(x.dst_sh);
    u.v_lo = (int64_t)ufl64((uint64_t)x.v_lo); u.v_hi = (int64_t)ufl64((uint64_t)x.v_hi);
    u.d_lo = (int64_t)ufl64((uint64_t)x.d_lo); u.d_hi = (int64_t)ufl64((uint64_t)x.d_hi);
    u.a_src = (int64_t)ufl64((uint64_t)x.a_src); u.a_dst = (int64_t)ufl64((uint64_t)x.a_dst);
    u.e0 = ufl64(x.e0); u.units = ufl64(x.units); u.ctl = ufl32(x.ctl);
    return make_dv(u);
}

// Row r's descriptor when the rows' windows are aligned chunks (rows_aligned),
// each row's at the phase of its own source.
__device__ __forceinline__ DV row_chunks(const DV &d0, const Pitch &P, uint64_t r)
{
    DV d = d0;
    const uint64_t s = d0.src_sh + d0.o + r * P.spitch;
    d.o = (uint32_t)s & 15u;
    const int64_t ro = (int64_t)d0.o - (int64_t)d.o;
    d.src_sh = s - d.o;
    d.a_src += ro + (int64_t)(r * P.spitch);
    d.a_dst += ro + (int64_t)(r * P.dpitch);
    d.units = ((P.width - 1 + d.o) >> 4) + 1;
    return d;
}

// findings of one row (row-relative byte indices) into a record's
// accumulator: byte c of row r is byte r * width + c of the record
__device__ __forceinline__ void acc_add_row(Acc &acc, const Acc &ra, uint32_t rflags, uint64_t rfirst, uint64_t base)
{
    acc.flags |= ra.flags | rflags;
    acc.undef += ra.undef;
    if (ra.first != NONE) acc_min(acc, (int64_t)(base + ra.first));
    if (rfirst != NONE) acc_min(acc, (int64_t)(base + rfirst));
}

// ---------------------------------------------------------------------------
// k_pointers: pointer queries (kernel arguments) against the live allocations
// ---------------------------------------------------------------------------
// Bound by lines fetched at random from beyond L2 (the table is larger than
// an XCD's 4 MB) and by the latency of dependent loads.  So as many steps of
// the search as fit run in LDS: each workgroup stages the table's middle level
// (up to 8,192 bases, 64 KiB: two workgroups of 16 waves per CU).  What is
// below it is searched in global memory four ways at a time: for a million
// allocations the 8 entries of the fine level (every 16th base, small enough
// to stay in L2), then the 16 bases of one line, so that a pointer costs two
// lines from beyond L2, its bases' and its end's.  One search answers both
// questions: the last base at or below p belongs to the allocation that holds
// p or, when none does, to the one that p may be one past the end of (an
// allocation ending at p with a later base at or below p would overlap it).
// 1,000,000 pointers against 965,250 allocations: 67 us; 133 us with a top
// level of 1,024 entries, two searches and binary steps; 81 to 73 us with
// 16,384 entries and four to two pointers per thread (half the waves per CU).

// The last entry of a at or below p among [lo, hi), where a[lo] <= p and
// hi <= lo + w, in rounds of three loads.
__device__ __forceinline__ uint64_t search4(const uint64_t *a, uint64_t w, uint64_t p, uint64_t lo, uint64_t hi)
{
    while (w > 1) {
        const uint64_t q = (w + 3) >> 2;
        uint64_t b[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) b[j] = lo + (j + 1) * q < hi ? a[lo + (j + 1) * q] : ~0ull;
        uint64_t c = 0;
#pragma unroll
        for (int j = 0; j < 3; ++j) c += lo + (j + 1) * q < hi && b[j] <= p ? 1u : 0u;
        lo += c * q;
        hi = lo + q < hi ? lo + q : hi;
        w = q;
    }
    return lo;
}

// Few pointers (`few`) stage the top level of 1,024 entries instead: a few
// thousand lookups do not repay 64 KiB (335 pointers against 11,734
// allocations: 13.2 us with the middle level, 12.1 with the top level).  Where
// the line lies matters little: 262,143 pointers (top level) and 262,144
// (middle level) took 10.8 and 10.6 us against 1,000 allocations, 12.9 and 12.3
// against 10,000, 15.7 and 16.1 against 100,000, 25.1 and 24.2 against 975,000.
__global__ void __launch_bounds__(1024) k_pointers(const DevState *stp, const uint64_t *ptrs, uint64_t count,
                                                   cg_ptr_check *out, bool few)
{
    extern __shared__ uint64_t smid[];
    const TableView tb = stp->table;
    const uint64_t *level = few ? tb.top : tb.mid;
    const uint32_t nl = few ? tb.ntop : tb.nmid, lsh = few ? tb.top_shift : tb.mid_shift;
    for (uint32_t k = threadIdx.x; k < nl; k += blockDim.x) smid[k] = level[k];
    __syncthreads();
    const uint32_t half = nl ? 1u << (31u - (uint32_t)__builtin_clz(nl)) : 0u;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += stride) {
        const uint64_t p = ptrs[t];
        uint32_t pos = 0;   // staged entries at or below p
        for (uint32_t s = half; s; s >>= 1)
            if (pos + s <= nl && smid[pos + s - 1] <= p) pos += s;
        cg_ptr_check o;
        o.flags = CG_PTR_UNALLOC;
        o.reserved = 0;
        o.base = 0;
        o.avail = 0;
        if (pos) {
            uint64_t j = (uint64_t)(pos - 1) << lsh;
            uint32_t sh = lsh;
            if (sh > kFineShift) {
                const uint64_t nf = (tb.n + (1ull << kFineShift) - 1) >> kFineShift;
                const uint64_t f = j >> kFineShift, f1 = f + (1ull << (sh - kFineShift));
                j = search4(tb.fine, 1ull << (sh - kFineShift), p, f, f1 < nf ? f1 : nf) << kFineShift;
                sh = kFineShift;
            }
            const uint64_t j1 = j + (1ull << sh);
            j = search4(tb.base, 1ull << sh, p, j, j1 < tb.n ? j1 : tb.n);
            const uint64_t base = tb.base[j], end = tb.end[j];
            if (p <= end) {
                o.flags = 0;
                o.base = base;
                o.avail = end - p;
            }
        }
        out[t] = o;
    }
}

// MI355X has 8 XCDs, each with its own L2; the blocks of a launch are placed
// on them round robin (block b on XCD b mod 8).
constexpr uint32_t kXcds = 8;
constexpr uint64_t kNoTile = ~0ull;

// A batch worked as segments (lds_meta not null) is worked by k_batched_lds,
// unless it was left in its order: then by k_batched, as one chunk.  Both are
// launched, and one of them leaves at once.
__device__ __forceinline__ bool lds_works(const BatchArgs &a) { return a.lds_meta && a.lds_meta[3] == 0; }

// The tile size of `total` units: tile_units while every wave of the
// persistent grid gets a few of them; otherwise one equal tile per wave, which
// the waves take by their index (354 MB in 2,000 requests: 20,000 tiles of the
// least size, taken one by one from a counter, 216 us; one per wave, 90 us);
// and few enough to fit tile_start.
__device__ __forceinline__ uint64_t tile_size(uint64_t total, uint32_t tile_units, uint32_t waves, uint64_t cap)
{
    uint64_t tu = tile_units;
    if ((total + tu - 1) / tu < waves) {
        tu = ((total + waves - 1) / waves + 63) & ~63ull;
        if (tu < kMinTile) tu = kMinTile;
    }
    while ((total + tu - 1) / tu > cap) tu <<= 1;
    return tu;
}

__device__ __forceinline__ void put_tiles(const BatchArgs &a, uint64_t total, uint64_t tu)
{
    a.ctl->total_units = total;
    a.ctl->tile_units = tu;
    a.ctl->ntiles = (total + tu - 1) / tu;
    for (int x = 0; x < kXcds; ++x) {
        a.ctl->counter[x] = 0;
        a.ctl->lds_counter[x] = 0;
    }
    a.prefix[a.count] = total;
}

// The shadow indexes' states back to 0 for the next batch, except whether
// units are left (kIdxLeft, which every block of k_plan_tiles reads here and
// the next classify clears): when they answered every record, the scan has no
// tile.
__device__ __forceinline__ void reset_states(const BatchArgs &a, uint32_t tid)
{
    if (tid < 2 * kIdxState && tid != kIdxLeft) a.index_bytes[tid / kIdxState][tid % kIdxState] = 0;
}

// ---------------------------------------------------------------------------
// k_scan_sums: one block, exclusive scan of the classify-block sums
// ---------------------------------------------------------------------------
// (waves: of the scan kernel's grid, or of k_batched_lds's for a batch that it works)
__global__ void __launch_bounds__(1024) k_scan_sums(BatchArgs a, uint32_t tile_units, uint32_t waves, uint32_t lds_waves)
{
    if (lds_works(a)) waves = lds_waves;
    __shared__ uint64_t wsum[16];
    const uint32_t tid = threadIdx.x, lane = lane_id(), wid = tid >> 6;
    if (a.index_bytes[0]) {
        reset_states(a, tid);
        if (a.index_bytes[0][kIdxLeft] == 0) {
            if (tid == 0) put_tiles(a, 0, kMinTile);
            return;
        }
    }
    const uint64_t nb = (a.count + kClassifyBlock - 1) / kClassifyBlock;
    const uint64_t per = (nb + 1023) / 1024;
    const uint64_t b0 = tid * per, b1 = (b0 + per < nb) ? b0 + per : nb;
    uint64_t s = 0;
    for (uint64_t b = b0; b < b1; ++b) s += a.bsum[b];
    uint64_t x = s;
    for (uint32_t d = 1; d < 64u; d <<= 1) {
        const uint64_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63u) wsum[wid] = x;
    __syncthreads();
    uint64_t off = 0;
    for (uint32_t k = 0; k < wid; ++k) off += wsum[k];
    uint64_t run = off + x - s;
    for (uint64_t b = b0; b < b1; ++b) {
        a.boff[b] = run;
        run += a.bsum[b];
    }
    if (tid == 1023) {
        const uint64_t total = off + x;
        const uint64_t tu = tile_size(total, tile_units, waves, a.tiles_cap);
        put_tiles(a, total, tu);
    }
}

// ---------------------------------------------------------------------------
// k_prefix_tiles: global prefix; k_tile_starts: first record of every tile
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_prefix_tiles(BatchArgs a)
{
    const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= a.count || a.ctl->ntiles == 0) return;
    a.prefix[t] = a.local[t] + a.boff[t / kClassifyBlock];
}

// One lane per tile (grid-stride): the last record whose prefix is at or
// below the tile's first unit.  Prefixes strictly increase (weights >= 1)
// except over a tail of empty positions of weight 0 (a segmented batch),
// where they equal the total, above every unit.
__global__ void __launch_bounds__(256) k_tile_starts(BatchArgs a)
{
    const uint64_t ntiles = a.ctl->ntiles, tu = a.ctl->tile_units;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < ntiles; j += stride) {
        const uint64_t u = j * tu;
        uint64_t lo = 0, hi = a.count - 1;
        while (lo < hi) {
            const uint64_t mid = (lo + hi + 1) >> 1;
            if (a.prefix[mid] <= u) lo = mid; else hi = mid - 1;
        }
        a.tile_start[j] = (uint32_t)lo;
    }
}

// ---------------------------------------------------------------------------
// k_plan_tiles: the three kernels above in one, for up to kPlanSums classify
// blocks.  Every block scans the block sums for itself, in LDS, and so needs no
// other block's result: a tile's first record is searched among the block sums
// in LDS and then in that block's local prefixes.  Each of the three took
// about 4.7 us, nearly all of it the launch: 2,000 requests 135.2 -> 131.4 us,
// 800 pitched copies of 2,000 rows 182.9 -> 178.7.  (Block 0 resets the states while the
// others still read: they read kIdxLeft only, which stays.  With the last
// block to finish, found by a counter, as the one to reset: no gain.)
// ---------------------------------------------------------------------------
constexpr uint32_t kPlanSums = 1024, kPlanGrid = 256;
__global__ void __launch_bounds__(256) k_plan_tiles(BatchArgs a, uint32_t tile_units, uint32_t waves,
                                                    uint32_t lds_waves)
{
    if (lds_works(a)) waves = lds_waves;
    __shared__ uint64_t boff[kPlanSums], wsum[4];
    const uint32_t tid = threadIdx.x, lane = lane_id(), wid = tid >> 6;
    if (a.index_bytes[0]) {
        if (blockIdx.x == 0) reset_states(a, tid);
        if (a.index_bytes[0][kIdxLeft] == 0) {
            if (blockIdx.x == 0 && tid == 0) put_tiles(a, 0, kMinTile);
            return;
        }
    }
    const uint32_t nb = (uint32_t)((a.count + kClassifyBlock - 1) / kClassifyBlock);
    const uint32_t per = (nb + 255) / 256, b0 = tid * per;
    uint64_t v[kPlanSums / 256], sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < kPlanSums / 256; ++k) {
        v[k] = k < per && b0 + k < nb ? a.bsum[b0 + k] : 0;
        sum += v[k];
    }
    uint64_t x = sum;
    for (uint32_t d = 1; d < 64u; d <<= 1) {
        const uint64_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63u) wsum[wid] = x;
    __syncthreads();
    uint64_t run = x - sum, total = 0;
    for (uint32_t k = 0; k < 4; ++k) {
        if (k < wid) run += wsum[k];
        total += wsum[k];
    }
#pragma unroll
    for (uint32_t k = 0; k < kPlanSums / 256; ++k) {
        if (k < per && b0 + k < nb) boff[b0 + k] = run;
        run += v[k];
    }
    __syncthreads();
    const uint64_t tu = tile_size(total, tile_units, waves, a.tiles_cap), ntiles = (total + tu - 1) / tu;
    if (blockIdx.x == 0 && tid == 0) put_tiles(a, total, tu);
    const uint64_t t = (uint64_t)blockIdx.x * kClassifyBlock + tid;
    if (t < a.count) a.prefix[t] = a.local[t] + boff[blockIdx.x];
    for (uint64_t j = (uint64_t)blockIdx.x * 256 + tid; j < ntiles; j += (uint64_t)gridDim.x * 256) {
        const uint64_t u = j * tu;
        uint32_t lo = 0, hi = nb - 1;
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (boff[mid] <= u) lo = mid; else hi = mid - 1;
        }
        const uint64_t t0 = (uint64_t)lo * kClassifyBlock, w = u - boff[lo];
        lo = 0;
        hi = (uint32_t)(a.count - t0 < kClassifyBlock ? a.count - t0 : kClassifyBlock) - 1;
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (a.local[t0 + mid] <= w) lo = mid; else hi = mid - 1;
        }
        a.tile_start[j] = (uint32_t)t0 + lo;
    }
}

// ---------------------------------------------------------------------------
// k_batched: persistent kernel over the tiles of the flattened unit space
// ---------------------------------------------------------------------------

// Units [k0, k1) of a pitched record whose rows follow row 0 and have fewer
// than kFlatUnits units each, by the whole wave: the rows' units follow each
// other with no gap (upr is a row's units), and each lane works its own unit
// of an iteration in whichever row it falls, so that short rows and row ends
// share iterations.  d is row 0's descriptor (o = 0 here); row r's source and
// destination lie r * spitch and r * dpitch further on, at any alignment (a
// check takes this way for rows of up to 16 bytes at most: rows_aligned).
// Every byte of a row is valid; only a row's last window may pass its end.
// Offsets are taken from the iteration's first row, in 32 bits (24-bit
// products run at full rate), so the pitches are below kFlatPitch; rows
// further apart are worked row by row, or one unit per lane when they are
// short: each of them is in pages of its own, and their loads' latency bounds
// either way.  333-byte rows at 512 bytes carried: 482 us one unit per lane
// with its row's descriptor, 140 us flat.
constexpr uint64_t kFlatUnits = 4096, kFlatPitch = 1u << 20;

__device__ __forceinline__ bool rows_flat(const Pitch &P)
{
    return P.uniform == kRowsUniform && P.upr < kFlatUnits && (P.spitch | P.dpitch) < kFlatPitch;
}

// run_rows_flat for a check whose rows' windows are aligned chunks
// (rows_aligned): nothing is shifted, and one test over all windows tells that
// a wave has no finding.  A row whose phase gives one chunk fewer than upr
// loads its last one twice and keeps it once.
template <int U, bool NT>
__device__ __forceinline__ void check_rows_flat(const DV &d, const Pitch &P, const Region &R, uint64_t k0, uint64_t k1,
                                                Acc &acc)
{
    const uint32_t lane = lane_id();
    const uint32_t ur = (uint32_t)P.upr;
    const uint32_t inv = ufl32((uint32_t)(0xFFFFFFFFu / ur) + 1u);   // n * inv >> 32 = n / ur for n < 2^13 (ur > 1)
    const uint32_t sp = (uint32_t)P.spitch, dp = (uint32_t)P.dpitch;
    const int32_t width = (int32_t)P.width;
    const bool src_host = (d.ctl & CTL_SRC_HOST) != 0;
    const bool dsta = (d.ctl & CTL_DST_A) != 0;
    k0 = ufl64(k0);
    k1 = ufl64(k1);
    uint64_t rb = ufl64(k0 / ur);
    uint32_t jb = ufl32((uint32_t)(k0 - rb * ur));   // row and unit of the iteration's first unit
    for (uint64_t kb = k0; kb < k1; kb += 64u * U) {
        // row rb's first chunk, the row's start in it, and the chunk's A bits
        const uint64_t s = d.src_sh + d.o + rb * sp, sb = s & ~15ull;
        const uint32_t so = (uint32_t)s & 15u;
        const uint64_t ab = (uint64_t)R.a16 + ((uint64_t)(d.a_src + (int64_t)(d.o + rb * sp) - (int64_t)so) >> 3);
        const uint32_t left = k1 - kb < 64u * U ? (uint32_t)(k1 - kb) : 64u * U;
        u32x4 v[U];
        uint32_t a[U], x[U];
        int32_t i[U];   // the window's first byte in its row
#pragma unroll
        for (int j = 0; j < U; ++j) {
            // (lanes past the end work the last unit again and keep nothing)
            const uint32_t c = 64u * j + lane;
            const uint32_t n = jb + (c < left ? c : left - 1);
            x[j] = ur > 1 ? __umulhi(n, inv) : n;   // rows past rb
            const uint32_t b = __umul24(x[j], sp) + so;
            i[j] = 16 * (int32_t)(n - __umul24(x[j], ur)) - (int32_t)(b & 15u);
            const uint32_t rel = b + (uint32_t)(i[j] < width ? i[j] : i[j] - 16);
            v[j] = ld16<NT>(sb + rel);
            a[j] = src_host ? ld_half(ab + (rel >> 3)) : 0xFFFFu;
        }
        if (dsta) {
            // (from 16 bits before row rb: a window may start before its row)
            const AWords A(R, d.a_dst + (int64_t)(d.o + rb * dp) - 16);
#pragma unroll
            for (int j = 0; j < U; ++j) a[j] = A.bits((int32_t)__umul24(x[j], dp) + i[j] + 16);
        }
        uint32_t bad = 0;
#pragma unroll
        for (int j = 0; j < U; ++j) bad |= v[j].x | v[j].y | v[j].z | v[j].w | (a[j] ^ 0xFFFFu);
        if (__ballot(bad != 0u)) {
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const uint32_t m = 64u * j + lane < left ? rmask32(-i[j], width - i[j]) : 0u;
                const int64_t i0 = (int64_t)((rb + x[j]) * P.width) + i[j];
                if (dsta) dst_findings(acc, i0, m & ~a[j]);
                src_findings(acc, i0, v[j], src_host ? m & a[j] : m, src_host ? m & ~a[j] : 0u);
            }
        }
        const uint32_t n = jb + 64u * U, dx = ur > 1 ? __umulhi(n, inv) : n;
        rb += ufl32(dx);
        jb = ufl32(n - dx * ur);
    }
}

template <int U, bool NT, bool PROP>
__device__ __forceinline__ void run_rows_flat(const DV &d, const Pitch &P, const Region &R, uint64_t k0, uint64_t k1,
                                              Acc &acc)
{
    const uint32_t lane = lane_id();
    const uint32_t ur = (uint32_t)P.upr;
    const uint32_t inv = ufl32((uint32_t)(0xFFFFFFFFu / ur) + 1u);   // n * inv >> 32 = n / ur for n < 2^13 (ur > 1)
    const uint32_t width = (uint32_t)P.width, sp = (uint32_t)P.spitch, dp = (uint32_t)P.dpitch;
    const bool check = (d.ctl & CTL_CHECK) != 0;
    const bool prop = PROP && (d.ctl & CTL_PROP) != 0;
    const bool src_host = (d.ctl & CTL_SRC_HOST) != 0;
    const bool dst_host = (d.ctl & CTL_DST_HOST) != 0;
    const bool dwork = prop || (d.ctl & CTL_DST_A) != 0;
    // the last row's last chunk: no load passes it
    const uint64_t last = (d.src_sh + (P.rows - 1) * P.spitch + P.width - 1) & ~15ull;
    k0 = ufl64(k0);
    k1 = ufl64(k1);
    uint64_t rb = ufl64(k0 / ur);
    uint32_t jb = ufl32((uint32_t)(k0 - rb * ur));   // row and unit of the iteration's first unit
    for (uint64_t kb = k0; kb < k1; kb += 64u * U) {
        const uint64_t sb = d.src_sh + rb * sp, db = d.dst_sh + rb * dp;
        const uint32_t left = k1 - kb < 64u * U ? (uint32_t)(k1 - kb) : 64u * U;
        const int32_t lrel = clamp32((int64_t)(last - sb));   // at least -15
        u32x4 v[U];
        uint32_t ok[U], m[U], x[U], q[U];
        bool moved = false;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            // (lanes past the end work the last unit again and keep nothing)
            const uint32_t c = 64u * j + lane;
            const uint32_t n = jb + (c < left ? c : left - 1);
            x[j] = ur > 1 ? __umulhi(n, inv) : n;   // rows past rb
            q[j] = n - __umul24(x[j], ur);
            const int32_t rel = (int32_t)(__umul24(x[j], sp) + 16u * q[j]);
            const int32_t y = rel < lrel ? rel : lrel;
            v[j] = ld16<NT>(sb - 16u + (uint32_t)(y + 16));
            moved |= y != rel;
        }
        if (src_host) {
            const AWords A(R, d.a_src + (int64_t)(rb * sp));
#pragma unroll
            for (int j = 0; j < U; ++j) ok[j] = A.bits((int32_t)(__umul24(x[j], sp) + 16u * q[j]));
        } else {
#pragma unroll
            for (int j = 0; j < U; ++j) ok[j] = 0xFFFFu;
        }
        if (__ballot(moved)) {
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int32_t s = (int32_t)(__umul24(x[j], sp) + 16u * q[j]) - lrel;
                if (s > 0 && s < 16) v[j] = byte_shift(v[j], s);
            }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint32_t rest = width - 16u * q[j];   // bytes of the row from this window on
            m[j] = 64u * j + lane < left ? (rest >= 16u ? 0xFFFFu : (1u << rest) - 1u) : 0u;
            const uint32_t un = m[j] & ~ok[j];
            ok[j] &= m[j];
            if (check && ((v[j].x | v[j].y | v[j].z | v[j].w) || un))
                src_findings(acc, (int64_t)((rb + x[j]) * width + 16u * q[j]), v[j], ok[j], un);
        }
        if (dwork) {
            const AWords A(R, d.a_dst + (int64_t)(rb * dp));
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const uint32_t rel = __umul24(x[j], dp) + 16u * q[j];
                uint32_t wm = m[j];
                if (dst_host) {
                    wm &= A.bits((int32_t)rel);
                    if (check) dst_findings(acc, (int64_t)((rb + x[j]) * width + 16u * q[j]), m[j] & ~wm);
                }
                if (prop && wm) store_masked(db + rel, prop_val(v[j], ok[j]), wm);
            }
        }
        const uint32_t n = jb + 64u * U, dx = ur > 1 ? __umulhi(n, inv) : n;
        rb += ufl32(dx);
        jb = ufl32(n - dx * ur);
    }
}

// Units [k0, k1) of pitched position t, by the whole wave: rows that follow
// row 0 flat, or, when they are long, row by row through the wave-uniform
// loop; rows that do not follow row 0 are looked up (64 table entries per
// step) and classified here, and their range-derived flags join the record's
// (OR and min: a row worked in parts by several waves adds them more than
// once to the same effect).
template <int U, bool NT, bool PROP>
__device__ __forceinline__ void run_pitched(const BatchArgs &a, const Region &R, uint64_t t, uint64_t k0, uint64_t k1, Acc &acc)
{
    const Pitch P = ld_uniform(a.pitch + t);
    const DV d0 = load_desc_uniform(a.desc, t);
    if constexpr (!PROP) {
        const bool contig = P.uniform == kRowsContig;
        if (contig || (P.uniform && rows_aligned(a.mode, P))) {
            if (!contig && rows_flat(P)) {
                check_rows_flat<U, NT>(d0, P, R, k0, k1, acc);
                return;
            }
            // one transfer, or one per row; the edges two windows at a time, for the
            // registers (386 copies of rows of 8,209 bytes 246.3 us with four, 244.8
            // with two; 1,500 of 4,030 bytes without an index 692 and 686)
            const uint64_t ra = contig ? 0 : k0 / P.upr, rb = contig ? 0 : (k1 - 1) / P.upr;
            for (uint64_t r = ra; r <= rb; ++r) {
                const uint64_t b = r * P.upr, j0 = k0 > b ? k0 - b : 0, j1 = k1 - b < P.upr ? k1 - b : P.upr;
                const DV d = contig ? d0 : row_chunks(d0, P, r);
                Acc x;
                acc_reset(x);
                run_check<U, NT, (U > 2 ? 2 : U)>(d, R, j0, j1 < d.units ? j1 : d.units, x);
                acc_add_row(acc, x, 0u, NONE, r * P.width);
            }
            return;
        }
    }
    if (rows_flat(P)) {
        // (two windows per lane at most: each has a row's worth of indices)
        run_rows_flat<(U > 2 ? 2 : U), NT, PROP>(d0, P, R, k0, k1, acc);
        return;
    }
    const DevState *st = a.st;
    const uint64_t r0 = k0 / P.upr;
    for (uint64_t r = r0; r * P.upr < k1; ++r) {
        const uint64_t j0 = (k0 > r * P.upr ? k0 : r * P.upr) - r * P.upr;
        const uint64_t j1 = (k1 < (r + 1) * P.upr ? k1 : (r + 1) * P.upr) - r * P.upr;
        uint32_t rflags = 0;
        uint64_t rfirst = NONE;
        DV d = d0;
        if (P.uniform) {
            d.src_sh += r * P.spitch;
            d.dst_sh += r * P.dpitch;
            d.a_src += (int64_t)(r * P.spitch);
            d.a_dst += (int64_t)(r * P.dpitch);
        } else {
            const cg_transfer row = row_record(P, r);
            const int64_t js = dev_src(row) ? table_lookup_wave(st->table, row.src) : -1;
            const int64_t jd = dev_dst(row) ? table_lookup_wave(st->table, row.dst) : -1;
            Desc x;
            cg_verdict v;
            classify_rec(row, a.mode, *st, js, jd, x, v);
            rflags = ufl32(v.flags);
            rfirst = ufl64(v.first_bad);
            d = dv_uniform(x);
        }
        Acc ra;
        acc_reset(ra);
        const uint64_t e = j1 < d.units ? j1 : d.units;
        if (e > j0) run_uniform<U, NT, PROP>(d, R, j0, e, ra);
        acc_add_row(acc, ra, rflags, rfirst, r * P.width);
    }
}

// Unit k of pitched position t, by one lane (short rows, tile ends).
template <bool NT, bool PROP>
__device__ __forceinline__ void run_unit_pitched(const BatchArgs &a, const Region &R, uint64_t t, uint64_t k, Acc &acc)
{
    const DevState *st = a.st;
    const Pitch P = a.pitch[t];
    if (P.upr == 0) return;   // no rows, or a bad kind: nothing to work
    if (!PROP && P.uniform == kRowsContig) {
        const DV d = load_desc(a.desc, t);
        if (k < d.units) run_unit<NT, false, true>(d, R, k, acc);
        return;
    }
    const uint64_t r = (k | P.upr) >> 32 ? k / P.upr : (uint32_t)k / (uint32_t)P.upr, j = k - r * P.upr;
    if constexpr (!PROP) {
        if (P.uniform && rows_aligned(a.mode, P)) {
            const DV d = row_chunks(load_desc(a.desc, t), P, r);
            Acc x;
            acc_reset(x);
            if (j < d.units) run_unit<NT, false, true>(d, R, j, x);
            acc_add_row(acc, x, 0u, NONE, r * P.width);
            return;
        }
    }
    uint32_t rflags = 0;
    uint64_t rfirst = NONE;
    Desc x;
    if (P.uniform) {
        x = row_desc(a.desc[t], P, r);
    } else {
        const cg_transfer row = row_record(P, r);
        const int64_t js = dev_src(row) ? table_lookup(st->table, st->table.top, row.src) : -1;
        const int64_t jd = dev_dst(row) ? table_lookup(st->table, st->table.top, row.dst) : -1;
        cg_verdict v;
        classify_rec(row, a.mode, *st, js, jd, x, v);
        rflags = v.flags;
        rfirst = v.first_bad;
    }
    const DV d = make_dv(x);
    Acc ra;
    acc_reset(ra);
    if (j < d.units) run_unit<NT, PROP, false>(d, R, j, ra);
    acc_add_row(acc, ra, rflags, rfirst, r * P.width);
}

// Blocks b = x, x + nch, x + 2 nch, ... of the grid run on XCD x; b / nch is
// their rank there.  A work queue split into nch chunks gives each claiming
// block of XCD x a first item of chunk x by rank, without an atomic.  claim
// 0: every block claims; 1: the blocks of even rank; 2: those of odd rank.
__device__ __forceinline__ uint32_t claimers_on(uint32_t x, uint32_t nch, int claim)
{
    const uint32_t n = (gridDim.x + nch - 1 - x) / nch;
    return claim == 0 ? n : (claim == 1 ? (n + 1) / 2 : n / 2);
}

__device__ __forceinline__ int64_t claim_rank(uint32_t nch, int claim)
{
    const uint32_t r = blockIdx.x / nch;
    if (claim == 0) return r;
    return (int)(r & 1u) == claim - 1 ? (int64_t)(r >> 1) : -1;
}

// The waves' loop of the scan kernel (claim: which blocks take first tiles;
// PITCH: the positions are pitched 2D records, a.pitch).
template <int U, bool NT, bool PROP, bool PITCH, int CLAIM>
__device__ void batched_loop(const BatchArgs &a)
{
    const uint32_t lane = lane_id();
    const uint64_t ntiles = ufl64(a.ctl->ntiles);
    const uint64_t tu = ufl64(a.ctl->tile_units);
    const uint64_t total = ufl64(a.ctl->total_units);
    const uint64_t T = a.count;
    const Region R = ld_uniform(&a.st->region);
    Acc acc;
    acc_reset(acc);
    // Tiles are split into kXcds contiguous chunks, chunk x worked by the
    // waves of the blocks that run on XCD x, in ascending order, so that the
    // neighbouring segments of a batch sorted by source block share that
    // XCD's L2.
    // First tile: the wave's own index in its chunk (no atomic, so that the
    // waves of a small batch leave at once); later tiles from the chunk's
    // counter; a wave whose chunk is used up takes tiles from the others'.
    // Only a batch worked as segments has that locality to keep; any
    // other batch is one chunk for all waves (tiles interleaved over XCDs).
    const uint32_t nch = a.perm && (!a.lds_meta || lds_works(a)) ? kXcds : 1u;
    const uint32_t wpb = blockDim.x >> 6;
    const uint32_t xcd = blockIdx.x % nch;
    auto chunk_lo = [&](uint32_t x) { return ntiles * x / nch; };
    auto waves_on = [&](uint32_t x) { return (uint64_t)claimers_on(x, nch, CLAIM) * wpb; };
    const int64_t rank = claim_rank(nch, CLAIM);
    uint64_t jn = kNoTile;
    if (rank >= 0) {
        jn = chunk_lo(xcd) + (uint64_t)rank * wpb + (threadIdx.x >> 6);
        if (jn >= chunk_lo(xcd + 1)) jn = kNoTile;
    }
    uint32_t y = xcd, left = nch;
    for (;;) {
        while (jn == kNoTile && left > 0) {
            // a chunk no larger than its number of waves is all first tiles:
            // nothing to take there, and no atomic (small batches leave at once)
            const uint64_t lo = chunk_lo(y), hi = chunk_lo(y + 1);
            uint64_t c = hi;
            if (hi - lo > waves_on(y)) {
                uint32_t nx = 0;
                if (lane == 0) nx = atomicAdd(&a.ctl->counter[y], 1u);
                c = lo + waves_on(y) + ufl32(__shfl(nx, 0));
            }
            if (c < hi) {
                jn = c;
            } else {
                y = (y + 1) % nch;
                --left;
            }
        }
        if (jn == kNoTile) break;
        const uint64_t j = ufl64(jn);
        jn = kNoTile;
        uint64_t u = (uint64_t)j * tu;
        const uint64_t u_end = (u + tu < total) ? u + tu : total;
        uint64_t t = ufl32(a.tile_start[j]);
        uint64_t pt = ld_uniform(a.prefix + t), pt1 = ld_uniform(a.prefix + t + 1);   // record t's units
        while (u < u_end) {
            // a run of 64 units or more goes through the wave-uniform loop whole
            // (its last iteration may be partial); shorter runs, which may hold
            // several records, go one unit per lane
            const uint64_t seg_end = pt1 < u_end ? pt1 : u_end;
            uint64_t nfull = seg_end - u >= 64 ? seg_end - u : 0;
            // short rows that are not worked flat go one unit per lane (many
            // rows per wave); all others share the wave's iterations
            if constexpr (PITCH) {
                const Pitch P = ld_uniform(a.pitch + t);
                if (nfull && P.upr < 64 && P.uniform != kRowsContig && !rows_flat(P)) nfull = 0;
            }
            if (nfull) {
                if constexpr (PITCH) run_pitched<U, NT, PROP>(a, R, t, u - pt, u - pt + nfull, acc);
                else run_units<U, NT, PROP>(load_desc_uniform(a.desc, t), R, u - pt, u - pt + nfull, acc);
                if (a.out) flush_wave(acc, a.out, a.perm ? ld_uniform(a.perm + t) : t);
                u += nfull;
                if (u == pt1 && u < u_end) {
                    ++t;
                    pt = pt1;
                    pt1 = ld_uniform(a.prefix + t + 1);
                }
                continue;
            }
            // up to 64 units, one per lane, possibly of several records
            const uint64_t g_end = (u + 64 < u_end) ? u + 64 : u_end;
            const uint64_t ul = u + lane;
            const bool act = ul < g_end;
            // each lane's record: lane l looks at where record t + l starts; the
            // starts inside the group, as bits, count the records before a unit
            // (weights are at least 1, so at most 64 records meet the group)
            const uint64_t mine = a.prefix[t + lane < T ? t + lane : T];
            const uint64_t rel = mine - u;   // (wraps for t itself, which starts at or before u)
            const uint64_t starts = wave_or64(lane > 0 && rel < 64 ? 1ull << rel : 0ull);
            const uint32_t before = (uint32_t)__builtin_popcountll(starts & ((2ull << lane) - 1ull));
            const uint64_t tl = t + before;
            const uint64_t pl = ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(mine >> 32), (int)before) << 32) |
                                (uint32_t)__shfl((int)(uint32_t)mine, (int)before);
            if (PITCH && act) {
                run_unit_pitched<NT, PROP>(a, R, tl, ul - pl, acc);
            } else if (act) {
                const DV d = load_desc(a.desc, tl);
                const uint64_t k = ul - pl;
                if (k < d.units) run_unit<NT, PROP, !PROP>(d, R, k, acc);
            }
            if (a.out && __ballot(acc.flags != 0u))
                flush_segmented(acc, act ? (a.perm ? (uint64_t)a.perm[tl] : tl) : ~0ull, a.out);
            else acc_reset(acc);
            if (g_end < u_end) {
                const uint64_t t63 = ufl64(__shfl(tl, 63));
                t = (ld_uniform(a.prefix + t63 + 1) <= g_end) ? t63 + 1 : t63;
                pt = ld_uniform(a.prefix + t);
                pt1 = ld_uniform(a.prefix + t + 1);
            }
            u = g_end;
        }
    }
}

template <int U, bool NT, bool PROP>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(PROP ? 1 : 3))) k_batched(BatchArgs a)
{
    if (lds_works(a)) return;
    batched_loop<U, NT, PROP, false, 0>(a);
}

// the scan kernel over pitched 2D records (check_transfers_2d)
template <int U, bool NT, bool PROP>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(PROP ? 1 : 3))) k_batched_2d(BatchArgs a)
{
    batched_loop<U, NT, PROP, true, 0>(a);
}

// ---------------------------------------------------------------------------
// k_host_lds: host-source segments with their source bytes staged in LDS
// ---------------------------------------------------------------------------
// A batch worked as segments reads each host byte many times (about 160 on
// the 1M-record configuration), and through the vector memory path every
// re-read costs an address and an L2-to-L1 transfer.  Here the host-source
// positions (sorted last, by block of source memory) are taken in tasks of
// kTaskPos consecutive positions, each by one workgroup: for every window of
// kWinChunks chunks that the task's segments of one block touch, the window's
// V bytes and A bits are copied into LDS once, and every segment overlapping
// it is checked from there by one wave.  Only check-only host-to-device
// records have host sources worked here: their destination needs no check
// of its own.  Findings go to each position's record with the same atomics
// as in k_batched.  Tasks are split into one contiguous range per XCD, like
// k_batched's tiles, so that the tasks of one block stage it from one L2.
constexpr uint32_t kWinChunks = 2048;   // 32 KiB of V bytes per window
constexpr uint32_t kTaskPos = 256;      // positions per task, at most

// One position of a task, as the waves need it: absolute chunk indices (the
// shadow address over 16) of the segment's chunks [c_lo, c_hi), the record
// byte index i0 of chunk c_lo's first byte, the record's valid source bytes
// [v_lo, v_hi), and the verdict it reports to.
struct HostPos {
    int64_t c_lo, c_hi, i0, v_lo, v_hi;
    uint64_t blk;
    uint32_t rec, pad;
};

template <int U>
__device__ __forceinline__ void lds_segment(const HostPos &P, int64_t wc0, int64_t wc1, const u32x4 *sv,
                                            const uint16_t *sa, Acc &acc)
{
    const int64_t ca = P.c_lo > wc0 ? P.c_lo : wc0;
    const int64_t cb = P.c_hi < wc1 ? P.c_hi : wc1;
    const int32_t lane = (int32_t)lane_id();
    for (int64_t c = ca; c < cb; c += 64 * U) {
        const int64_t i0f = P.i0 + 16 * (c - P.c_lo);
        const int32_t base = (int32_t)(c - wc0);
        const int32_t n = (int32_t)(cb - c < 64 * U ? cb - c : 64 * U);
        // all U reads issued back to back: lanes past the segment's chunks in
        // this window read its last chunk again and ignore it
        u32x4 v[U];
        uint32_t av[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int32_t k = 64 * j + lane;
            const int32_t kk = k < n ? k : n - 1;
            v[j] = sv[base + kk];
            av[j] = sa[base + kk];
        }
        // every chunk of the iteration wholly valid: one test over them
        if (i0f >= P.v_lo && i0f + 16 * n <= P.v_hi) {
            uint32_t bad = 0;
#pragma unroll
            for (int j = 0; j < U; ++j) bad |= v[j].x | v[j].y | v[j].z | v[j].w | (av[j] ^ 0xFFFFu);
            if (__ballot(bad != 0u) == 0) continue;
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int32_t k = 64 * j + lane;
            const int64_t i0 = i0f + 16 * k;
            const uint32_t m = k < n ? rmask(P.v_lo - i0, P.v_hi - i0) : 0u;
            src_findings(acc, i0, v[j], m & av[j], m & ~av[j]);
        }
    }
}

// The workgroups' loop over the host-source tasks (claim: which blocks take
// first tasks, as in batched_loop); sv / sa / sp / s_task / s_next / s_list
// are the block's LDS.
template <int U>
__device__ void host_loop(const BatchArgs &a, const uint64_t *meta, int claim, u32x4 *sv, uint16_t *sa, HostPos *sp,
                          uint64_t *s_task, uint32_t *s_next, uint16_t *s_list)
{
    const uint64_t p_begin = meta[2], p_end = meta[0];
    if (p_begin >= p_end) return;
    const uint32_t lb = (uint32_t)meta[1];
    const uint32_t tp = a.task_pos ? a.task_pos : kTaskPos;   // positions per task, at most kTaskPos
    const uint64_t ntasks = (p_end - p_begin + tp - 1) / tp;
    const Region R = a.st->region;
    const int64_t vbase = (int64_t)((uint64_t)R.v >> 4);     // V is 16-byte aligned
    const int64_t nvch = (int64_t)((R.hl + 15) >> 4);         // chunks of V
    const int64_t nach = (int64_t)(((R.hl + 63) >> 6) * 4);   // 16-bit A words
    const gcptr<u32x4> gv = reinterpret_cast<gcptr<u32x4>>((uint64_t)R.v);
    const gcptr<uint16_t> ga = reinterpret_cast<gcptr<uint16_t>>((uint64_t)R.a16);
    // tasks in kXcds contiguous chunks, chunk x taken by the workgroups on XCD x
    auto chunk_lo = [&](uint32_t x) { return ntasks * x / kXcds; };
    auto groups_on = [&](uint32_t x) { return (uint64_t)claimers_on(x, kXcds, claim); };
    const uint32_t xcd = blockIdx.x % kXcds;
    const int64_t rank = claim_rank(kXcds, claim);
    uint64_t jn = kNoTile;
    if (rank >= 0) {
        jn = chunk_lo(xcd) + (uint64_t)rank;
        if (jn >= chunk_lo(xcd + 1)) jn = kNoTile;
    }
    uint32_t y = xcd, left = kXcds;
    Acc acc;
    acc_reset(acc);
    for (;;) {
        if (threadIdx.x == 0) {
            while (jn == kNoTile && left > 0) {
                const uint64_t lo = chunk_lo(y), hi = chunk_lo(y + 1);
                uint64_t c = hi;
                if (hi - lo > groups_on(y)) c = lo + groups_on(y) + atomicAdd(&a.ctl->lds_counter[y], 1u);
                if (c < hi) jn = c;
                else {
                    y = (y + 1) % kXcds;
                    --left;
                }
            }
            *s_task = jn;
        }
        __syncthreads();
        const uint64_t j = *s_task;
        jn = kNoTile;
        __syncthreads();
        if (j == kNoTile) break;
        const uint64_t q0 = p_begin + j * tp;
        const uint32_t np = (uint32_t)(p_end - q0 < tp ? p_end - q0 : tp);
        for (uint32_t t = threadIdx.x; t < np; t += blockDim.x) {
            const Desc d = a.desc[q0 + t];
            const int64_t e = (int64_t)d.e0;   // (a check's windows are aligned source chunks)
            HostPos h;
            h.c_lo = (int64_t)(d.src_sh >> 4) + e;
            h.c_hi = h.c_lo + (int64_t)d.units;
            h.i0 = 16 * e - (int64_t)desc_o(d);
            h.v_lo = d.v_lo;
            h.v_hi = d.v_hi;
            h.blk = (uint64_t)h.c_lo >> (lb - 4);
            h.rec = a.perm[q0 + t];
            h.pad = 0;
            sp[t] = h;
        }
        __syncthreads();
        // the task's positions by block (they are sorted by block)
        for (uint32_t g0 = 0; g0 < np;) {
            const uint64_t blk = sp[g0].blk;
            uint32_t g1 = g0 + 1;
            int64_t cmin = sp[g0].c_lo, cmax = sp[g0].c_hi;
            while (g1 < np && sp[g1].blk == blk) {
                cmin = sp[g1].c_lo < cmin ? sp[g1].c_lo : cmin;
                cmax = sp[g1].c_hi > cmax ? sp[g1].c_hi : cmax;
                ++g1;
            }
            for (int64_t wc0 = (cmin / kWinChunks) * kWinChunks; wc0 < cmax; wc0 += kWinChunks) {
                const int64_t wc1 = wc0 + kWinChunks;
                // stage the window: V chunks and A words inside the buffers,
                // zeros elsewhere; every load is issued (at a clamped index,
                // inside the buffer) before the first is used
                // (passes of 4 chunks per thread: 2 for 256 threads, 1 for 512)
                for (uint32_t k0 = 0; k0 < kWinChunks; k0 += 4 * blockDim.x) {
                    u32x4 gvv[4];
                    uint32_t gav[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int64_t c = wc0 + k0 + threadIdx.x + i * blockDim.x - vbase;
                        gvv[i] = gv[c < 0 ? 0 : (c < nvch ? c : nvch - 1)];
                        gav[i] = ga[c < 0 ? 0 : (c < nach ? c : nach - 1)];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t k = k0 + threadIdx.x + i * blockDim.x;
                        const int64_t c = wc0 + k - vbase;
                        sv[k] = (c >= 0 && c < nvch) ? gvv[i] : u32x4{0u, 0u, 0u, 0u};
                        sa[k] = (uint16_t)((c >= 0 && c < nach) ? gav[i] : 0u);
                    }
                }
                // the group's positions that overlap the window, listed once
                if (threadIdx.x == 0) {
                    s_next[0] = 0;
                    s_next[1] = 0;
                }
                __syncthreads();
                for (uint32_t t = threadIdx.x; t < g1 - g0; t += blockDim.x) {
                    const HostPos &P = sp[g0 + t];
                    if (P.c_hi > wc0 && P.c_lo < wc1) s_list[atomicAdd(&s_next[1], 1u)] = (uint16_t)(g0 + t);
                }
                __syncthreads();
                const uint32_t nlist = s_next[1];
                // listed positions taken one at a time by whichever wave is
                // free, so that a few long segments do not hold up the others
                for (;;) {
                    uint32_t q = 0;
                    if (lane_id() == 0) q = atomicAdd(&s_next[0], 1u);
                    q = ufl32(__shfl(q, 0));
                    if (q >= nlist) break;
                    const HostPos P = sp[s_list[q]];
                    lds_segment<U>(P, wc0, wc1, sv, sa, acc);
                    if (a.out) flush_wave(acc, a.out, P.rec);
                }
                __syncthreads();
            }
            g0 = g1;
        }
    }
}

// A check-only batch worked as segments with its host-source positions left
// to LDS: blocks of even rank on their XCD start with the scan kernel's tiles,
// blocks of odd rank with the host-source tasks, and each turns to the other
// queue when its own is used up, so that the HBM-bound device-source work and
// the LDS-bound host-source work run side by side to the end.
template <int U, bool NT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(3))) k_batched_lds(BatchArgs a)
{
    __shared__ u32x4 sv[kWinChunks];
    __shared__ uint16_t sa[kWinChunks];
    __shared__ HostPos sp[kTaskPos];
    __shared__ uint64_t s_task;
    __shared__ uint32_t s_next[2];
    __shared__ uint16_t s_list[kTaskPos];
    if (!lds_works(a)) return;
    if (((blockIdx.x / kXcds) & 1u) != 0) {
        host_loop<4>(a, a.lds_meta, 2, sv, sa, sp, &s_task, s_next, s_list);
        __syncthreads();
        batched_loop<U, NT, false, false, 1>(a);
    } else {
        batched_loop<U, NT, false, false, 1>(a);
        __syncthreads();
        host_loop<4>(a, a.lds_meta, 2, sv, sa, sp, &s_task, s_next, s_list);
    }
}

// ---------------------------------------------------------------------------
// k_plain: one record per launch, waves split its units evenly
// ---------------------------------------------------------------------------
template <int U, bool NT, bool PROP>
__global__ void __launch_bounds__(512) k_plain(BatchArgs a, uint64_t t, uint64_t units)
{
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    const uint64_t w = (uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    uint64_t span = (units + waves - 1) / waves;
    span = (span + 63) & ~63ull;
    const uint64_t k0 = w * span;
    if (k0 >= units) return;
    const uint64_t k1 = (k0 + span < units) ? k0 + span : units;
    const DV d = load_desc_uniform(a.desc, t);
    Acc acc;
    acc_reset(acc);
    run_units<U, NT, PROP>(d, ld_uniform(&a.st->region), k0, k1, acc);
    if (a.out) flush_wave(acc, a.out, t);
}

// ---------------------------------------------------------------------------
// k_small: a small batch in one launch
// ---------------------------------------------------------------------------

// A batch of few records in one launch, up to `bpr` blocks per record.  The
// blocks a record uses follow from its byte count alone (at most one per
// kSmallUnits units), so that every block of the record agrees on them and
// the unused ones leave after one load.  Block b of record t: waves 0 and 1
// look up the record's source and destination pointers side by side, one
// lane classifies it; the record's iterations
// are dealt out to its blocks' waves in turn (the wave-uniform loop).  A record
// of one block gets its whole verdict from that
// block.  Otherwise a block that finds something merges it into the record's
// accumulator with atomics; the last of the record's blocks to finish (the
// accumulator's counter) writes the whole verdict -- the range-derived fields
// of its own classification and the findings of all blocks -- and puts the
// accumulator back to its starting state {NONE, 0, 0, 0}, so that the next
// call needs no clearing.

template <int U, bool NT, bool PROP>
__global__ void __launch_bounds__(1024)
k_small(BatchArgs a, SmallAcc *acc, uint32_t bpr)
{
    __shared__ Desc sd;
    __shared__ cg_verdict sv;
    __shared__ uint64_t su;
    __shared__ uint64_t wfirst[16], wund[16];
    __shared__ uint32_t wfl[16];
    __shared__ int64_t sj[2];   // the source's and the destination's allocation (-1: none)
    const uint32_t lane = lane_id(), wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint64_t t = blockIdx.x / bpr;
    const uint32_t b = blockIdx.x % bpr;
    const cg_transfer r = a.recs[t];
    // units never exceed n / 16 + 2 (one per 16-byte chunk the bytes touch)
    const uint64_t most = r.kind <= CG_D2D && r.n ? r.n / 16 + 2 : 1;
    const uint64_t want = (most + kSmallUnits - 1) / kSmallUnits;
    const uint32_t nb = want < bpr ? (uint32_t)want : bpr;   // blocks of this record, at least 1
    if (b >= nb) return;
    const DevState *st = a.st;
    if (wid < 2) {
        // the source's lookup on wave 0, the destination's on wave 1, side by side
        const bool src = wid == 0;
        int64_t j = -1;
        if (src ? dev_src(r) : dev_dst(r)) j = table_lookup_wave(st->table, src ? r.src : r.dst);
        if (lane == 0) sj[wid] = j;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        Desc ds;
        cg_verdict v;
        su = classify_rec(r, a.mode, *st, sj[0], sj[1], ds, v);
        sd = ds;
        sv = v;
    }
    __syncthreads();
    const uint64_t units = su;
    // the record's iterations dealt out to its blocks' waves in turn, so that
    // all of them work side by side on one stretch of the shadow (2 GiB carried
    // by one stretch per wave: 850 us in a plain copy, 780 dealt out)
    const uint64_t k0 = ((uint64_t)b * nw + wid) * 64u * U;
    Acc ac;
    acc_reset(ac);
    if (k0 < units) {
        const DV d = dv_uniform(sd);
        run_units<U, NT, PROP>(d, ld_uniform(&st->region), k0, units, ac, (uint64_t)nb * nw * 64u * U);
    }
    if (!a.out) return;   // propagation only: no verdict (uniform over the grid)
    uint64_t f = NONE, u = 0;
    uint32_t fl = 0;
    if (__ballot(ac.flags != 0u)) {
        f = wave_min64(ac.first);
        u = wave_sum64(ac.undef);
        fl = wave_or32(ac.flags);
    }
    if (lane == 0) {
        wfirst[wid] = f;
        wund[wid] = u;
        wfl[wid] = fl;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (uint32_t w = 1; w < nw; ++w) {
        f = wfirst[w] < f ? wfirst[w] : f;
        u += wund[w];
        fl |= wfl[w];
    }
    cg_verdict v = sv;
    if (nb > 1) {
        SmallAcc &x = acc[t];
        if (fl) {
            atomicOr(&x.flags, fl);
            if (f != NONE) atomicMin((unsigned long long *)&x.first, (unsigned long long)f);
            if (u) atomicAdd((unsigned long long *)&x.undef, (unsigned long long)u);
        }
        __threadfence();
        if (atomicAdd(&x.done, 1u) != nb - 1) return;
        __threadfence();
        // the last block of the record: every other block's findings are in
        fl |= __hip_atomic_load(&x.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t af = __hip_atomic_load(&x.first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        u = __hip_atomic_load(&x.undef, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        f = af < f ? af : f;
        __hip_atomic_store(&x.flags, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&x.first, NONE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&x.undef, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&x.done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    v.flags |= fl;
    v.first_bad = f < v.first_bad ? f : v.first_bad;
    v.undef_bytes = u;
    a.out[t] = v;
}

// accumulators to their starting state
__global__ void __launch_bounds__(256) k_small_reset(SmallAcc *acc, uint64_t n)
{
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) acc[i] = SmallAcc{NONE, 0, 0, 0};
}

// ---------------------------------------------------------------------------
// shadow fills and bandwidth probes
// ---------------------------------------------------------------------------
// A small upload from coherent host memory: one block copies n 8-byte words
// with system-scope loads (they observe the host's latest writes); for the
// kilobytes of a table delta or of fill ranges that are too many for a
// launch's arguments, a launch waits less than a DMA copy.
__global__ void __launch_bounds__(256) k_upload(const uint64_t *src, uint64_t *dst, uint64_t n)
{
    for (uint64_t i = threadIdx.x; i < n; i += 256)
        dst[i] = __hip_atomic_load(src + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One block sets one range (pieces of at most 1 MiB): bytes to the first
// 16-byte boundary, 16-byte stores, the last bytes.
__device__ __forceinline__ void fill_range(const FillRange &fr)
{
    uint8_t *p = reinterpret_cast<uint8_t *>(fr.ptr);
    const uint8_t v = (uint8_t)fr.val;
    const uint64_t len = fr.len;
    uint64_t head = (16u - (fr.ptr & 15u)) & 15u;
    head = head < len ? head : len;
    if (threadIdx.x < head) p[threadIdx.x] = v;
    const uint64_t body = (len - head) & ~15ull;
    const uint32_t w = 0x01010101u * v;
    const u32x4 vv{w, w, w, w};
    for (uint64_t o = head + 16ull * threadIdx.x; o < head + body; o += 16ull * blockDim.x)
        *reinterpret_cast<u32x4 *>(p + o) = vv;
    const uint64_t tail = len - head - body;
    if (threadIdx.x < tail) p[head + body + threadIdx.x] = v;
}

__global__ void __launch_bounds__(256) k_fill(const FillRange *ranges, uint64_t k)
{
    for (uint64_t i = blockIdx.x; i < k; i += gridDim.x) fill_range(ranges[i]);
}

// The ranges of one allocation, or of a few fills, read from the launch's
// arguments: no upload before the fill.
__global__ void __launch_bounds__(256) k_fill_inline(FillArgs f) { fill_range(f.r[blockIdx.x]); }

__global__ void __launch_bounds__(256) k_probe_read(const u32x4 *p, uint64_t n16, uint64_t *sink)
{
    u32x4 acc{0u, 0u, 0u, 0u};
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n16; i += 4 * stride) {
        const u32x4 a = __builtin_nontemporal_load(p + i);
        const u32x4 b = __builtin_nontemporal_load(p + i + stride);
        const u32x4 c = __builtin_nontemporal_load(p + i + 2 * stride);
        const u32x4 d = __builtin_nontemporal_load(p + i + 3 * stride);
        acc ^= a ^ b ^ c ^ d;
    }
    for (; i < n16; i += stride) acc ^= __builtin_nontemporal_load(p + i);
    const uint32_t x = acc.x ^ acc.y ^ acc.z ^ acc.w;
    if (x == 0x9E3779B9u) atomicXor((unsigned long long *)sink, (unsigned long long)x);
}

// L2-resident read ceiling: block b reads slice b mod 8 (the XCD it runs on)
// `passes` times with the same cached 16-byte loads as the scan kernel, each
// block from its own starting offset, so that the blocks sharing a CU do not
// hit in its L1 on each other's lines; a slice that fits its XCD's L2 is then
// served from L2 to the L1s.
__global__ void __launch_bounds__(256) k_probe_l2(const u32x4 *p, uint64_t slice16, uint32_t passes, uint64_t *sink)
{
    const u32x4 *q = p + (uint64_t)(blockIdx.x % kXcds) * slice16;
    const uint64_t step = 4ull * blockDim.x;
    const uint64_t groups = slice16 / step;   // whole groups of 4 loads per thread
    uint64_t g = ((uint64_t)(blockIdx.x / kXcds) * 37u) % (groups ? groups : 1);
    u32x4 acc{0u, 0u, 0u, 0u};
    for (uint64_t k = 0; k < groups * passes; ++k) {
        const u32x4 *r = q + g * step + threadIdx.x;
        const u32x4 a = r[0], b = r[blockDim.x], c = r[2 * blockDim.x], d = r[3 * blockDim.x];
        acc ^= a ^ b ^ c ^ d;
        g = g + 1 == groups ? 0 : g + 1;
    }
    const uint32_t x = acc.x ^ acc.y ^ acc.z ^ acc.w;
    if (x == 0x9E3779B9u) atomicXor((unsigned long long *)sink, (unsigned long long)x);
}

__global__ void __launch_bounds__(256) k_probe_copy(u32x4 *d, const u32x4 *p, uint64_t n16)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
        d[i] = __builtin_nontemporal_load(p + i);
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_classify(const BatchArgs &a, hipStream_t s)
{
    const uint64_t blocks = (a.count + kClassifyBlock - 1) / kClassifyBlock;
    hipLaunchKernelGGL(k_classify, dim3((uint32_t)blocks), dim3(kClassifyBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_reweigh(const BatchArgs &a, hipStream_t s)
{
    const uint64_t blocks = (a.count + kClassifyBlock - 1) / kClassifyBlock;
    if (!a.index_bytes[0]) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_reweigh, dim3((uint32_t)blocks), dim3(kClassifyBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_classify_2d(const BatchArgs &a, const cg_transfer2d *recs2d, Pitch *pitch, hipStream_t s)
{
    const uint64_t blocks = (a.count + kClassifyBlock - 1) / kClassifyBlock;
    hipLaunchKernelGGL(k_classify_2d, dim3((uint32_t)blocks), dim3(kClassifyBlock), 0, s, a, recs2d, pitch);
    return hipGetLastError();
}

// Workgroups of the scan kernel: the persistent grid the launch shape asks
// for, or, when the number of blocks is not the caller's, four times as many (at
// most 16 of 256 threads per CU), so that a batch worked as one tile per wave is
// levelled out by the hardware's own dispatch (3,000 requests kept in their
// order 141 us with 16 blocks per CU, 165 with 8, 189 with 4).
static uint32_t scan_grid(const LaunchShape &sh)
{
    if (!sh.spread) return sh.grid;
    const uint32_t most = sh.cus * 16u * 256u / sh.block;
    return sh.grid >= most ? sh.grid : std::min(4u * sh.grid, most);
}

hipError_t launch_tiles(const BatchArgs &a, const LaunchShape &sh, hipStream_t s)
{
    const uint64_t blocks = (a.count + kClassifyBlock - 1) / kClassifyBlock;
    const uint32_t waves = scan_grid(sh) * (sh.block / 64), lds_waves = sh.grid * (sh.block / 64);
    if (blocks <= kPlanSums) {
        hipLaunchKernelGGL(k_plan_tiles, dim3(std::max((uint32_t)blocks, kPlanGrid)), dim3(256), 0, s, a,
                           sh.tile_units, waves, lds_waves);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, s, a, sh.tile_units, waves, lds_waves);
    hipLaunchKernelGGL(k_prefix_tiles, dim3((uint32_t)blocks), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_tile_starts, dim3(1024), dim3(256), 0, s, a);
    return hipGetLastError();
}

// the host-source tasks alone (the LDS path run after the scan kernel)
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) k_host_lds(BatchArgs a)
{
    __shared__ u32x4 sv[kWinChunks];
    __shared__ uint16_t sa[kWinChunks];
    __shared__ HostPos sp[kTaskPos];
    __shared__ uint64_t s_task;
    __shared__ uint32_t s_next[2];
    __shared__ uint16_t s_list[kTaskPos];
    host_loop<4>(a, a.lds_meta, 0, sv, sa, sp, &s_task, s_next, s_list);
}

// Pitched rows are worked in at most four windows a lane, two when they
// propagate, whatever the unroll asked for: more of them do not fit the
// registers beside the rows' own state (248 and 244 bytes of scratch a lane at
// four, propagating).  64 copies of 2,000 rows of 4,030 bytes carried from the
// host: 264 us with two, 520 with four; of 200,000-byte rows 239 and 334; 8 of 64
// rows of 70,000 bytes 2 MiB apart 42 and 95.
template <int U, bool NT>
static void launch_batched_t(const BatchArgs &a, const LaunchShape &sh, hipStream_t s)
{
    if (a.pitch && (a.mode & CG_PROPAGATE)) {
        hipLaunchKernelGGL((k_batched_2d<(U > 2 ? 2 : U), NT, true>), dim3(scan_grid(sh)), dim3(sh.block), 0, s, a);
    } else if (a.pitch) {
        hipLaunchKernelGGL((k_batched_2d<(U > 4 ? 4 : U), NT, false>), dim3(scan_grid(sh)), dim3(sh.block), 0, s, a);
    } else if (a.lds_meta && sh.lds_after) {
        BatchArgs d = a;
        d.lds_meta = nullptr;
        hipLaunchKernelGGL((k_batched<U, NT, false>), dim3(sh.grid), dim3(sh.block), 0, s, d);
        hipLaunchKernelGGL(k_host_lds, dim3(sh.cus * 3), dim3(256), 0, s, a);
    } else if (a.lds_meta) {
        hipLaunchKernelGGL((k_batched_lds<U, NT>), dim3(sh.grid), dim3(sh.block), 0, s, a);
        hipLaunchKernelGGL((k_batched<U, NT, false>), dim3(scan_grid(sh)), dim3(sh.block), 0, s, a);
    } else if (a.mode & CG_PROPAGATE)
        hipLaunchKernelGGL((k_batched<U, NT, true>), dim3(scan_grid(sh)), dim3(sh.block), 0, s, a);
    else
        hipLaunchKernelGGL((k_batched<U, NT, false>), dim3(scan_grid(sh)), dim3(sh.block), 0, s, a);
}

template <int U, bool NT>
static void launch_plain_t(const BatchArgs &a, uint64_t t, uint64_t units, uint32_t grid, uint32_t block,
                           hipStream_t s)
{
    if (a.mode & CG_PROPAGATE)
        hipLaunchKernelGGL((k_plain<U, NT, true>), dim3(grid), dim3(block), 0, s, a, t, units);
    else
        hipLaunchKernelGGL((k_plain<U, NT, false>), dim3(grid), dim3(block), 0, s, a, t, units);
}

#define XC_DISPATCH(FN, ...)                                                   \
    do {                                                                       \
        const bool nt_ = sh.nontemporal != 0;                                  \
        switch (sh.unroll) {                                                   \
        case 1: nt_ ? FN<1, true>(__VA_ARGS__) : FN<1, false>(__VA_ARGS__); break; \
        case 2: nt_ ? FN<2, true>(__VA_ARGS__) : FN<2, false>(__VA_ARGS__); break; \
        case 8: nt_ ? FN<8, true>(__VA_ARGS__) : FN<8, false>(__VA_ARGS__); break; \
        default: nt_ ? FN<4, true>(__VA_ARGS__) : FN<4, false>(__VA_ARGS__); break; \
        }                                                                      \
    } while (0)

hipError_t launch_batched(const BatchArgs &a, const LaunchShape &sh, hipStream_t s)
{
    if (a.lds_meta && (a.mode & CG_PROPAGATE)) return hipErrorInvalidValue;   // check-only
    XC_DISPATCH(launch_batched_t, a, sh, s);
    return hipGetLastError();
}

// At most four windows a lane: a block of 1,024 threads leaves a lane 128
// registers, which eight pass, and eight are nowhere faster (1 GiB checked in
// one record 195 us with four, 204 with eight; 256 records of 1 MiB 83 and 92).
template <int U, bool NT>
static void launch_small_t(const BatchArgs &a, SmallAcc *acc, uint32_t bpr, uint32_t block, hipStream_t s)
{
    constexpr int V = U > 4 ? 4 : U;
    const dim3 grid((uint32_t)(a.count * bpr));
    if (a.mode & CG_PROPAGATE)
        hipLaunchKernelGGL((k_small<V, NT, true>), grid, dim3(block), 0, s, a, acc, bpr);
    else
        hipLaunchKernelGGL((k_small<V, NT, false>), grid, dim3(block), 0, s, a, acc, bpr);
}

hipError_t launch_small(const BatchArgs &a, SmallAcc *acc, uint32_t bpr, const LaunchShape &sh, hipStream_t s)
{
    if (a.count == 0 || bpr == 0 || a.count * bpr > 0x7FFFFFFFull || sh.block > 1024 || sh.block % 64)
        return hipErrorInvalidValue;
    XC_DISPATCH(launch_small_t, a, acc, bpr, sh.block, s);
    return hipGetLastError();
}

hipError_t launch_small_reset(SmallAcc *acc, uint64_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_small_reset, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, acc, n);
    return hipGetLastError();
}

// Waves of two windows a lane (what a record's edge is worked in) while the
// grid allows, and the unroll no larger than a wave's share: a share below a
// whole iteration is worked as an edge throughout, two windows after two.
// Records of 5 MB, 4,096 waves of 128 units: unroll 4 7.6 us a launch, unroll
// 2 4.7; records of 64 KiB in one block of four waves 6.2 us, in eight 4.5.
hipError_t launch_plain(const BatchArgs &a, uint64_t rec, uint64_t units, const LaunchShape &shape, hipStream_t s)
{
    LaunchShape sh = shape;
    const uint32_t wpb = sh.block / 64;
    const uint64_t per_block = (uint64_t)wpb * 128u;
    uint64_t grid = (units + per_block - 1) / per_block;
    if (grid > sh.grid) grid = sh.grid;
    if (grid == 0) grid = 1;
    const uint64_t waves = grid * wpb, share = ((units + waves - 1) / waves + 63) & ~63ull;   // as k_plain's
    while (sh.unroll > 1 && 64u * sh.unroll > share) sh.unroll >>= 1;
    XC_DISPATCH(launch_plain_t, a, rec, units, (uint32_t)grid, sh.block, s);
    return hipGetLastError();
}

hipError_t launch_pointers(const DevState *st, uint32_t nmid, uint32_t cus, const uint64_t *ptrs, uint64_t count,
                           cg_ptr_check *out, hipStream_t s)
{
    if (nmid > (uint32_t)kMaxMid) return hipErrorInvalidValue;
    // a workgroup's LDS is the middle level: as many workgroups as the CUs
    // hold at once.  Few pointers go in workgroups of 256, so that more CUs
    // take part; many, in workgroups of 1,024, so that the waves of a CU share
    // one or two staged levels.
    const bool few = count < 262144;
    const uint32_t lds = (few ? std::min<uint32_t>(nmid, kMaxTop) : nmid) * 8u;   // (the top level is no larger)
    const uint32_t block = few ? 256u : 1024u;
    const uint32_t fit = lds ? (160u * 1024u) / lds : 8u;
    const uint32_t per_cu = std::max(1u, std::min(fit, 2048u / block));
    const uint64_t want = (count + block - 1) / block;
    const uint32_t grid = (uint32_t)std::min<uint64_t>(want, (uint64_t)cus * per_cu);
    hipLaunchKernelGGL(k_pointers, dim3(grid), dim3(block), lds, s, st, ptrs, count, out, few);
    return hipGetLastError();
}

hipError_t launch_upload(const void *src, void *dst, uint64_t bytes, hipStream_t s)
{
    if (bytes == 0) return hipSuccess;
    hipLaunchKernelGGL(k_upload, dim3(1), dim3(256), 0, s, static_cast<const uint64_t *>(src),
                       static_cast<uint64_t *>(dst), bytes / 8);
    return hipGetLastError();
}

hipError_t launch_fill(const FillRange *ranges_dev, uint64_t k, hipStream_t s)
{
    if (k == 0) return hipSuccess;
    const uint32_t grid = (uint32_t)(k < 65536 ? k : 65536);
    hipLaunchKernelGGL(k_fill, dim3(grid), dim3(256), 0, s, ranges_dev, k);
    return hipGetLastError();
}

hipError_t launch_fill_inline(const FillArgs &f, uint64_t k, hipStream_t s)
{
    if (k == 0) return hipSuccess;
    if (k > kFillInline) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_fill_inline, dim3((uint32_t)k), dim3(256), 0, s, f);
    return hipGetLastError();
}

hipError_t launch_probe_read(const void *p, uint64_t bytes, uint64_t *sink, hipStream_t s)
{
    hipLaunchKernelGGL(k_probe_read, dim3(8192), dim3(256), 0, s, reinterpret_cast<const u32x4 *>(p), bytes / 16,
                       sink);
    return hipGetLastError();
}

hipError_t launch_probe_l2(const void *p, uint64_t slice_bytes, uint32_t passes, uint32_t blocks, uint64_t *sink,
                           hipStream_t s)
{
    hipLaunchKernelGGL(k_probe_l2, dim3(blocks), dim3(256), 0, s, reinterpret_cast<const u32x4 *>(p), slice_bytes / 16,
                       passes, sink);
    return hipGetLastError();
}

hipError_t launch_probe_copy(void *d, const void *p, uint64_t bytes, hipStream_t s)
{
    hipLaunchKernelGGL(k_probe_copy, dim3(8192), dim3(256), 0, s, reinterpret_cast<u32x4 *>(d),
                       reinterpret_cast<const u32x4 *>(p), bytes / 16);
    return hipGetLastError();
}

}  // namespace xc
