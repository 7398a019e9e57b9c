// Device helpers of the scans that look at text positions known beforehand
// (mpm_scan_gram.hip): a wave takes 4 KiB of text, 64 contiguous bytes per
// lane, as 2-bit character codes.
#pragma once
#include "mpm_scan_impl.h"

namespace mpm {
namespace {

constexpr uint32_t GBLOCK = 4096;  // text bytes per wave and step

// Set in the epoch of these scans' status words. Their chunks differ from the
// walkers', so on a shared workspace a status word may hold what a walker
// staged there, a (position, string) pair: its top bit, and so this bit of
// the epoch field, is clear.
constexpr uint32_t GRAM_EPOCH = 1u << 25;

typedef v4u v4u_any __attribute__((aligned(1)));

// Other lanes' LDS writes before this point are visible after it (one wave's
// LDS operations complete in order).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 2-bit codes of 16 bytes, the first in the low bits: per word one shift,
// one mask and one byte dot product with 1, 4, 16, 64.
__device__ __forceinline__ uint32_t codes16(const v4u c, uint32_t sh)
{
    const uint32_t a = __builtin_amdgcn_udot4((c.x >> sh) & 0x03030303u, 0x40100401u, 0u, false);
    const uint32_t b = __builtin_amdgcn_udot4((c.y >> sh) & 0x03030303u, 0x40100401u, 0u, false);
    const uint32_t d = __builtin_amdgcn_udot4((c.z >> sh) & 0x03030303u, 0x40100401u, 0u, false);
    const uint32_t e = __builtin_amdgcn_udot4((c.w >> sh) & 0x03030303u, 0x40100401u, 0u, false);
    return a | b << 8 | d << 16 | e << 24;
}

// The text seen from the 16-byte boundary at or before its first byte: byte v
// of this view is text byte v - lo; bytes outside [lo, hi) are not read.
struct View {
    glb_cptr<uint8_t> p;
    uint32_t lo;
    uint64_t hi;

    // 16 bytes at v, zero where outside the text
    __device__ __forceinline__ v4u piece(uint64_t v) const
    {
        if (v >= lo && v + 16 <= hi)
            return *(const GLB_AS v4u_any *)(p + v);
        uint64_t w0 = 0, w1 = 0;
#pragma unroll 1
        for (uint32_t j = 0; j < 16; ++j) {
            const uint64_t q = v + j;
            if (q >= lo && q < hi) {
                const uint64_t x = (uint64_t)p[q] << (8 * (j & 7));
                if (j < 8)
                    w0 |= x;
                else
                    w1 |= x;
            }
        }
        return v4u{(uint32_t)w0, (uint32_t)(w0 >> 32), (uint32_t)w1, (uint32_t)(w1 >> 32)};
    }
};

struct Raw {
    v4u r[4], tail;
};

// Block b of the view: each lane's 64 bytes and the 16 after the block.
__device__ __forceinline__ void load_block(const View &T, uint64_t b, uint32_t lane, Raw &x)
{
    const uint64_t v = b * GBLOCK;
    if (v >= T.lo && v + GBLOCK + 16 <= T.hi) {
        glb_cptr<v4u> q = (glb_cptr<v4u>)(T.p + v + lane * 64);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            x.r[k] = q[k];
        x.tail = *(glb_cptr<v4u>)(T.p + v + GBLOCK);
    } else {
        // the first and last blocks of a text
#pragma unroll 1
        for (uint32_t k = 0; k < 5; ++k) {
            const v4u t = T.piece(k < 4 ? v + lane * 64 + 16 * k : v + GBLOCK);
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i)
                if (i == k)
                    x.r[i] = t;
            x.tail = t;
        }
    }
}

// Lanes below this one set in bal.
__device__ __forceinline__ uint32_t below(uint64_t bal)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
}

__device__ __forceinline__ uint64_t uniform64(uint64_t x)
{
    return (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(x >> 32)) << 32 |
           __builtin_amdgcn_readfirstlane((uint32_t)x);
}

}  // namespace
}  // namespace mpm
