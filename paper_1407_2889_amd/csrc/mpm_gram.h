// Device helpers of the scans that look at text positions known beforehand
// (mpm_scan_gram.hip, mpm_scan_direct.hip): a wave takes 4 KiB of text, 64
// contiguous bytes per lane, as 2-bit character codes.
#pragma once
#include "mpm_scan_impl.h"

namespace mpm {
namespace {

typedef v4u v4u_any __attribute__((aligned(1)));
typedef uint64_t u64_any __attribute__((aligned(1)));
typedef uint32_t u32_any __attribute__((aligned(1)));

// Other lanes' LDS writes before this point are visible after it (one wave's
// LDS operations complete in order).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 2-bit codes (byte >> sh) & 3 of 16 bytes, the first in the low bits: per
// word one mask and one byte dot product with 1, 4, 16, 64, which leaves the
// word's eight code bits sh places up; sh <= 6.
__device__ __forceinline__ uint32_t codes16(const v4u c, uint32_t sh)
{
    const uint32_t k = 0x03030303u << sh;
    const uint32_t a = __builtin_amdgcn_udot4(c.x & k, 0x40100401u, 0u, false);
    const uint32_t b = __builtin_amdgcn_udot4(c.y & k, 0x40100401u, 0u, false);
    const uint32_t d = __builtin_amdgcn_udot4(c.z & k, 0x40100401u, 0u, false);
    const uint32_t e = __builtin_amdgcn_udot4(c.w & k, 0x40100401u, 0u, false);
    return a >> sh | b << (8 - sh) | d << (16 - sh) | e << (24 - sh);
}

// The next lane's x (lane 63: last).
__device__ __forceinline__ uint32_t from_next(uint32_t x, uint32_t last)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)x, 0x130, 0xf, 0xf, false);  // wave_shl:1
}

// The text (of 16 bytes or more) seen from the 16-byte boundary at or before
// its first byte: byte v of this view is text byte v - lo. Only bytes of the
// text, [lo, hi), are read: a 16-byte piece that reaches past either end is
// loaded from the nearest place inside, and its codes are shifted.
struct View {
    glb_cptr<uint8_t> p;
    uint32_t lo;
    uint64_t hi;

    __device__ __forceinline__ uint64_t inside(uint64_t v) const
    {
        return v < lo ? lo : v + 16 > hi ? hi - 16 : v;
    }
    __device__ __forceinline__ v4u piece(uint64_t v) const
    {
        return *(const GLB_AS v4u_any *)(p + inside(v));
    }
    // c: the codes of piece(v); zero where the piece lies outside the text
    __device__ __forceinline__ uint32_t fix(uint32_t c, uint64_t v) const
    {
        const int64_t d = (int64_t)(v - inside(v));
        return d >= 16 ? 0u : d >= 0 ? c >> (2 * (uint32_t)d) : c << (2 * (uint32_t)-d);
    }
    // Whether the 1024 * N bytes at v lie inside the text.
    template <int N>
    __device__ __forceinline__ bool whole(uint64_t v) const
    {
        return v >= lo && v + 1024 * N <= hi;
    }
    // Those bytes (v a multiple of their number): 16 * N contiguous ones per lane.
    template <int N>
    __device__ __forceinline__ void load(uint64_t v, uint32_t lane, v4u (&r)[N]) const
    {
        if (whole<N>(v)) {
            glb_cptr<v4u> q = (glb_cptr<v4u>)(p + v + lane * (16 * N));
#pragma unroll
            for (int k = 0; k < N; ++k)
                r[k] = q[k];
        } else {
#pragma unroll
            for (int k = 0; k < N; ++k)
                r[k] = piece(v + lane * (16 * N) + 16 * k);
        }
    }
    // Their codes.
    template <int N>
    __device__ __forceinline__ void codes(uint64_t v, uint32_t lane, const v4u (&r)[N], uint32_t sh,
                                          uint32_t (&c)[N]) const
    {
#pragma unroll
        for (int k = 0; k < N; ++k)
            c[k] = codes16(r[k], sh);
        if (!whole<N>(v)) {
#pragma unroll
            for (int k = 0; k < N; ++k)
                c[k] = fix(c[k], v + lane * (16 * N) + 16 * k);
        }
    }
};

// The same value, hidden from the optimizer: addresses derived from it are
// computed where they are used and not kept in registers across the passes
// over a wave's text (91 instead of 128 registers).
__device__ __forceinline__ uint64_t hidden(uint64_t x)
{
    asm volatile("" : "+s"(x));
    return x;
}

// Inclusive prefix sum over the wave's lanes: four row shifts and two row
// broadcasts, one add each.
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return x;
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

// First output slot of this wave's pairs: the wave's place in the chunk plus
// the pairs of all earlier chunks. cnt is uniform over the wave; s_scan holds
// 2 * W / 64 words. With at most WIDE_CHUNKS chunks in a launch the whole
// workgroup reads the earlier chunks' counts at once, one per thread (chunks
// of one round finish together, so that few could be skipped by a running
// total, and reading them 64 at a time is a chain of memory round trips);
// launches of more chunks look back as the walkers do.
constexpr uint64_t WIDE_CHUNKS = 1024;

// End of a launch with one chunk per workgroup and wide offsets: the last
// chunk's workgroup has seen every other chunk's count, so every workgroup
// has taken its ticket and read the epoch, and the header is made ready for
// the next launch without a counter of finished workgroups.
__device__ __forceinline__ void finish_wide(uint32_t *hdr, uint32_t epoch)
{
    __hip_atomic_store(&hdr[WS_TICKET], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&hdr[WS_EPOCH], epoch + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int W>
__device__ __forceinline__ uint64_t wave_offset(uint32_t cnt, uint64_t *s_scan, uint64_t *status, uint64_t g,
                                                uint64_t ntiles, uint64_t *total, uint32_t epoch, uint32_t *err)
{
    constexpr uint32_t NW = W / 64;
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    if (lane == 0)
        s_scan[wave] = cnt;
    __syncthreads();
    // every wave adds up the waves' counts, one per lane
    uint64_t c = lane < NW ? s_scan[lane] : 0, b4 = lane < wave ? c : 0;
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) {
        c += __shfl_xor(c, o, 16);
        b4 += __shfl_xor(b4, o, 16);
    }
    const uint64_t agg = uniform64(c), before = uniform64(b4);
    uint64_t part = 0;
    if (ntiles <= WIDE_CHUNKS) {
        const uint64_t tag = status_tag(epoch);
        if (threadIdx.x == 0)
            st_status(&status[g], make_status(epoch, 1, agg));
        if (agg == 0 && g + 1 != ntiles)  // nothing to place
            return 0;
        uint32_t spins = 0;
#pragma unroll 1
        for (uint64_t k = wave * 64; k < g; k += W) {
            const bool mine = k + lane < g;
            uint64_t v = 0;
            while (true) {
                if (mine)
                    v = ld_status(&status[g - 1 - k - lane]);
                if (__ballot(mine && v >> 38 != tag) == 0)
                    break;
                if (++spins > SPIN_LIMIT) {  // never expected; keeps every wave finite
                    if (lane == 0)
                        atomicOr(err, (uint32_t)WS_ERR_LOOKBACK);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            part += v & ST_VAL_MASK;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1)
            part += __shfl_xor(part, o, 64);
    } else if (wave == 0) {
        part = look_back(status, g, 0, agg, epoch, err);
    }
    if (lane == 0)
        s_scan[NW + wave] = part;
    __syncthreads();
    uint64_t excl = lane < NW ? s_scan[NW + lane] : 0;
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1)
        excl += __shfl_xor(excl, o, 16);
    excl = uniform64(excl);
    if (threadIdx.x == 0 && g + 1 == ntiles)
        *total = excl + agg;
    return excl + before;
}

}  // namespace
}  // namespace mpm
