// Building blocks of the single-pass compress kernels (tsq_fused.hip, tsq_direct.hip): the words through which
// workgroups tell one another the sizes of their tokens, the row in LDS, and the payload image in LDS.
#pragma once

#include <hip/hip_runtime.h>

#include "tsq_device.hpp"
#include "tsq_internal.hpp"

namespace tsq {

constexpr uint32_t kTicketBits = 24, kTicketMask = (1u << kTicketBits) - 1u;
enum { kCntTickets = 0, kCntDone = 1 };      // words of a class's counter line

// Table word: bits 31..30 = tag of the call (0 = never written), bits 29..26 = width of the token,
// bits 15..0 = its outliers (<= 32768).
// Prefix word: bits 63..62 = tag, bits 61..32 = payload words before the token, bits 31..0 =
// outliers before the token.
__device__ __forceinline__ uint32_t word_load(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void word_store(uint32_t *p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t prefix_load(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void prefix_store(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A zero the compiler knows nothing about, in a vector register: an address formed with it is
// not provably the same in every lane, so loads and atomics through it stay vector operations
// that go to memory (a provably uniform one may become a scalar load, or a wave-wide reduction
// whose result is waited for on the spot).
__device__ __forceinline__ uint32_t opaque_zero() {
    uint32_t zero = 0;
    asm volatile("" : "+v"(zero));
    return zero;
}

// A uniform value that the compiler is to keep as it is now, instead of deriving it again from its (wider)
// sources wherever it is used.
__device__ __forceinline__ uint32_t as_computed(uint32_t v) {
    asm volatile("" : "+s"(v));
    return v;
}

// One more round of a bounded wait: false when the limit is reached or somebody has already
// given up (checked now and then, so that a broken run ends quickly everywhere).
__device__ __forceinline__ bool keep_waiting(uint32_t &spins, uint32_t limit, const uint32_t *error_flag) {
    if (++spins >= limit) return false;
    if ((spins & 255u) == 0 && __hip_atomic_load(error_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
    __builtin_amdgcn_s_sleep(2);
    return true;
}
__device__ __forceinline__ void raise_error(uint32_t *error_flag) {
    // with its result: the atomic has been performed when the wave goes on
    const uint32_t old = __hip_atomic_fetch_or(error_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::"v"(old));
}

// ---- the row in LDS: 16 dwords per run, no padding.  The four 16-byte chunks of run r are
// stored in the order k ^ ((r >> 1) & 3), which spreads eight neighbouring runs over all 32
// banks for 16-byte accesses.  Every wave moves, reads and overwrites only the 4 KB of the row
// that its own lanes own (runs 64w .. 64w+63), so the row needs no workgroup barrier.
// (A row loaded straight into LDS, without the registers in between, does not pay here: the
// compiler makes every later LDS access of the wave wait for such a load, the reductions of
// the width search included.) ----
template <bool FULL>
__device__ __forceinline__ void write_row_part_sw(uint32_t *lrow, uint32_t runs, const RowPart &pre) {
    const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
    const uint32_t q0 = 256u * wv + lane;                  // first 16-byte piece of the row this lane moves
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t q = q0 + 64u * k, r = q >> 2, c = (q & 3u) ^ ((r >> 1) & 3u);
        if (FULL || r < runs)
            *reinterpret_cast<uint4 *>(lrow + r * 16u + c * 4u) =
                make_uint4(pre.w[4 * k], pre.w[4 * k + 1], pre.w[4 * k + 2], pre.w[4 * k + 3]);
    }
}
__device__ __forceinline__ void load_run_sw(const uint32_t *lrow, uint32_t r, uint32_t (&w)[16]) {
    const uint32_t sw = (r >> 1) & 3u;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        const uint4 q = *reinterpret_cast<const uint4 *>(lrow + r * 16u + ((k ^ sw) << 2));
        w[4 * k] = q.x; w[4 * k + 1] = q.y; w[4 * k + 2] = q.z; w[4 * k + 3] = q.w;
    }
}
__device__ __forceinline__ uint32_t raw_element_sw(const uint32_t *lrow, uint32_t r, uint32_t j) {
    // byte 2j of the run, its 16-byte chunk index xor-ed with the run's swizzle: the run's part of
    // the address does not depend on j
    const uint32_t at = ((r * 64u) | (((r >> 1) & 3u) << 4)) ^ (j << 1);
    return *reinterpret_cast<const uint16_t *>(reinterpret_cast<const uint8_t *>(lrow) + at);
}

// A run's 16-bit values two by two, for the packing (which takes their signs): fp16 has them in registers; bf16 reads its
// row from LDS once more, which costs less than the instructions that take the signs out of 32 binary32 values, and than
// those values' registers (131072 x 8192 bf16 705 us -> 684).
template <int DT>
__device__ __forceinline__ void signed_values(const Mags<DT> &mg, const uint32_t *lrow, uint32_t r, uint32_t (&w)[16]) {
    if constexpr (DT == kF16) {
#pragma unroll
        for (int k = 0; k < 16; ++k) w[k] = mg.v[k];
    } else {
        load_run_sw(lrow, r, w);
    }
}

// nd dwords of packed codes of a run into the token's payload image in LDS
template <int B, bool FULL>
__device__ __forceinline__ void put_codes(uint32_t *dst, const uint32_t (&o)[8], uint32_t nd) {
    if (FULL || nd >= (uint32_t)B) {
        int k = 0;
        // the image is 16-byte aligned and run*B dwords in: use the widest stores the alignment allows
        if (B % 4 == 0) {
#pragma unroll
            for (; k + 4 <= B; k += 4) *reinterpret_cast<uint4 *>(dst + k) = make_uint4(o[k], o[k + 1], o[k + 2], o[k + 3]);
        } else if (B % 2 == 0) {
#pragma unroll
            for (; k + 2 <= B; k += 2) *reinterpret_cast<uint2 *>(dst + k) = make_uint2(o[k], o[k + 1]);
        } else {
#pragma unroll
            for (; k < B; ++k) dst[k] = o[k];
        }
    } else {
#pragma unroll
        for (int k = 0; k < B; ++k)
            if ((uint32_t)k < nd) dst[k] = o[k];
    }
}
template <int B, bool FULL>
__device__ __forceinline__ void pack_to_image(const uint32_t (&m)[8], const uint32_t (&w)[16], uint32_t *dst, uint32_t nd) {
    uint32_t o[8];
    {
        uint32_t t[B];
        pack_regs<B>(m, w, t);
#pragma unroll
        for (int k = 0; k < B; ++k) o[k] = t[k];
    }
    put_codes<B, FULL>(dst, o, nd);
}

__device__ __forceinline__ uint64_t prefix_word(uint32_t tag, uint32_t ew, uint32_t ec) {
    return ((uint64_t)((tag << 30) | ew) << 32) | ec;
}

}  // namespace tsq
