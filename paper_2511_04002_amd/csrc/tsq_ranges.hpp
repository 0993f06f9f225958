// Admissibility of offsets and sizes that a kernel reads from memory it does not own (a blob, an
// entropy-coded blob, a workspace) before it uses them as addresses.  Plain integer predicates on
// plain values, written without sums of untrusted values (which could wrap), compiled for the
// device (the kernels call them) and for the host (tsq_check_* in tsq_api.hip evaluates them
// for tests that need no GPU).  Also here, for the same reason: the one piece of the entropy coder's
// arithmetic whose exactness rests on a rounding argument.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define TSQ_HD __host__ __device__ __forceinline__
#else
#define TSQ_HD inline
#endif

namespace tsq {

// bytes of one token's payload at width b: b bits per element, padded to a 4-byte multiple
TSQ_HD uint32_t payload_row_bytes(uint32_t hidden, uint32_t b) { return 4u * ((hidden * b + 31u) >> 5); }

// A token of width b whose payload starts at byte po of a payload section of `capacity` bytes:
// a width of the format, 4-byte aligned, and wholly inside the section.
TSQ_HD bool payload_span_ok(uint32_t hidden, uint64_t capacity, uint32_t b, uint64_t po) {
    if (b < 2 || b > 8 || (po & 3u) || po > capacity) return false;
    return payload_row_bytes(hidden, b) <= capacity - po;
}

// The CSR slice [rp0, rp1) of a token as restore reads it: ordered and inside the side stream.
TSQ_HD bool csr_slice_ok(uint64_t rp0, uint64_t rp1, uint64_t capacity) { return rp0 <= rp1 && rp1 <= capacity; }

// The CSR slice of a token as compress writes it: it must also hold exactly the token's `cnt` outliers.
TSQ_HD bool csr_slice_holds(uint64_t rp0, uint64_t rp1, uint64_t capacity, uint32_t cnt) {
    return csr_slice_ok(rp0, rp1, capacity) && rp1 - rp0 == (uint64_t)cnt;
}

// A column index read from the side stream.
TSQ_HD bool column_ok(uint32_t col, uint32_t hidden) { return col < hidden; }

// The stream [a, b) of one token inside the streams section of an entropy-coded blob: ordered, 4-byte
// aligned, inside the section, at least the `coders` 32-bit states long and no longer than a slot.
TSQ_HD bool stream_span_ok(uint64_t a, uint64_t b, uint64_t capacity, uint32_t coders, uint32_t slot_bytes) {
    if (a > b || b > capacity || (a & 3u)) return false;
    const uint64_t n = b - a;
    return n >= 4ull * coders && n <= (uint64_t)slot_bytes;
}

// A coded stream of `bytes` bytes moving from its slot to byte `at` of the streams section.
TSQ_HD bool stream_move_ok(uint32_t bytes, uint32_t coders, uint32_t slot_bytes, uint64_t at, uint64_t capacity) {
    if (bytes < 4u * coders || bytes > slot_bytes || at > capacity) return false;
    return (uint64_t)((bytes + 3u) & ~3u) <= capacity - at;
}

// Index into the 4096-entry cumulative-frequency table from a coder state.
TSQ_HD uint32_t frequency_slot(uint32_t state) { return state & 4095u; }

// The entropy coder's division: floor(x / f) for f <= x < 2^32 and 1 <= f <= 4096, from a binary64 number `above` in
// (1 / f, (1 + d) / f] with d <= 2^-34.  The exact product v = x * above is then more than x / f and at most
// x / f + 1 / (4 f), so it has the integer part of x / f and stays at least 3 / (4 f) below the next integer.  The one
// rounding of v + (2^52 - 1/2), to a multiple of 1 since the sum is 2^52 or more (v > 1), is to the nearest: v - 1/2 lies
// strictly between floor(v) - 1/2 and floor(v) + 1/2, so the result is 2^52 + floor(v), whose lower word is the quotient.
// The lowest 16 bits of `above` are free: it is the rounded 1 / f with those bits cut off, plus 2^16 units of its last
// place, plus any `low` < 2^16 units (at most 2^17 of them beyond 1 / f: d <= 2^-35).
TSQ_HD double reciprocal_just_above(uint32_t f, uint32_t low) {
    const uint64_t r = __builtin_bit_cast(uint64_t, 1.0 / (double)f);
    return __builtin_bit_cast(double, (r & ~0xFFFFull) + 0x10000ull + low);
}
constexpr double kQuotientAddend = 4503599627370495.5;      // 2^52 - 1/2
// addend: kQuotientAddend, which a kernel keeps in registers for all its divisions.  There the product is named as the
// instruction that it is: left to itself the compiler copies the addend for half of them, to accumulate into the copy.
TSQ_HD uint32_t quotient(uint32_t x, double above, double addend) {
#if defined(__HIP_DEVICE_COMPILE__)
    double v;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(v) : "v"((double)x), "v"(above), "v"(addend));
#else
    const double v = __builtin_fma((double)x, above, addend);
#endif
    return (uint32_t)__builtin_bit_cast(uint64_t, v);
}

// A workspace's recorded shape against the plan's.
TSQ_HD bool workspace_shape_ok(uint32_t ws_tokens, uint32_t ws_hidden, uint32_t tokens, uint32_t hidden) {
    return ws_tokens == tokens && ws_hidden == hidden;
}

}  // namespace tsq
