// Entropy coding of the packed codes (gfx950): the rANS stage that the paper places after TAB-Q
// (Sec. II-C.2, last paragraph).  The paper leaves the coder to a third-party package; format and
// kernels here are this library's own.
//
// Format.  One frequency table per width class (all tokens of one width share it): pooled code
// counts scaled to 12 bits.  Every token is coded on its own by 64 interleaved rANS coders, one
// per lane of a wave (state in [2^16, 2^32), 16-bit renormalisation).  The token's codes are cut
// into runs of 32, as everywhere in this library; coder l owns the runs l, l + 64, ...; step i
// handles element i % 32 of run number i / 32 of every coder.  The encoder walks the steps
// backwards, the decoder forwards; the 16-bit words that the coders shed in one step are stored
// in lane order (a ballot and a population count give every lane its place).  A token's stream
// is the final states of the coders that own a run (min(64, runs) of them) followed by the words
// in the order the decoder reads them, padded to 4 bytes.
//
// Encode: code counts per width, a set per counting workgroup (k_code_pool) -> sets added up,
// tables (k_rans_tables) -> one wave per token codes its stream into a slot of the workspace
// (k_rans_encode) and adds its length to the stream bytes of its block of 256 tokens -> every token
// finds its offset from the block sums before it and the lengths before it inside its block, and its
// stream moves to its place (k_rans_gather).
// Decode: workgroups of sixteen waves, a token per wave at a time (k_rans_decode); a workgroup lays out in LDS,
// for every width class among its tokens, what each of the 4096 slots decodes to, and its waves share that.
//
// Times in this file are of calls repeated on the same buffers, unless something else is said.  On buffers that are not in the caches
// a call on 8192 x 8192 bf16 takes 3 to 5 us longer (encode 72.5 us, decode 37.5).
#include <hip/hip_runtime.h>

#include "tsq_device.hpp"
#include "tsq_internal.hpp"

namespace tsq {

typedef int i32x4 __attribute__((ext_vector_type(4)));
constexpr uint32_t kProbBits = 12, kProbScale = 1u << kProbBits, kRansLow = 1u << 16;
static_assert(kProbScale == 4096, "frequency_slot() masks 12 bits");

__device__ __forceinline__ bool eblob_is_valid(const Params &p, const EntropyLayout &e, const uint8_t *eblob) {
    // (without short cuts, as blob_is_plans)
    const EntropyHeader *h = reinterpret_cast<const EntropyHeader *>(eblob);
    const uint64_t off = h->off_streams ^ e.off_streams;
    const uint32_t unlike = (h->magic ^ kEntropyMagic) | (h->version ^ kVersion) | (h->tokens ^ p.tokens) | (h->hidden ^ p.hidden);
    return ((unlike | (uint32_t)off | (uint32_t)(off >> 32)) == 0) & (h->stream_bytes <= e.stream_capacity);
}

// ---------------------------------------------------------------- pooled counts and tables

// Counts -> 12-bit frequencies, per width class.  f_c = max(1, floor(n_c * 4096 / N))
// for n_c > 0; while the sum exceeds 4096, one is taken from the largest f (lowest code on ties);
// a remaining deficit goes to the code with the largest count (lowest code on ties).
// Taking E times one from the current largest entry is a cut at a level: with
// g(v) = sum_c max(f_c - v, 0), the level is the v with g(v + 1) < E <= g(v); every entry above
// v + 1 comes down to v + 1, and the first E - g(v + 1) entries (in code order) that then stand at
// v + 1 go down to v.  The level is found by bisection, each probe a sum over the wave.
// By one wave, lane l the codes 4l .. 4l + 3 with counts nc.
__device__ __forceinline__ void build_table(const uint32_t (&nc)[4], uint16_t *table) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t N = wave_sum_u32(nc[0] + nc[1] + nc[2] + nc[3]);
    uint32_t f[4], s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // (4096 n_c and N are exact in binary64; a quotient below an integer is so by 2^-32 at least, more than its rounding)
        f[i] = nc[i] ? (uint32_t)((double)((uint64_t)nc[i] << kProbBits) / (double)N) : 0u;
        if (nc[i] && f[i] == 0) f[i] = 1;
        s += f[i];
    }
    const uint32_t S = wave_sum_u32(s);
    auto above_level = [&](uint32_t v) {
        uint32_t g = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) g += f[i] > v ? f[i] - v : 0u;
        return wave_sum_u32(g);
    };
    if (S > kProbScale) {
        const uint32_t E = S - kProbScale;
        // g(lo) >= E always (g(0) = S > E, and the largest entry alone gives g(most - E) >= E); g(hi) = 0 < E
        const uint32_t a = f[0] > f[1] ? f[0] : f[1], b = f[2] > f[3] ? f[2] : f[3], most = wave_max_u32(a > b ? a : b);
        uint32_t lo = most > E ? most - E : 0u, hi = most;
        while (hi - lo > 1u) {                   // invariant: g(lo) >= E > g(hi)
            const uint32_t mid = (lo + hi) >> 1;
            if (above_level(mid) >= E) lo = mid; else hi = mid;
        }
        // level lo: g(lo + 1) < E <= g(lo)
        const uint32_t rest = E - above_level(lo + 1u);     // entries at lo + 1 (after the cut) that go one further down
        uint32_t n = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) n += f[i] > lo ? 1u : 0u;
        uint32_t rank = wave_incl_scan_u32(n) - n;          // of the lane's first code among those above the level
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (f[i] > lo) {
                f[i] = rank < rest ? lo : lo + 1u;
                ++rank;
            }
    } else if (N && S < kProbScale) {
        // the lowest code among those with the largest count: the largest of 256 - c over them
        const uint32_t a = nc[0] > nc[1] ? nc[0] : nc[1], b = nc[2] > nc[3] ? nc[2] : nc[3];
        const uint32_t most = wave_max_u32(a > b ? a : b);
        uint32_t mine = 0;
#pragma unroll
        for (int i = 3; i >= 0; --i)
            if (nc[i] == most) mine = 256u - (4u * lane + i);
        const uint32_t pick = wave_max_u32(mine);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (256u - (4u * lane + i) == pick) f[i] += kProbScale - S;
    }
    *reinterpret_cast<uint2 *>(table + 4u * lane) = make_uint2(f[0] | (f[1] << 16), f[2] | (f[3] << 16));
}

// Workgroup (s, k): the sets 64 s .. 64 s + 63 of the counting workgroups are added up for width class k.  With more than one
// slice the sums travel through the workspace (agent scope), and whoever arrives last adds those up and builds the
// class's table; nobody waits for anybody.
// A set per counting workgroup, up to 512 of them, is 1 MB to add up: by one workgroup per class it took longer than the
// kernel that zeroed sixteen shared sets (8192 x 8192 90 us a call against 87).
constexpr uint32_t kTableThreads = 1024;
__global__ void __launch_bounds__(kTableThreads)
k_rans_tables(const Params p, const EntropyLayout e, const uint8_t *__restrict__ blob, uint8_t *__restrict__ eblob,
              uint8_t *__restrict__ ews) {
    __shared__ uint32_t sums[4][256];
    __shared__ uint32_t last;
    const uint32_t slice = blockIdx.x, slices = gridDim.x, k = blockIdx.y, c = threadIdx.x & 255u, q = threadIdx.x >> 8;
    const uint32_t codes = 4u << k, at_set = codes - 4u + (c & (codes - 1u));   // the code's word of a set
    const uint32_t *sets = reinterpret_cast<const uint32_t *>(ews + e.ws_pooled) + at_set;
    const uint32_t g0 = slice * kTableSlice, left = e.pool_groups - g0;
    // (all loads at once: what is beyond the class's codes or the last set is read within them and dropped)
    uint32_t v[kTableSlice / 4u], n = 0;
#pragma unroll
    for (uint32_t i = 0; i < kTableSlice / 4u; ++i) {
        const uint32_t g = 4u * i + q;
        v[i] = sets[(size_t)(g0 + (g < left ? g : 0u)) * kPoolSetWords];
    }
    if (!blob_is_plans<false>(p, blob)) return;
#pragma unroll
    for (uint32_t i = 0; i < kTableSlice / 4u; ++i) n += 4u * i + q < left ? v[i] : 0u;
    sums[q][c] = c < codes ? n : 0u;
    __syncthreads();
    uint32_t *parts = reinterpret_cast<uint32_t *>(ews + e.ws_parts) + at_set;
    if (slices > 1u) {
        if (q == 0 && c < codes) {
            n = sums[0][c] + sums[1][c] + sums[2][c] + sums[3][c];
            __hip_atomic_store(parts + slice * kPoolSetWords, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // (performed before the arrival is counted)
        }
        __syncthreads();
        if (threadIdx.x == 0)
            last = __hip_atomic_fetch_add(reinterpret_cast<uint32_t *>(ews + e.ws_arrived) + k * kBlockStride, 1u,
                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == slices - 1u;
        __syncthreads();
        if (!last) return;
        const uint32_t a = __hip_atomic_load(parts + (q < slices ? q : 0u) * kPoolSetWords, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t b = __hip_atomic_load(parts + (q + 4u < slices ? q + 4u : 0u) * kPoolSetWords, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sums[q][c] = c < codes ? (q < slices ? a : 0u) + (q + 4u < slices ? b : 0u) : 0u;
        __syncthreads();
    }
    if (threadIdx.x >= 64u) return;
    uint32_t nc[4];
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t at = 4u * threadIdx.x + i;
        nc[i] = sums[0][at] + sums[1][at] + sums[2][at] + sums[3][at];
    }
    static_assert(kMaxTableSlices == 8, "two parts per thread");
    build_table(nc, reinterpret_cast<uint16_t *>(eblob + e.off_tables) + k * 256u);
}

// What a step of the encoder needs of a code with frequency f, in LDS: a binary64 reciprocal of f (see quotient()) whose
// lowest 16 bits are cum (the exclusive running sum, < 4096), and 4096 - f.  Two arrays of eight-byte places, read at one
// offset by an instruction each: what is read sixteen bytes at a time (one entry, or two places by one instruction) meets
// in the banks of LDS far more often (26 cycles a step against 11, counted on 8192 x 8192; 103 us a call against 80).
struct EncodeTable {
    double above[256];
    uint2 step[256];           // .x: 4096 - f
};
// The table of a token's class, by one wave (lane l owns the codes 4l .. 4l+3).
// A code the table does not know (f = 0; cannot happen for a table built from the blob that is
// coded) is entered with f = 1, which keeps the division defined.
__device__ __forceinline__ void load_table(const uint16_t *table, EncodeTable &ftab) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t f[4], s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) { f[i] = table[4u * lane + i]; s += f[i]; }
    uint32_t cum = wave_incl_scan_u32(s) - s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t fi = f[i] ? f[i] : 1u;
        ftab.above[4u * lane + i] = reciprocal_just_above(fi, cum & (kProbScale - 1u));
        ftab.step[4u * lane + i].x = kProbScale - fi;
        cum += f[i];
    }
}

// How many of the lanes before this one are set in `who`.
__device__ __forceinline__ uint32_t rank_in(uint64_t who) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
}

// ---------------------------------------------------------------- encode

// A SIMD holds the waves of eight tokens, each a chain of dependent steps, and its arbiter prefers the oldest
// wave: left alone, the waves finish one after the other and the last ones run with the SIMD half idle.  A wave
// therefore lowers its issue priority as it gets ahead (by quarters of its rounds), which keeps the eight in step.
// `done` of `total` rounds are behind the wave (uniform).
__device__ __forceinline__ void priority_by_progress(uint32_t done, uint32_t total) {
    switch ((4u * done) / total) {
        case 0: __builtin_amdgcn_s_setprio(3); break;
        case 1: __builtin_amdgcn_s_setprio(2); break;
        case 2: __builtin_amdgcn_s_setprio(1); break;
        default: __builtin_amdgcn_s_setprio(0); break;
    }
}

// a * b + c of 24-bit factors in one instruction (left to itself the compiler adds c and what it is the sum of to the
// product, one instruction more and all of them behind the product)
__device__ __forceinline__ uint32_t mad_u24(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t d;
    asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
// x >> 16, in x's own register
__device__ __forceinline__ void drop_word(uint32_t &x) { asm volatile("v_lshrrev_b32 %0, 16, %0" : "+v"(x)); }
// 8 times byte k of w in one instruction
__device__ __forceinline__ uint32_t eight_times_byte(uint32_t w, int k) {
    uint32_t d;
    const uint32_t three = 3;
    if (k == 0) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(d) : "v"(three), "v"(w));
    else if (k == 1) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(d) : "v"(three), "v"(w));
    else if (k == 2) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(d) : "v"(three), "v"(w));
    else asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(d) : "v"(three), "v"(w));
    return d;
}

// A 16-bit store to byte `offset` (uniform) + 2 * `index` of a buffer of 2-byte elements.
__device__ void store_short(short v, i32x4 window, int index, int zero, int offset, int policy) __asm("llvm.amdgcn.struct.buffer.store.i16");
__device__ __forceinline__ i32x4 words_window(const void *base, uint32_t words) {
    const uint64_t a = (uint64_t)base;
    return i32x4{(int)(uint32_t)a, (int)((uint32_t)(a >> 32) & 0xFFFFu) | (2 << 16), (int)words, 0x00027000};
}

// The steps of one round (run number `round` of every lane), last element first.  The words go
// straight to the token's slot in the workspace, which fills from its end downwards.
// Bound by the issue of vector instructions, 10 to 12 a step and about four cycles each, six scalar ones (4.15 cycles each on
// the unit that four SIMDs share), and 11 cycles of LDS a step and compute unit: a step takes a SIMD 74 cycles; without the
// look-ups it would take 61, without the stores 72.  Two instructions less (the place of a shed word by the memory pipeline, no
// copies of the quotient's addend): 8192 x 8192 bf16 72.4 us a call -> 71.3, 32768 x 4096 f16 147.8 -> 146.6.
// (Before that, the quotient from binary64 instead of a binary32 estimate with its correction: 87 -> 76, 169 -> 157.  Entries of
// four bytes a table, two addresses, were slower; so was a code's limit looked up, too, in sixteen bytes at once.)
// WHOLE: the run of every lane that takes part lies inside the row (valid >= 32), so no step needs a range check.
template <int B, bool WHOLE>
__device__ __forceinline__ void encode_round(const uint32_t *src_row, uint32_t run, int valid, const EncodeTable &ftab,
                                             i32x4 out, uint32_t &ptr, uint32_t &x) {
    uint32_t d[B];
    const uint32_t nd = (WHOLE || valid >= 32) ? (uint32_t)B : (valid > 0 ? ((uint32_t)valid * B + 31u) >> 5 : 0u);
    if (WHOLE) {
        load_run_words<B>(src_row + run * B, d);
    } else {
#pragma unroll
        for (int k = 0; k < B; ++k) d[k] = (uint32_t)k < nd ? src_row[run * B + k] : 0u;
    }
    // what the next step needs is looked up a step ahead
    auto look_up = [&](int j, double &above, uint32_t &step) {
        uint32_t at;                                               // 8 * code
        if constexpr (B == 8) {
            at = eight_times_byte(d[j >> 2], j & 3);
        } else {
            const int off = j * B, k = off >> 5, sh = off & 31;
            uint32_t code = d[k] >> sh;
            if (sh + B > 32) code |= d[k + 1 < B ? k + 1 : k] << (32 - sh);
            at = (code & ((1u << B) - 1u)) << 3;
        }
        above = *reinterpret_cast<const double *>(reinterpret_cast<const uint8_t *>(ftab.above) + at);
        step = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const uint8_t *>(ftab.step) + at);
    };
    double above, next_above, addend = kQuotientAddend;
    asm("" : "+v"(addend));
    uint32_t step, next_step;
    look_up(31, next_above, next_step);
#pragma unroll
    for (int j = 31; j >= 0; --j) {
        const bool active = WHOLE || j < valid;
        above = next_above;
        step = next_step;
        if (j > 0) look_up(j - 1, next_above, next_step);
        // q = floor(x / f); the state sheds a word if x >= f << 20, that is q >= 2^20, and the quotient of what is left
        // is then q >> 16
        uint32_t q = quotient(x, above, addend);
        const bool over = q >= (1u << 20), shed = active && over;
        const uint64_t who = WHOLE ? __builtin_amdgcn_ballot_w64(over) : __builtin_amdgcn_ballot_w64(active) & __builtin_amdgcn_ballot_w64(over);
        ptr -= 2u * (uint32_t)__builtin_popcountll(who);
        if (shed) {
            // (the memory pipeline doubles the rank: no instruction for the address)
            store_short((short)x, out, (int)rank_in(who), 0, (int)ptr, 0);
            drop_word(x);
            drop_word(q);
        }
        // x -> (q << 12) + (x - q f) + cum = q (4096 - f) + (x + cum)
        const uint32_t cum = (uint32_t)__builtin_bit_cast(uint64_t, above) & 0xFFFFu;
        const uint32_t y = mad_u24(q, step, x + cum);
        if (active) x = y;
    }
}

// Slot of a token in the workspace: room for 64 states (256 bytes), then room for one word per element of
// the padded row; the words stand at the END of that room (the encoder fills it backwards).
__global__ void __launch_bounds__(64)
k_rans_encode(const Params p, const EntropyLayout e, const uint8_t *__restrict__ blob, const uint8_t *__restrict__ eblob,
              uint8_t *__restrict__ ews) {
    __shared__ EncodeTable ftab;
    const uint32_t t = blockIdx.x, lane = threadIdx.x;
    uint32_t *len = reinterpret_cast<uint32_t *>(ews + e.ws_len);
    if (!blob_is_plans<false>(p, blob)) return;
    const uint32_t width = blob[p.off_bits + t];
    const uint64_t po = reinterpret_cast<const uint64_t *>(blob + p.off_pay_off)[t];
    if (!token_in_range(p, width, po)) {
        if (lane == 0) len[t] = 0;
        return;
    }
    load_table(reinterpret_cast<const uint16_t *>(eblob + e.off_tables) + (width - 2u) * 256u, ftab);
    __syncthreads();
    const uint32_t *src_row = reinterpret_cast<const uint32_t *>(blob + p.off_payload + po);
    uint8_t *slot = ews + e.ws_slots + (size_t)t * e.slot_bytes;
    const uint32_t rounds = (p.runs + 63u) / 64u, cap = e.slot_bytes - 256u;   // one word per element at most
    const i32x4 out = words_window(slot + 256, cap >> 1);
    uint32_t x = kRansLow, ptr = cap;                             // ptr: the place of the last word that was shed, in bytes
    for (uint32_t r = rounds; r-- > 0;) {
        if (rounds > 1u) priority_by_progress(rounds - 1u - r, rounds);
        const uint32_t run = lane + 64u * r;
        const int valid = (int)p.hidden - (int)(run * kRun);          // may be <= 0: nothing of this run exists
#define TSQ_ENCODE_ROUND(WHOLE)    \
    switch (width) {               \
        case 2: encode_round<2, WHOLE>(src_row, run, valid, ftab, out, ptr, x); break;  \
        case 3: encode_round<3, WHOLE>(src_row, run, valid, ftab, out, ptr, x); break;  \
        case 4: encode_round<4, WHOLE>(src_row, run, valid, ftab, out, ptr, x); break;  \
        case 5: encode_round<5, WHOLE>(src_row, run, valid, ftab, out, ptr, x); break;  \
        case 6: encode_round<6, WHOLE>(src_row, run, valid, ftab, out, ptr, x); break;  \
        case 7: encode_round<7, WHOLE>(src_row, run, valid, ftab, out, ptr, x); break;  \
        default: encode_round<8, WHOLE>(src_row, run, valid, ftab, out, ptr, x); break; \
    }
        if (__builtin_amdgcn_ballot_w64(valid > 0 && valid < 32) == 0) {
            // no run is cut: the lanes whose run lies beyond the row (the last ones, if any) sit the round out
            if (valid > 0) {
                TSQ_ENCODE_ROUND(true)
            }
            ptr = uniform(ptr);
        } else {
            TSQ_ENCODE_ROUND(false)
        }
#undef TSQ_ENCODE_ROUND
    }
    const uint32_t coders = p.runs < 64u ? p.runs : 64u;  // coders that own a run; the others still hold 2^16
    if (lane < coders) reinterpret_cast<uint32_t *>(slot)[lane] = x;
    if (lane == 0) {
        const uint32_t bytes = 4u * coders + (cap - ptr);
        len[t] = bytes;                                     // unpadded; the stream is padded to 4 bytes when it is placed
        // padded stream bytes of the token's block of kLenBlock tokens (kLenBlock slots of at most 64 KiB + 256
        // bytes: the sum fits 32 bits)
        atomicAdd(reinterpret_cast<uint32_t *>(ews + e.ws_block) + (t / kLenBlock) * kBlockStride, (bytes + 3u) & ~3u);
    }
}

// A token's stream moves from its slot to its place, by one wave: the (padded) lengths of all streams
// before it are the sums of the blocks before its block plus the lengths before it inside its block
// (64-bit: tokens * slot size may exceed 32 bits; a lane's share stays below 2^40, so it is split at bit
// 24 into two parts whose sums over 64 lanes fit 32 bits).  The first words of the stream are asked for
// ahead of those lengths: where they come from depends on the token's own length only.  The wave
// of the last token also writes the end offset and the header.
//
// The words stand at the end of the slot's room, which holds an even number of them: they start at an
// odd word exactly when their number is odd.  They move eight at a time by 16-byte loads that need no more than the two
// bytes' alignment of a word (put together from 4-byte aligned words, the loads of an odd stream waited for one another: the
// kernel took 17.3 us of 8192 x 8192's call, by the kernel trace, and takes 16.8); the last ones, fewer than eight, move two at a time, with the
// padding to 4 bytes behind an odd one.
// Three round trips bound it beside the copy: the token's length; the words, for all of which a wave waits where the compiler
// has made a branch of the second of the last two (any stream with two words or more behind its last whole piece); the lengths, state
// and block sums.
typedef uint32_t Words4_a2 __attribute__((ext_vector_type(4), aligned(2)));

// 16-byte pieces per lane that are loaded before the offset is known: 6 KB, a whole stream of up to about 8192 elements (2 KB:
// 8192 x 8192 76.5 us a call against 75.2, 32768 x 4096 157.8 / 154.7, 16384 x 8192 135.0 / 132.6; 8 KB as 6)
constexpr uint32_t kGatherEarly = 6;
__global__ void __launch_bounds__(64)
k_rans_gather(const Params p, const EntropyLayout e, const uint8_t *__restrict__ blob, uint8_t *__restrict__ eblob,
              const uint8_t *__restrict__ ews) {
    static_assert(kLenBlock == 256, "four lengths per lane inside a block");
    if (!blob_is_plans<false>(p, blob)) return;
    const uint32_t t = blockIdx.x, lane = threadIdx.x;
    const uint32_t *len = reinterpret_cast<const uint32_t *>(ews + e.ws_len);
    const uint32_t *block = reinterpret_cast<const uint32_t *>(ews + e.ws_block);
    const uint32_t blk = t / kLenBlock;
    const uint32_t coders = p.runs < 64u ? p.runs : 64u;
    const uint32_t bytes = len[t];                          // states + words, unpadded
    const uint32_t padded = (bytes + 3u) & ~3u;
    const uint32_t room = (e.slot_bytes - 256u) >> 1;
    const uint8_t *slot = ews + e.ws_slots + (size_t)t * e.slot_bytes;
    // (a length that k_rans_encode wrote passes; anything else moves nothing)
    const bool sane = bytes >= 4u * coders && bytes <= e.slot_bytes && ((bytes - 4u * coders) >> 1) <= room;
    const uint32_t nwords = sane ? (bytes - 4u * coders) >> 1 : 0u;
    const uint32_t pieces = nwords >> 3;
    const uint32_t at_words = 256u + 2u * (room - nwords);  // of the stream's words in the slot
    Words4 early[kGatherEarly];
#pragma unroll
    for (uint32_t k = 0; k < kGatherEarly; ++k) {
        const uint32_t c = lane + 64u * k;
        // (on every path, or these loads would wait for one another: a piece that is not there is the slot's first 16 bytes)
        early[k] = *reinterpret_cast<const Words4_a2 *>(slot + (c < pieces ? at_words + 16u * c : 0u));
    }
    // the last words, fewer than eight, two per lane (a word that is not there: the slot's first)
    const uint32_t i = 8u * pieces + 2u * lane;
    const uint32_t lo = *reinterpret_cast<const uint16_t *>(slot + (i < nwords ? at_words + 2u * i : 0u));
    const uint32_t hi = *reinterpret_cast<const uint16_t *>(slot + (i + 1u < nwords ? at_words + 2u * i + 2u : 0u));
    const uint32_t pair = i + 1u < nwords ? lo | (hi << 16) : lo;
    const uint32_t state = reinterpret_cast<const uint32_t *>(slot)[lane];     // (the room for 64 states is always there)

    uint32_t before[kLenBlock / 64u];
#pragma unroll
    for (uint32_t k = 0; k < kLenBlock / 64u; ++k) {
        const uint32_t u = blk * kLenBlock + lane + 64u * k;
        before[k] = len[u < t ? u : t];
    }
    uint64_t s = 0;
    for (uint32_t b = lane; b < blk; b += 64u) s += block[b * kBlockStride];
#pragma unroll
    for (uint32_t k = 0; k < kLenBlock / 64u; ++k) s += blk * kLenBlock + lane + 64u * k < t ? (before[k] + 3u) & ~3u : 0u;
    const uint64_t at = (uint64_t)wave_sum_u32((uint32_t)s & 0xFFFFFFu) + ((uint64_t)wave_sum_u32((uint32_t)(s >> 24)) << 24);

    uint64_t *off = reinterpret_cast<uint64_t *>(eblob + e.off_stream_off);
    if (lane == 0) {
        off[t] = at;
        if (t == p.tokens - 1u) {
            off[p.tokens] = at + padded;
            EntropyHeader h = {};
            h.magic = kEntropyMagic; h.version = kVersion; h.tokens = p.tokens; h.hidden = p.hidden;
            h.stream_bytes = at + padded;
            h.off_tables = e.off_tables; h.off_stream_off = e.off_stream_off; h.off_streams = e.off_streams;
            h.stream_capacity = e.stream_capacity;
            *reinterpret_cast<EntropyHeader *>(eblob) = h;
        }
    }
    if (!sane || !stream_move_ok(bytes, coders, e.slot_bytes, at, e.stream_capacity)) return;
    uint8_t *dst = eblob + e.off_streams + at;
    if (lane < coders) reinterpret_cast<uint32_t *>(dst)[lane] = state;
    uint32_t *out = reinterpret_cast<uint32_t *>(dst + 4u * coders);
    if (pieces >= 64u) {
        // Streams of more than a wave's stores are not read by this call or the next: they bypass the caches, which keep the codes and
        // the slots instead.  8192 x 8192 71.7 us a call -> 69.4, 32768 x 4096 145.8 -> 135.7; streams of a few hundred bytes, whose
        // lines are shared, would lose: 20000 x 768 51.5 / 52.0.
#pragma unroll
        for (uint32_t k = 0; k < kGatherEarly; ++k) {
            const uint32_t c = lane + 64u * k;
            if (c < pieces) __builtin_nontemporal_store(early[k], reinterpret_cast<Words4 *>(out + 4u * c));
        }
        for (uint32_t c = lane + 64u * kGatherEarly; c < pieces; c += 64u)
            __builtin_nontemporal_store(Words4(*reinterpret_cast<const Words4_a2 *>(slot + at_words + 16u * c)), reinterpret_cast<Words4 *>(out + 4u * c));
    } else if (lane < pieces) {
        *reinterpret_cast<Words4 *>(out + 4u * lane) = early[0];
    }
    if (i < nwords) out[i >> 1] = pair;
}

// ---------------------------------------------------------------- decode

// What a slot decodes to, in one word: f << 20 | c << 8 | code with c = (slot - cum) - floor(f slot / 4096), which lies
// between -1024 and 1024 (as f + cum <= 4096), so that a step of the decoder is one look-up and
// x -> f (x >> 12) + slot - cum = floor((f << 20) x / 2^32) + c: the product's upper half, with no shift of x or f before it.
// (f = 4096, the only code of its class, is entered as 0: see decode_round.)  A class's 4096 words take 16 KB; two workgroups'
// worth of LDS holds three such tables each, for the classes that most of the workgroup's tokens have.  The other classes (four at most) get
// 5 KB: the rank of a slot's code among the codes that occur, a byte per slot, and a list of those codes, (f - 1) << 20 |
// cum << 8 | code.  (Four tables, and a second turn for the tokens of further classes: 8192 x 8192 bf16 with five
// classes 57 us, this form 42, a token per workgroup 45.)
//
// What bounds it is instruction issue, vector and scalar (and, at few tokens, the chain of a step: table, product, comparison, place, word).
// 8192 x 8192 bf16: 13 vector instructions a step (49 cycles of a SIMD's issue; a word of f - 1, slot - cum and code had one
// more) and four scalar ones, and a third of what changes with a portion of the stream, which was 16 scalar and five vector
// instructions and is seven and one: 39.2 us a call -> 35.2; 32768 x 4096 f16 72.3 / 68.9, 20000 x 768 bf16 30.4 / 27.7, 2048 x
// 4096 f16 16.8 / 16.1.  (With a token per workgroup of one wave, and tables of its own in two steps, 48.)
constexpr uint32_t kDecWaves = 16, kDecThreads = 64u * kDecWaves, kDecTables = 3, kDecTableWords = kProbScale;
constexpr uint32_t kDecLists = 4, kDecListBytes = kProbScale + 256u * 4u;     // ranks, then the list
// A wave's words of the stream: a ring of two halves of 128 words, and the first half once more behind it, so
// that the up to 64 words of a step always stand in a row.
constexpr uint32_t kHalfWords = 128, kRingWords = 3 * kHalfWords;
constexpr uint32_t kDecLdsLists = kDecTables * kDecTableWords * 4u, kDecLdsRings = kDecLdsLists + kDecLists * kDecListBytes;
constexpr uint32_t kDecLdsBytes = kDecLdsRings + kDecWaves * kRingWords * 2u;
// While tables are laid out the rings' place holds, per class, one bit per slot where a code's range starts (128
// words) and the number of those bits before each of these words, and behind them the lists of the classes with a table
// (256 words each).
constexpr uint32_t kMarkWords = 128, kDecClasses = kDecTables + kDecLists;
static_assert((kDecClasses * 2u * kMarkWords + kDecTables * 256u + 2u) * 4u <= kDecWaves * kRingWords * 2u, "scratch of the table builders");
static_assert(kDecClasses == 7, "a place for every width");
static_assert(2u * kDecLdsBytes <= 160u * 1024u, "two workgroups per compute unit");

// Step 1, by one wave per class: lane l takes the codes 4l .. 4l+3, whose frequencies are f, cum and rank what lies before
// them.  The codes that occur are listed in the form of a list (RANKS), or with f in the place of f - 1; the slots where
// their ranges start are marked, and the marks counted.
struct Codes {
    uint32_t f[4], cum, rank;
};
__device__ __forceinline__ Codes codes_of(uint2 four) {
    Codes c;
    c.f[0] = four.x & 0xFFFFu; c.f[1] = four.x >> 16; c.f[2] = four.y & 0xFFFFu; c.f[3] = four.y >> 16;
    uint32_t s = 0, n = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s += c.f[i];
        n += c.f[i] ? 1u : 0u;
    }
    c.cum = wave_incl_scan_u32(s) - s;
    c.rank = wave_incl_scan_u32(n) - n;
    return c;
}
__device__ __forceinline__ void list_codes(Codes c, uint32_t *list, uint32_t *starts, bool ranks) {
    const uint32_t lane = threadIdx.x & 63u;
    *reinterpret_cast<uint2 *>(starts + 2u * lane) = make_uint2(0u, 0u);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (c.f[i]) {
            const uint32_t at = frequency_slot(c.cum);            // masked: a damaged table stays inside the array
            list[c.rank] = ((ranks ? c.f[i] - 1u : c.f[i]) << 20) | (at << 8) | (4u * lane + i);
            atomicOr(starts + (at >> 5), 1u << (at & 31u));
            ++c.rank;
        }
        c.cum += c.f[i];
    }
    const uint2 marks = *reinterpret_cast<const uint2 *>(starts + 2u * lane);
    const uint32_t a = (uint32_t)__builtin_popcount(marks.x), b = (uint32_t)__builtin_popcount(marks.y);
    const uint32_t before = wave_incl_scan_u32(a + b) - a - b;
    *reinterpret_cast<uint2 *>(starts + kMarkWords + 2u * lane) = make_uint2(before, before + a);
}
// Step 2, by all threads, four slots each: the rank of a slot's code is the number of ranges that start up to it.  Fills the
// table, or (RANKS) the ranks.
template <bool RANKS>
__device__ __forceinline__ void fill_table(const uint32_t *list, const uint32_t *starts, uint32_t *table) {
    static_assert(kDecThreads * 4u == kProbScale, "four slots a thread");
    const uint32_t word = threadIdx.x >> 3, shift = 4u * (threadIdx.x & 7u);
    const uint32_t marks = starts[word];
    uint32_t upto = starts[kMarkWords + word] + (uint32_t)__builtin_popcount(marks & ((1u << shift) - 1u)), out[4];
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        upto += (marks >> (shift + k)) & 1u;
        out[k] = upto ? upto - 1u : 0u;                           // (0: only in a damaged table)
    }
    if (RANKS) {
        table[threadIdx.x] = (out[0] & 255u) | ((out[1] & 255u) << 8) | ((out[2] & 255u) << 16) | (out[3] << 24);
    } else {
        uint32_t entry[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) entry[k] = list[out[k] & 255u];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t slot = 4u * threadIdx.x + k, f = entry[k] >> 20, cum = (entry[k] >> 8) & 0xFFFu;
            const uint32_t c = slot - cum - (__umul24(f, slot) >> kProbBits);
            out[k] = bitop3<kSelect>(0xFFFu << 8, c << 8, entry[k]);
        }
        *reinterpret_cast<uint4 *>(table + 4u * threadIdx.x) = make_uint4(out[0], out[1], out[2], out[3]);
    }
}

typedef __attribute__((address_space(3))) uint8_t *LdsBytes;
__device__ __forceinline__ uint32_t lds_address(const void *p) { return (uint32_t)(uintptr_t)(LdsBytes)p; }
template <typename T> __device__ __forceinline__ T lds_at(uint32_t address) {
    return *reinterpret_cast<const __attribute__((address_space(3))) T *>(address);
}

// The words of a token's stream on their way into the wave's ring, 128 (two per lane) at a time: two portions in
// the ring, one in a register, which replaces the older of the two when that is used up, and the one behind it
// is asked for.  What lies past the end of the stream is read as zeros: a stream that is not damaged never gets there.
// A portion lasts about three steps, so what changes with it counts, too: the memory pipeline checks the range, and every lane
// writes the copy behind the ring.
typedef uint32_t __attribute__((may_alias)) TwoWords;       // (written two words at a time, read one at a time)
typedef __attribute__((address_space(3))) TwoWords *RingWords;
struct Words {
    __amdgpu_buffer_rsrc_t src;
    uint32_t next, ahead;      // the lane's byte of the portion that is asked for next; the portion in the register
    uint32_t put;              // LDS address of the lane's two words in the first half
    uint32_t ring;             // ... of the wave's ring
    uint32_t at, end;          // ... of the next word, and of the end of the half it is in
};
__device__ __forceinline__ uint32_t load_word(__amdgpu_buffer_rsrc_t src, uint32_t at) {
    return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(src, (int)at, 0, 0);
}
__device__ __forceinline__ uint32_t next_portion(Words &q) {
    const uint32_t v = load_word(q.src, q.next);
    q.next += 2u * kHalfWords;
    return v;
}
__device__ __forceinline__ void put_first(const Words &q, uint32_t v) {
    RingWords ring = reinterpret_cast<RingWords>(q.put);
    ring[0] = v;
    ring[kHalfWords] = v;                                     // (words are counted in pairs)
}
__device__ __forceinline__ void put_second(const Words &q, uint32_t v) { reinterpret_cast<RingWords>(q.put)[kHalfWords / 2u] = v; }
// The words of the stream in window src, from byte `first` on, are asked for; when the ring is the wave's, they go there.
struct FirstWords {
    uint32_t first, second, ahead, next;
};
__device__ __forceinline__ FirstWords ask_for_words(__amdgpu_buffer_rsrc_t src, uint32_t first) {
    const uint32_t at = first + 4u * (threadIdx.x & 63u);
    return {load_word(src, at), load_word(src, at + 2u * kHalfWords), load_word(src, at + 4u * kHalfWords), at + 6u * kHalfWords};
}
__device__ __forceinline__ void words_open(Words &q, __amdgpu_buffer_rsrc_t src, const FirstWords &w, uint32_t ring) {
    q.src = src;
    q.next = w.next;
    q.ahead = w.ahead;
    q.ring = ring;
    q.put = ring + 4u * (threadIdx.x & 63u);
    put_first(q, w.first);
    put_second(q, w.second);
    q.at = ring;
    q.end = ring + 2u * kHalfWords;
}
// `n` (at most 64) more words have been read
__device__ __forceinline__ void words_advance(Words &q, uint32_t n) {
    q.at += 2u * n;
    if (q.at >= q.end) {                                      // (uniform)
        if (q.end == q.ring + 2u * kHalfWords) {
            put_first(q, q.ahead);
            q.end = q.ring + 4u * kHalfWords;
        } else {
            put_second(q, q.ahead);
            q.at -= 4u * kHalfWords;
            q.end = q.ring + 2u * kHalfWords;
        }
        q.ahead = next_portion(q);
    }
}

// The code of a step behind the codes that word d already holds: the low `bits` bits of `entry` become the top ones.
__device__ __forceinline__ uint32_t append_code(uint32_t entry, uint32_t d, int bits) {
    return __builtin_amdgcn_alignbit(entry, d, bits);
}

// store_run_words with streaming stores: see kCachedCodes.
template <int B>
__device__ __forceinline__ void store_run_words_past_caches(uint32_t *dst, const uint32_t (&d)[B]) {
    int k = 0;
#pragma unroll
    for (; k + 4 <= B; k += 4) {
        Words4 v; v.x = d[k]; v.y = d[k + 1]; v.z = d[k + 2]; v.w = d[k + 3];
        __builtin_nontemporal_store(v, reinterpret_cast<Words4 *>(dst + k));
    }
    if (k + 2 <= B) {
        Words2 v; v.x = d[k]; v.y = d[k + 1];
        __builtin_nontemporal_store(v, reinterpret_cast<Words2 *>(dst + k));
        k += 2;
    }
    if (k < B) __builtin_nontemporal_store(d[k], dst + k);
}

// The 32 steps of one round (a lane's run number `run`).  WHOLE: every lane's run lies inside the row or wholly
// beyond it (valid >= 32 or <= 0): no step needs a range check, the lanes beyond the row run idle with a limit that
// keeps them from taking words.  table: LDS address of the class's table, a multiple of its size, or (RANKS) of its
// ranks and list.
// A step is bound by instruction issue, so what the compiler would make more of than there is to it is pinned down by
// empty asm statements: the comparison with a register, the word read by every lane.
// takes: a state below it takes a word (kRansLow; 0 for a class whose only code has f = 4096: its states never change, and
// what they are does not matter, since every slot holds that code).
template <int B, bool WHOLE, bool RANKS>
__device__ __forceinline__ void decode_round(uint32_t *dst_row, uint32_t run, int valid, uint32_t table, uint32_t takes, bool past_caches,
                                             Words &q, uint32_t &x) {
    uint32_t d[B];
#pragma unroll
    for (int k = 0; k < B; ++k) d[k] = 0;
    uint32_t limit = valid > 0 ? takes : 0u, mask = 4u * (kDecTableWords - 1u), base = table;
    asm("" : "+v"(limit), "+v"(mask), "+v"(base));
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        uint32_t entry, y;
        if (RANKS) {
            const uint32_t xh = x >> kProbBits, slot = frequency_slot(x);
            entry = lds_at<uint32_t>(table + kProbScale + 4u * lds_at<uint8_t>(table + slot));
            y = xh + slot - ((entry >> 8) & 0xFFFu);
            asm("" : "+v"(y));
            y = __umul24(entry >> 20, xh) + y;                             // f <= 2^12, x >> 12 < 2^20
        } else {
            entry = lds_at<uint32_t>(bitop3<kAndOr>(x << 2, mask, base));
            y = __umulhi(entry & 0xFFF00000u, x) + (uint32_t)((int)(entry << 12) >> 20);
        }
        const int off = j * B, k = off >> 5, room = 32 - (off & 31);
        d[k] = append_code(entry, d[k], room < B ? room : B);
        if (room < B) d[k + 1 < B ? k + 1 : k] = (entry >> room) << (32 - (B - room));
        // (beyond the end of the row the limit is 0: arithmetic, since a mask per step would fill the scalar registers)
        const bool need = y < (WHOLE ? limit : limit & (uint32_t)((j - valid) >> 31));
        const uint64_t who = __builtin_amdgcn_ballot_w64(need);
        // (every lane reads: the words of a step and the up to 64 behind them are in the ring)
        uint32_t word = lds_at<uint16_t>((rank_in(who) << 1) + q.at);
        asm("" : "+v"(word));
        x = need ? (y << 16) | word : y;
        words_advance(q, (uint32_t)__builtin_popcountll(who));
    }
    if (WHOLE) {
        if (valid > 0) {
            if (past_caches) {                                // (uniform)
                // (the fences keep the two forms apart: the compiler makes one of them, an ordinary store, where it can)
                asm volatile("" ::: "memory");
                store_run_words_past_caches<B>(dst_row + run * B, d);
                asm volatile("" ::: "memory");
            } else {
                store_run_words<B>(dst_row + run * B, d);
            }
        }
    } else {
        // what the steps beyond the end of the row left in the last word goes
        const int bits = (valid < 32 ? valid : 32) * B;
#pragma unroll
        for (int k = 0; k < B; ++k)
            if (32 * k < bits) dst_row[run * B + k] = bits - 32 * k >= 32 ? d[k] : d[k] & ((1u << (bits - 32 * k)) - 1u);
    }
}

// What a wave knows of a token before it decodes it.
struct CodedToken {
    uint32_t width;
    uint64_t po, a, b;         // payload offset; stream [a, b)
};
__device__ __forceinline__ void ask_for_token(const Params &p, const EntropyLayout &e, const uint8_t *blob, const uint8_t *eblob,
                                              uint32_t t, CodedToken &k) {
    const uint64_t *off = reinterpret_cast<const uint64_t *>(eblob + e.off_stream_off);
    k.width = blob[p.off_bits + t];
    k.po = reinterpret_cast<const uint64_t *>(blob + p.off_pay_off)[t];
    k.a = off[t];
    k.b = off[t + 1];
}
// ... and what it has asked for: states and first words.  A damaged token (ok = 0) is skipped rather than read or written out
// of bounds: its stream has no bytes.
struct OpenToken {
    uint32_t ok, width;
    uint64_t po;
    __amdgpu_buffer_rsrc_t stream;
    uint32_t state;
    FirstWords words;
};
__device__ __forceinline__ OpenToken open_token(const Params &p, const EntropyLayout &e, const uint8_t *eblob, const CodedToken &c, uint32_t coders) {
    OpenToken o;
    o.width = uniform(c.width);
    o.po = c.po;
    o.ok = token_in_range(p, o.width, c.po) && stream_span_ok(c.a, c.b, e.stream_capacity, coders, e.slot_bytes) ? 1u : 0u;
    const uint64_t at = (uint64_t)(eblob + e.off_streams) + (o.ok ? c.a : 0u);
    o.stream = raw_window(reinterpret_cast<void *>((uint64_t)uniform((uint32_t)(at >> 32)) << 32 | uniform((uint32_t)at)),
                          uniform(o.ok ? (uint32_t)(c.b - c.a) : 0u));
    o.state = load_word(o.stream, 4u * (threadIdx.x & 63u));
    o.words = ask_for_words(o.stream, 4u * coders);
    return o;
}

// How many of the tokens t0 .. t1 - 1 have which width, and the places of the classes that occur, the most frequent first:
// places 0 .. kDecTables - 1 are tables.  Four bits per class: its place; and the number of classes.  By one
// wave (every wave for itself, with scalar comparisons, took 1.9 us of 8192 x 8192's 35).
struct Places {
    uint32_t place_of, n;
};
__device__ __forceinline__ Places places_of(const uint8_t *bits, uint32_t t0, uint32_t t1) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t count[kDecClasses] = {};
    for (uint32_t i = t0; i < t1; i += 64u) {
        const uint32_t b = i + lane < t1 ? bits[i + lane] : 0u;
#pragma unroll
        for (uint32_t k = 0; k < kDecClasses; ++k) count[k] += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(b == k + 2u));
    }
    // lane k: class k's count, and before it the lower class's that has the same
    uint32_t mine = 0;
#pragma unroll
    for (uint32_t k = 0; k < kDecClasses; ++k) mine = lane == k ? (count[k] << 3) + 7u - k : mine;
    uint32_t place = 0;
#pragma unroll
    for (uint32_t k = 0; k < kDecClasses; ++k) place += lane_value(mine, (int)k) > mine ? 1u : 0u;
    const bool is_class = lane < kDecClasses;
    Places r;
    r.place_of = wave_sum_u32(is_class ? place << (4u * lane) : 0u);
    r.n = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(is_class && (mine >> 3)));
    return r;
}

// A call that writes more than kCachedCodes bytes of codes stores them past the caches: restore finds few of them there by the
// time it reads them, and on their way they push out the streams.  Up to there restore reads them from the memory-side cache (256
// MB), which is worth more to the two calls than what decode gains by itself.  Decode with restore behind it, stored past the
// caches against not: 25 MB of codes (13000 x 8192 bf16 at two bits) 101.1 us / 88.7, 107 MB (16384 x 8192 f16) 123.1 / 117.7, 130 MB
// (20000 x 8192 bf16) 154.5 / 145.6; 158 MB (40000 x 5120 f16) 207.9 / 217.1, 206 MB (65536 x 4096 f16) 252.8 / 264.1, 198 MB (50000 x
// 5120) 252.8 / 269.6; rows of 8192 and more differ by 4 % either way from 150 to 250 MB.  Decode by itself: 13000 x 8192 48.5 /
// 50.0, 16384 x 8192 57.6 / 60.2, 20000 x 8192 73.2 / 74.8, 65536 x 4096 125.1 / 129.4.
// The bytes are those that the blob holds: what the plan has room for says little about them (a line at 96 MB of room for the largest
// width sent the 25 MB of the first example past the caches).
constexpr uint64_t kCachedCodes = 160ull << 20;

// Workgroup g decodes the tokens per * g .. per * g + per - 1, a token per wave and turn.  Before the first one can start, its
// workgroup's tables have to be laid out; the wave's first words and what the tables are made of are asked for together, and
// only then waited for.
__global__ void __launch_bounds__(kDecThreads, 8)    // 8 waves per SIMD: two workgroups per compute unit
k_rans_decode(const Params p, const EntropyLayout e, const uint8_t *__restrict__ eblob, uint8_t *__restrict__ blob, uint32_t per) {
    extern __shared__ __align__(4 * kDecTableWords) uint32_t lds[];     // (tables, each at a multiple of its size; then the rings)
    const uint32_t lane = threadIdx.x & 63u, wv = uniform(threadIdx.x >> 6);
    const uint32_t t0 = blockIdx.x * per, t1 = p.tokens - t0 < per ? p.tokens : t0 + per;
    const uint32_t coders = p.runs < 64u ? p.runs : 64u;  // states in the stream; the other coders start (and stay) at 2^16
    const uint32_t rounds = (p.runs + 63u) / 64u;
    const bool blob_ours = blob_is_plans<false>(p, blob), eblob_ours = eblob_is_valid(p, e, eblob);     // (no verdict waits for the other)
    if (!blob_ours || !eblob_ours) return;
    const bool past_caches = reinterpret_cast<const BlobHeader *>(blob)->payload_bytes > kCachedCodes;
    uint32_t t = t0 + wv;
    // (a wave without a token looks at the last one's and decodes none)
    CodedToken next;
    ask_for_token(p, e, blob, eblob, t < t1 ? t : t1 - 1u, next);
    const uint2 four = reinterpret_cast<const uint2 *>(eblob + e.off_tables)[(wv < kDecClasses ? wv : 0u) * 64u + lane];

    // ---- the tables
    uint32_t *scratch = lds + kDecLdsRings / 4u, *told = scratch + kDecClasses * 2u * kMarkWords + kDecTables * 256u;
    auto marks_at = [&](uint32_t place) { return scratch + place * 2u * kMarkWords; };
    auto list_at = [&](uint32_t place) {
        return place < kDecTables ? scratch + kDecClasses * 2u * kMarkWords + place * 256u
                                  : lds + (kDecLdsLists + (place - kDecTables) * kDecListBytes + kProbScale) / 4u;
    };
    if (wv == kDecWaves - 1u) {
        const Places r = places_of(blob + p.off_bits, t0, t1);
        if (lane == 0) { told[0] = r.place_of; told[1] = r.n; }
    }
    OpenToken o = open_token(p, e, eblob, next, coders);
    const Codes codes = codes_of(four);
    __syncthreads();
    const uint32_t place_of = uniform(told[0]), n = uniform(told[1]);
    const uint32_t own = (place_of >> (4u * (wv < kDecClasses ? wv : 0u))) & 15u;      // the place of the class that this wave lists
    if (wv < kDecClasses && own < n) list_codes(codes, list_at(own), marks_at(own), own >= kDecTables);
    __syncthreads();
    for (uint32_t place = 0; place < n; ++place) {
        if (place < kDecTables) fill_table<false>(list_at(place), marks_at(place), lds + place * kDecTableWords);
        else fill_table<true>(nullptr, marks_at(place), list_at(place) - kProbScale / 4u);
    }
    __syncthreads();

    const uint32_t ring = lds_address(lds) + kDecLdsRings + wv * kRingWords * 2u;
    // ---- the tokens
    while (t < t1) {
        const uint32_t width = o.width;
        if (o.ok) {
            const uint32_t place = (place_of >> (4u * (width - 2u))) & 15u;
            const bool ranks = place >= kDecTables;
            const uint32_t table = lds_address(lds) + (ranks ? kDecLdsLists + (place - kDecTables) * kDecListBytes : place * (4u * kDecTableWords));
            uint32_t x = lane < coders ? o.state : kRansLow;
            Words q;
            words_open(q, o.stream, o.words, ring);
            const uint32_t takes = ranks || lds_at<uint32_t>(table) >> 20 ? kRansLow : 0u;
            uint32_t *dst_row = reinterpret_cast<uint32_t *>(blob + p.off_payload + o.po);
            for (uint32_t r = 0; r < rounds; ++r) {
                priority_by_progress(r, rounds);
                const uint32_t run = lane + 64u * r;
                const int valid = (int)p.hidden - (int)(run * kRun);
#define TSQ_DECODE_ROUND(WHOLE, RANKS) \
    switch (width) {                   \
        case 2: decode_round<2, WHOLE, RANKS>(dst_row, run, valid, table, takes, past_caches, q, x); break;  \
        case 3: decode_round<3, WHOLE, RANKS>(dst_row, run, valid, table, takes, past_caches, q, x); break;  \
        case 4: decode_round<4, WHOLE, RANKS>(dst_row, run, valid, table, takes, past_caches, q, x); break;  \
        case 5: decode_round<5, WHOLE, RANKS>(dst_row, run, valid, table, takes, past_caches, q, x); break;  \
        case 6: decode_round<6, WHOLE, RANKS>(dst_row, run, valid, table, takes, past_caches, q, x); break;  \
        case 7: decode_round<7, WHOLE, RANKS>(dst_row, run, valid, table, takes, past_caches, q, x); break;  \
        default: decode_round<8, WHOLE, RANKS>(dst_row, run, valid, table, takes, past_caches, q, x); break; \
    }
                if (__builtin_amdgcn_ballot_w64(valid > 0 && valid < 32) == 0) {
                    if (ranks) {
                        TSQ_DECODE_ROUND(true, true)
                    } else {
                        TSQ_DECODE_ROUND(true, false)
                    }
                } else if (ranks) {
                    TSQ_DECODE_ROUND(false, true)
                } else {
                    TSQ_DECODE_ROUND(false, false)
                }
#undef TSQ_DECODE_ROUND
            }
        }
        t += kDecWaves;
        if (t < t1) {
            ask_for_token(p, e, blob, eblob, t, next);
            o = open_token(p, e, eblob, next, coders);
        }
    }
}

// ---------------------------------------------------------------- launchers

static hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

int launch_rans_encode(const Params &p, const EntropyLayout &e, const void *d_blob, void *d_eblob,
                       void *d_ews, void *stream) {
    const uint8_t *blob = static_cast<const uint8_t *>(d_blob);
    uint8_t *eblob = static_cast<uint8_t *>(d_eblob), *ews = static_cast<uint8_t *>(d_ews);
    hipStream_t s = as_stream(stream);
    int rc = launch_code_pool(p, e, d_blob, d_eblob, d_ews, stream);
    if (rc != 0) return rc;
    hipLaunchKernelGGL(k_rans_tables, dim3((e.pool_groups + kTableSlice - 1u) / kTableSlice, 7), dim3(kTableThreads), 0, s, p, e, blob,
                       eblob, ews);
    hipLaunchKernelGGL(k_rans_encode, dim3(p.tokens), dim3(64), 0, s, p, e, blob, eblob, ews);
    hipLaunchKernelGGL(k_rans_gather, dim3(p.tokens), dim3(64), 0, s, p, e, blob, eblob, ews);
    return (int)hipGetLastError();
}

int prepare_rans_kernels() {
    return (int)hipFuncSetAttribute(reinterpret_cast<const void *>(k_rans_decode), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDecLdsBytes);
}

int launch_rans_decode(const Params &p, const EntropyLayout &e, const void *d_eblob, void *d_blob, void *stream) {
    // one round of workgroups (two on each of 256 compute units), a token per wave if there are enough of them;
    // fewer tokens are spread over as many workgroups as there are
    const uint32_t per = (p.tokens + kMaxDecodeGroups - 1u) / kMaxDecodeGroups;
    hipLaunchKernelGGL(k_rans_decode, dim3((p.tokens + per - 1u) / per), dim3(kDecThreads), kDecLdsBytes, as_stream(stream), p, e,
                       static_cast<const uint8_t *>(d_eblob), static_cast<uint8_t *>(d_blob), per);
    return (int)hipGetLastError();
}

}  // namespace tsq
