// Single-pass compress for calls of few tokens and for rows of one wave (gfx950): one workgroup per token, or per eight
// tokens of one wave, or per two of two waves, dispatched in token order, nothing handed out and nobody in between.
//
// With as many workgroups as tokens a call is one chain of latencies: row from HBM, threshold split, width
// search, publication of the token's size, sizes of the tokens before it, stores.  The persistent kernel
// (tsq_fused.hip) adds to that chain a ticket before the row, a scanner's round between a token's publication
// and its prefix, and a count of finished waves that the scanner waits for before it closes the blob; those
// are worth their time when a workgroup has many tokens, and are most of the call when it has one.
//
// Placement: the tokens are cut into blocks of kDirectBlock.  A workgroup adds up, for itself, the published
// words of the tokens before it in its block (one or a few words per thread) and the prefix word of the
// block's first token, which the last token of the block before has published.
//
// Progress: whoever waits, waits for tokens of lower index only, and every die starts the workgroups it gets in the
// order of their index.  So when all tokens before one are finished, that one has started or is the next of its die to
// start, and the call ends whatever the number of workgroups that fit the device.  This rests on that order, and on
// other work leaving every die room for a workgroup (up to 16 waves and 97 KB of LDS with a token each; groups of eight
// short rows take 8 waves and up to 49 KB, where one of them by itself takes 1 and 6): a die that something else fills keeps its tokens from starting, and
// those on the other dies wait for them (the persistent kernel hands such tokens to workgroups that run, but its
// scanner waits for every workgroup in the end).  Every wait is bounded by p.spin_limit, about a second.
//
// The last token's workgroup closes the blob: by the time it has its prefix every token is published, so
// everybody has read the call's epoch and it can be moved on.  The header's status word is stored (device
// scope) before anything else by that workgroup, and it reads the workspace's error word after that store has
// been performed; a workgroup that fails raises the error word first and stores TSQ_ERR_INTERNAL into the status
// word after that.  Whichever comes first, a failure ends up in the header.
#include <hip/hip_runtime.h>

#include "tsq_device.hpp"
#include "tsq_internal.hpp"
#include "tsq_pass.hpp"

namespace tsq {

constexpr uint32_t kStatusWord = 9;                      // BlobHeader::status, in 32-bit words
static_assert(offsetof(BlobHeader, status) == 4 * kStatusWord, "status word of the header");
constexpr uint32_t kStatusFormat = 5u, kStatusInternal = 6u, kStatusCapacity = 3u;
// what a wave adds to its count of outliers when it has seen the workspace's error word, or another plan's shape: the
// sums over a workgroup's waves leave the counts (at most kMaxHidden in all) and one another alone
constexpr uint32_t kSawError = 1u << 20, kSawShape = 1u << 25;
static_assert(kMaxHidden < kSawError && kMaxHidden + kMaxWaves * kSawError < kSawShape && kMaxWaves * kSawShape < (1u << 31),
              "fields of the waves' sums");

__device__ __forceinline__ void store_status(uint8_t *blob, uint32_t status) {
    word_store(reinterpret_cast<uint32_t *>(blob) + kStatusWord, status);
}
__device__ __forceinline__ void memory_operations_performed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Payload words of a token of width b (0 for the width 0 of a word that counts nothing).
__device__ __forceinline__ uint32_t token_words(const Params &p, uint32_t b) { return (p.hidden * b + 31u) >> 5; }

template <int B>
__device__ __forceinline__ void pack_codes(const uint32_t (&m)[8], const uint32_t (&w)[16], uint32_t (&o)[8]) {
    uint32_t t[B];
    pack_regs<B>(m, w, t);
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = k < B ? t[k] : 0u;
}

// The pieces q, q + 64, q + 128 and q + 192 (16 bytes each) of a row at a uniform address, zeros for those behind its end, which
// the memory pipeline checks: a branch per piece made the loads of some rows wait for one another, and took its time where
// nothing else is to do.  Streaming: the input is read once.
template <bool FULL>
__device__ __forceinline__ void fetch_row_once(const uint16_t *row, uint32_t pieces, uint32_t q, RowPart &part) {
    const GlobalBytes src = (GlobalBytes)row;
    const __amdgpu_buffer_rsrc_t window = raw_window(const_cast<uint16_t *>(row), 16u * pieces);
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        u32x4 v;
        if constexpr (FULL) v = __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4 *)(src + 16u * q + 1024u * k));
        else v = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(window, (int)(16u * q + 1024u * k), 0, 2));
        part.w[4 * k] = v.x; part.w[4 * k + 1] = v.y; part.w[4 * k + 2] = v.z; part.w[4 * k + 3] = v.w;
    }
}

// The last workgroup's first wave closes the blob, also if its own wait has expired (nobody else writes a header).
// raised: the error word as it was before that workgroup published its size.
__device__ __forceinline__ void close_blob(const Params &p, uint8_t *blob, uint32_t *tickets, uint32_t *error_flag, uint32_t epoch,
                                           uint32_t bad, uint32_t words_in_all, uint64_t outliers_in_all, uint32_t raised) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t all_words = bad ? 0u : words_in_all;
    const uint64_t all_outliers = bad ? 0u : outliers_in_all;
    if (!bad) word_store(tickets + lane * kTicketStride + kCntTickets, ((epoch + 1u) % 3u) << kTicketBits);   // everybody has this call's
    if (lane == 0) {
        const bool full = all_outliers > p.outlier_capacity;
        if (full) {                            // (as the zero at the start: in its place before the error word is read again)
            store_status(blob, kStatusCapacity);
            memory_operations_performed();
            raised |= word_load(error_flag + opaque_zero());
        }
        reinterpret_cast<uint64_t *>(blob + p.off_row_ptr)[p.tokens] = all_outliers;
        reinterpret_cast<uint64_t *>(blob + p.off_pay_off)[p.tokens] = (uint64_t)all_words << 2;
        write_header_but_status(p, blob, all_outliers, (uint64_t)all_words << 2);
        if (raised) store_status(blob, kStatusInternal);
    }
}

// LDS map (dynamic): row: runs*16 dwords | codes: runs*8 | ring (rows of more than one wave): four reduce areas
constexpr uint32_t kDirectRing = 4u * 2u * kMaxWaves;
template <int DT, int NW, bool FULL>
__global__ void __launch_bounds__(64 * NW, DT == kF16 && NW <= 4 ? 8 : 5)
k_direct(const Params p, const uint16_t *__restrict__ in, uint8_t *__restrict__ blob, uint8_t *__restrict__ ws) {
    extern __shared__ __align__(16) uint32_t lds[];
    const uint32_t t = blockIdx.x, tid = threadIdx.x, lane = tid & 63u, wv = uniform(tid >> 6);
    const uint32_t runs = FULL ? 64u * NW : p.runs, pieces = FULL ? 256u * NW : p.pieces;
    const bool owns = FULL || tid < runs;
    const uint32_t left = FULL ? 4u : (owns ? pieces - 4u * tid : 0u);    // 16-byte pieces of the lane's run inside the row
    uint32_t *lrow = lds, *image = lds + runs * 16u, *ring = lds + runs * 24u;
    const bool last = t == p.tokens - 1u;

    RowPart part;
    fetch_row_once<FULL>(row_address(p, in, t, FULL ? 2048u * NW : p.hidden), pieces, 256u * wv + lane, part);

    // error word, shape and epoch of the workspace, one per lane of one load
    uint32_t *ctrl = reinterpret_cast<uint32_t *>(ws + p.ws_ctrl);
    uint32_t *tickets = reinterpret_cast<uint32_t *>(ws + p.ws_tickets);
    uint32_t *error_flag = ctrl + kCtlError;
    const uint32_t *mine = lane == 0 ? error_flag : lane == 1 ? ctrl + kCtlTokens : lane == 2 ? ctrl + kCtlHidden : tickets + kCntTickets;
    const uint32_t state = __hip_atomic_load(mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (NW > 1) {
        clear_areas(ring);
        lds_barrier();
    }

    write_row_part_sw<FULL>(lrow, runs, part);
    Mags<DT> mg;
    uint32_t omask = 0, amax_bits = 0, turn = 0;
    {
        uint32_t w[16];
        load_run_sw(lrow, owns ? tid : 0u, w);
        split_regs<DT, true>(w, p.thr_pk, mg, omask, amax_bits);
    }
    if (!owns) { omask = 0; amax_bits = 0; }

    // A workspace of another shape (or never reset), or one that a call left in its failed state: nothing in it is
    // touched, and the blob says so.  Every wave has looked for itself, and another workgroup may raise the error word
    // between two of the looks, so the waves decide together: what a wave saw travels above its count of outliers.
    const bool shape_ok = workspace_shape_ok(lane_value(state, 1), lane_value(state, 2), p.tokens, p.hidden);
    const uint32_t refused = (lane_value(state, 0) ? kSawError : 0u) + (shape_ok ? 0u : kSawShape);
    const uint32_t epoch = (lane_value(state, 3) >> kTicketBits) % 3u, tag = epoch + 1u;
    if (last && tid == 0) store_status(blob, 0u);

    const uint32_t nl = (uint32_t)__builtin_popcount(omask);
    const uint32_t upto = wave_incl_scan_u32(nl);                 // outliers of the wave's lanes up to this one
    const RowStats st = reduce_row_stats_counted<NW>(amax_bits, lane_value(upto, 63) + refused, ring, turn);
    if (st.cnt >= kSawError) {
        if (last && tid == 0) write_header(p, blob, 0, 0, st.cnt >= kSawShape ? kStatusFormat : kStatusInternal);
        return;
    }
    uint32_t m[8];
    const Choice c = search_width<DT, NW>(p, mg, st.amax, owns, ring, turn, m);

    uint32_t *sizes = reinterpret_cast<uint32_t *>(ws + p.ws_sizes);
    uint64_t *pre = reinterpret_cast<uint64_t *>(ws + p.ws_prefix);
    // (the last token's workgroup looks for failures now, with the status word's zero long in place, and not when it
    // closes the blob, where everybody would wait for the answer)
    uint32_t raised = 0;
    if (last && wv == 0) {
        memory_operations_performed();
        raised = word_load(error_flag + opaque_zero());
    }
    if (tid == 0) {
        word_store(sizes + t, (tag << 30) | (c.width << 26) | st.cnt);
        blob[p.off_bits + t] = (uint8_t)c.width;
        reinterpret_cast<float *>(blob + p.off_scale)[t] = c.scale;
    }

    // ---- codes of the lane's run at the chosen width
    uint32_t codes[8], values[16];
    signed_values<DT>(mg, lrow, owns ? tid : 0u, values);
    switch (c.width) {
        case 2: pack_codes<2>(m, values, codes); break;
        case 3: pack_codes<3>(m, values, codes); break;
        case 4: pack_codes<4>(m, values, codes); break;
        case 5: pack_codes<5>(m, values, codes); break;
        case 6: pack_codes<6>(m, values, codes); break;
        case 7: pack_codes<7>(m, values, codes); break;
        default: pack_codes<8>(m, values, codes); break;
    }
    // ---- ... into the wave's part of their place in LDS.  Before anybody looks for the tokens before: a look that comes
    //      too early costs a memory round trip (codes put there behind the wait, over the row: 512 x 5120 step 14.5 us
    //      against 12.6, 128 x 768 f16 6.7 / 5.9)
    if (owns) {
        uint32_t *dst = image + wv * (64u * 8u) + lane * c.width;
        const uint32_t nd = (FULL || left >= 4) ? c.width : ((left * c.width + 3u) >> 2);
        switch (c.width) {
            case 2: put_codes<2, FULL>(dst, codes, nd); break;
            case 3: put_codes<3, FULL>(dst, codes, nd); break;
            case 4: put_codes<4, FULL>(dst, codes, nd); break;
            case 5: put_codes<5, FULL>(dst, codes, nd); break;
            case 6: put_codes<6, FULL>(dst, codes, nd); break;
            case 7: put_codes<7, FULL>(dst, codes, nd); break;
            default: put_codes<8, FULL>(dst, codes, nd); break;
        }
    }
    uint32_t ew = 0, ec = 0, bad = 0, spins = 0;

    // ---- what lies before the token, 256 words at a time, the lowest first: by the time the next ones are asked for
    //      they have been published, too.  (512 words at a time: 700 x 8192 11.3 us against 9.7;
    //      2048 x 4096 f16, as it was with a token per workgroup, 13.3 / 12.1; 128: 14.6 / 12.1; all 2048 at once 18.7)
    constexpr uint32_t kReaders = NW < 4 ? NW : 4, kAhead = 4 / kReaders;
    const uint32_t t0 = t & ~(kDirectBlock - 1u);
    const uint32_t none = tag << 30;                              // a word that counts nothing
    uint64_t base = (uint64_t)none << 32;
    if (t0 && wv == 0) base = prefix_load(pre + t0 + opaque_zero());
    uint32_t w[kAhead];
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k) {
        const uint32_t j = t0 + tid + 64u * kReaders * k;
        w[k] = none;
        if (wv < kReaders && j < t) w[k] = word_load(sizes + j);
    }

    for (uint32_t j0 = t0;;) {
        for (;;) {
            bool missing = false;
#pragma unroll
            for (uint32_t k = 0; k < kAhead; ++k) missing |= (w[k] >> 30) != tag;
            if (__builtin_amdgcn_ballot_w64(missing) == 0) break;
            if (!keep_waiting(spins, p.spin_limit, error_flag)) { bad = 1; break; }
#pragma unroll
            for (uint32_t k = 0; k < kAhead; ++k)
                if ((w[k] >> 30) != tag) w[k] = word_load(sizes + j0 + tid + 64u * kReaders * k);
        }
#pragma unroll
        for (uint32_t k = 0; k < kAhead; ++k) {
            ew += token_words(p, (w[k] >> 26) & 15u);
            ec += w[k] & 0xFFFFu;
        }
        j0 += 64u * kReaders * kAhead;
        if (bad || j0 >= t) break;
#pragma unroll
        for (uint32_t k = 0; k < kAhead; ++k) {
            const uint32_t j = j0 + tid + 64u * kReaders * k;
            w[k] = none;
            if (wv < kReaders && j < t) w[k] = word_load(sizes + j);
        }
    }
    if (wv == 0) {
        while ((uint32_t)(base >> 62) != tag && !bad) {
            if (!keep_waiting(spins, p.spin_limit, error_flag)) bad = 1;
            else base = prefix_load(pre + t0 + opaque_zero());
        }
        if (lane == 0) {
            ew += (uint32_t)(base >> 32) & 0x3FFFFFFFu;
            ec += (uint32_t)base;
        }
    }
    if (NW > 1) {
        // (the third value travels in the waves' own words of the area)
        uint32_t *also = reduce_area(ring, turn) + kMaxWaves;
        if (lane == 0) also[wv] = bad;
        block_sum2_nw<NW>(ew, ec, ring, turn);
        bad = 0;
#pragma unroll
        for (int k = 0; k < NW; ++k) bad |= also[k];
        bad = uniform(bad);
    } else {
        block_sum2_nw<NW>(ew, ec, ring, turn);
    }

    const uint32_t words = token_words(p, c.width);
    const uint32_t payload_words = (uint32_t)(p.payload_capacity >> 2), outlier_capacity = (uint32_t)p.outlier_capacity;
    if ((uint64_t)ew + words > (uint64_t)payload_words) bad = 1;     // never leaves the section, whatever the tables said
    if (bad) {
        if (lane == 0) {
            raise_error(error_flag);
            store_status(blob, kStatusInternal);
        }
    } else {
        if (tid == 0) {
            if (((t + 1u) & (kDirectBlock - 1u)) == 0) prefix_store(pre + t + 1u, prefix_word(tag, ew + words, ec + st.cnt));
            reinterpret_cast<uint64_t *>(blob + p.off_pay_off)[t] = (uint64_t)ew << 2;
            reinterpret_cast<uint64_t *>(blob + p.off_row_ptr)[t] = ec;
        }

        // ---- T_above of the lane's run, in column order
        if (nl && (uint64_t)ec + st.cnt <= (uint64_t)outlier_capacity) {
            uint32_t pos = ec + st.cnt_before + upto - nl;
            uint16_t *col = reinterpret_cast<uint16_t *>(blob + p.off_out_col), *val = reinterpret_cast<uint16_t *>(blob + p.off_out_val);
            for (uint32_t rest = omask; rest; rest &= rest - 1u) {
                const uint32_t j = (uint32_t)__builtin_ctz(rest);
                col[pos] = (uint16_t)(tid * kRun + j);
                val[pos] = raw_element_sw(lrow, tid, j);
                ++pos;
            }
        }
        // ---- the codes to their place in the blob, 16 bytes per lane and step
        {
            const uint32_t first = 64u * wv * c.width;                    // the wave's first word of the row
            const uint32_t n = words > first ? (words - first < 64u * c.width ? words - first : 64u * c.width) : 0u;
            const uint32_t *img = image + wv * (64u * 8u);
            uint8_t *dst = blob + p.off_payload + 4ull * (ew + first);
            const uint32_t quads = n >> 2, rest = n & 3u;
            const __amdgpu_buffer_rsrc_t window = raw_window(dst, n << 2);
#pragma unroll
            for (uint32_t k = 0; k < 2; ++k) {
                const uint32_t i = lane + 64u * k;
                if (i < quads) store_quad_through(window, 16u * i, *reinterpret_cast<const u32x4 *>(img + 4u * i));
            }
            if (lane < rest) *reinterpret_cast<uint32_t *>(dst + 4u * (4u * quads + lane)) = img[4u * quads + lane];
        }
    }
    if (last && wv == 0) close_blob(p, blob, tickets, error_flag, epoch, bad, ew + words, (uint64_t)ec + st.cnt, raised);
}

// ---------------------------------------------------------------- eight short rows a workgroup

// Rows of one wave, calls of many tokens: a workgroup of eight waves takes eight consecutive tokens, one a wave, and places
// them together: one word per eight tokens is published (tag | payload words << 16 | outliers), looked for and added
// up, by all of the workgroup's waves, and the waves' own sums go through LDS.  With a workgroup per token thousands of waves
// at a time look for every word there is, and those looks hold up the stores that they wait for: 360 tokens per us, whatever
// the length of the rows.  131072 x 768 f16 352 us, now 156; 131072 x 2048 bf16 430 / 226; 65536 x 1024 f16 193 / 89;
// 10^6 x 8 f16 2823 / 1415; 4000 x 768 f16 15.0 / 9.9.  What bounds it now is the workgroup's life, from the row's arrival to
// the last store, and how many of them fit the device (24 to 32 waves a compute unit, none of which fetches ahead).
// Rows of two waves: two tokens a workgroup, which halves the polling and, more, the number of workgroups that live at once:
// 2000 x 4096 f16 12.0 us with a token per workgroup against 10.5; 3000 x 4096 15.6 / 12.8; 4000 x 4096 21.5 / 16.8; 3000 x
// 2304 bf16 16.0 / 13.4.  Four tokens a workgroup were slower than two, and rows of three and four waves gained nothing.
constexpr uint32_t group_tokens(uint32_t nw) { return nw == 1u ? 8u : 2u; }
constexpr uint32_t kGroupWaves = 8;                         // at most
static_assert(kGroupWaves * 512u < (1u << 14) && kGroupWaves * 2048u < (1u << 16), "fields of a group's word");
constexpr uint32_t kGroupExchange = 6u * kGroupWaves;       // dwords: three values per wave, twice
constexpr uint32_t kGroupRing = 4u * 2u * kMaxWaves;        // four reduce areas: two words per token; one word per wave

__device__ __forceinline__ void clear_group_area(uint32_t *ring, uint32_t turn) {
    if (threadIdx.x < 8u) reduce_area(ring, turn)[threadIdx.x] = 0;
}

// Algorithm 1 for the tokens of a workgroup, NW waves each (this wave's is number g of G), as search_width does it for one.
// The tokens go through the candidates together, since a barrier is the whole workgroup's: whoever is done waits there for
// the others; lane k of every wave makes the test of token k, so that all waves know who goes on.  present: bit k: there is
// a token k.
template <int DT, int NW, int G>
__device__ __forceinline__ Choice search_widths(const Params &p, const Mags<DT> &af, float amax, bool live, uint32_t g,
                                                uint32_t present, uint32_t *ring, uint32_t &turn, uint32_t (&m)[8]) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t quot_bits = __float_as_uint(quotients_of(p, amax));
    const uint32_t b0 = width_at(p, 0);
    const uint32_t Q0 = (1u << (b0 - 1)) - 1u;
    quantize_run<DT>(af, __uint_as_float(lane_value(quot_bits, 0)), m);
    uint32_t sel = b0, sel_i = 0;
    if (p.n_widths > 1) {
        uint32_t m0[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) m0[k] = m[k];
        double ss0d = 0.0;                                   // lane k: token k's
        uint32_t active = present;
        for (uint32_t i = 1; i < p.n_widths && active; ++i) {
            const uint32_t bi = width_at(p, i);
            const bool mine = (active >> g) & 1u;
            uint32_t *red = reduce_area(ring, turn);
            uint32_t mi[8];
            if (mine) {
                quantize_run<DT>(af, __uint_as_float(lane_value(quot_bits, (int)i)), mi);
                const uint32_t sad = row_sum_u32(live ? sad_run(m0, mi, b0 - bi) : kSadNone);
                if (i == 1) {
                    const uint32_t ss0 = row_sum_u32(live ? sum_squares_run(m0) : 0u);
                    if (first_of_row())
                        __hip_atomic_fetch_add(reinterpret_cast<uint64_t *>(red) + g + some_zero(), (uint64_t)ss0 << 32 | sad,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                } else if (first_of_row()) {
                    __hip_atomic_fetch_add(red + 2u * g + some_zero(), sad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            lds_barrier();
            const uint2 v = *reinterpret_cast<const uint2 *>(red + 2u * (lane & (G - 1)));
            clear_group_area(ring, turn + 2u);
            ++turn;
            if (i == 1) ss0d = (double)v.y;
            const bool over = violates(p.mode, p.test_rhs[i], Q0, 64u * NW * kSadNone - v.x, ss0d);
            const uint32_t fails = (uint32_t)__builtin_amdgcn_ballot_w64(over) & active;
            if (mine && (!((fails >> g) & 1u) || p.return_failing)) {
                sel = bi;
                sel_i = i;
#pragma unroll
                for (int k = 0; k < 8; ++k) m[k] = mi[k];
            }
            active &= ~fails;
        }
    }
    Choice c;
    c.width = sel;
    c.scale = __uint_as_float(lane_value(quot_bits, (int)(8u + sel_i)));
    return c;
}

// LDS map (dynamic): per token: row: runs*16 dwords, codes: runs*8 | exchange | ring (rows of more than one wave)
template <int DT, int NW, bool FULL>
__global__ void __launch_bounds__(64 * NW * group_tokens(NW), DT == kF16 ? 8 : 6)
k_direct_group(const Params p, const uint16_t *__restrict__ in, uint8_t *__restrict__ blob, uint8_t *__restrict__ ws) {
    extern __shared__ __align__(16) uint32_t lds[];
    constexpr uint32_t G = group_tokens(NW), W = NW * G;     // tokens and waves of the workgroup
    const uint32_t u = blockIdx.x, tid = threadIdx.x, lane = tid & 63u, wv = uniform(tid >> 6);
    const uint32_t g = wv / NW, part = wv % NW;              // the wave's token in the group, and its part of it
    const uint32_t t = u * G + g;
    const bool have = t < p.tokens, last = u == gridDim.x - 1u;
    const uint32_t runs = FULL ? 64u * NW : p.runs, pieces = FULL ? 256u * NW : p.pieces;
    const uint32_t run = 64u * part + lane;
    const bool owns = FULL || run < runs;
    const uint32_t left = FULL ? 4u : (owns ? pieces - 4u * run : 0u);    // 16-byte pieces of the lane's run inside the row
    uint32_t *lrow = lds + g * runs * 24u, *image = lrow + runs * 16u, *exchange = lds + G * runs * 24u, *ring = exchange + kGroupExchange;

    // (a token that is not there: the last one's row, whose results are dropped)
    RowPart piece;
    const uint32_t q0 = 256u * part + lane;
    fetch_row_once<FULL>(row_address(p, in, have ? t : p.tokens - 1u, FULL ? 2048u * NW : p.hidden), pieces, q0, piece);
    // error word, shape and epoch of the workspace, one per lane of one load
    uint32_t *ctrl = reinterpret_cast<uint32_t *>(ws + p.ws_ctrl);
    uint32_t *tickets = reinterpret_cast<uint32_t *>(ws + p.ws_tickets);
    uint32_t *error_flag = ctrl + kCtlError;
    const uint32_t *looked = lane == 0 ? error_flag : lane == 1 ? ctrl + kCtlTokens : lane == 2 ? ctrl + kCtlHidden : tickets + kCntTickets;
    const uint32_t state = __hip_atomic_load(looked, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (NW > 1) {
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) clear_group_area(ring, k);
        lds_barrier();
    }

#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        const uint32_t q = q0 + 64u * k, r = q >> 2, c = (q & 3u) ^ ((r >> 1) & 3u);
        if (FULL || r < runs)
            *reinterpret_cast<uint4 *>(lrow + r * 16u + c * 4u) =
                make_uint4(piece.w[4 * k], piece.w[4 * k + 1], piece.w[4 * k + 2], piece.w[4 * k + 3]);
    }
    Mags<DT> mg;
    uint32_t omask = 0, amax_bits = 0, turn = 0;
    {
        uint32_t w[16];
        load_run_sw(lrow, owns ? run : 64u * part, w);
        split_regs<DT, true>(w, p.thr_pk, mg, omask, amax_bits);
    }
    if (!owns || !have) { omask = 0; amax_bits = 0; }

    // (a workspace that must not be used: the waves decide together, as in k_direct)
    const bool shape_ok = workspace_shape_ok(lane_value(state, 1), lane_value(state, 2), p.tokens, p.hidden);
    const uint32_t refused = (lane_value(state, 0) ? kSawError : 0u) + (shape_ok ? 0u : kSawShape);
    const uint32_t epoch = (lane_value(state, 3) >> kTicketBits) % 3u, tag = epoch + 1u;
    if (last && tid == 0) store_status(blob, 0u);

    const uint32_t nl = (uint32_t)__builtin_popcount(omask);
    const uint32_t upto = wave_incl_scan_u32(nl);                 // outliers of the wave's lanes up to this one
    const uint32_t cnt = lane_value(upto, 63);                    // ... of the wave
    uint32_t m[8];
    Choice c;
    if constexpr (NW == 1) {
        const RowStats st = reduce_row_stats_counted<1>(amax_bits, cnt, nullptr, turn);
        c = search_width<DT, 1>(p, mg, st.amax, owns, nullptr, turn, m);
    } else {
        uint32_t *red = reduce_area(ring, turn);
        const uint32_t mx = row_max_u32(amax_bits);
        if (first_of_row()) __hip_atomic_fetch_max(red + 2u * g + some_zero(), mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        lds_barrier();
        const float amax = __uint_as_float(uniform(red[2u * g]));
        clear_group_area(ring, turn + 2u);
        ++turn;
        const uint32_t there = p.tokens - u * G < G ? (1u << (p.tokens - u * G)) - 1u : (1u << G) - 1u;
        c = search_widths<DT, NW, G>(p, mg, amax, owns, g, there, ring, turn, m);
    }
    const uint32_t words = have ? token_words(p, c.width) : 0u;   // of the token

    uint32_t *sizes = reinterpret_cast<uint32_t *>(ws + p.ws_sizes);
    uint64_t *pre = reinterpret_cast<uint64_t *>(ws + p.ws_prefix);
    // (the last workgroup looks for failures now, with the status word's zero in place: see k_direct)
    uint32_t raised = 0;
    if (last && wv == 0) {
        memory_operations_performed();
        raised = word_load(error_flag + opaque_zero());
    }
    if (lane == 0) { exchange[wv] = part == 0 ? words : 0u; exchange[W + wv] = cnt; exchange[2u * W + wv] = refused; }
    lds_barrier();
    // lane w has what wave w left; its own wave's share, and that of the workgroup
    const uint32_t gw = lane < W ? exchange[lane] : 0u, gc = lane < W ? exchange[W + lane] : 0u;
    const uint32_t gr = lane < W ? exchange[2u * W + lane] : 0u;
    if (__builtin_amdgcn_ballot_w64(gr != 0) != 0) {
        if (last && tid == 0) write_header(p, blob, 0, 0, __builtin_amdgcn_ballot_w64(gr >= kSawShape) != 0 ? kStatusFormat : kStatusInternal);
        return;
    }
    const uint32_t upto_w = wave_incl_scan_u32(gw), upto_c = wave_incl_scan_u32(gc);
    const uint32_t group_words = lane_value(upto_w, 63), group_outliers = lane_value(upto_c, 63);
    const uint32_t words_before = lane_value(upto_w - gw, (int)(wv - part));                // before the token
    const uint32_t token_first = lane_value(upto_c - gc, (int)(wv - part));                 // outliers before the token
    const uint32_t token_outliers = lane_value(upto_c, (int)(wv - part + NW - 1u)) - token_first;
    const uint32_t outliers_before = lane_value(upto_c - gc, (int)wv);                      // before the wave's part
    if (tid == 0) word_store(sizes + u, (tag << 30) | (group_words << 16) | group_outliers);
    if (lane == 0 && part == 0 && have) {
        blob[p.off_bits + t] = (uint8_t)c.width;
        reinterpret_cast<float *>(blob + p.off_scale)[t] = c.scale;
    }

    // ---- codes of the lane's run at the chosen width, into their place in LDS
    if (owns && have) {
        uint32_t values[16];
        signed_values<DT>(mg, lrow, run, values);
        uint32_t *dst = image + part * (64u * 8u) + lane * c.width;
        const uint32_t nd = (FULL || left >= 4) ? c.width : ((left * c.width + 3u) >> 2);
        switch (c.width) {
            case 2: pack_to_image<2, FULL>(m, values, dst, nd); break;
            case 3: pack_to_image<3, FULL>(m, values, dst, nd); break;
            case 4: pack_to_image<4, FULL>(m, values, dst, nd); break;
            case 5: pack_to_image<5, FULL>(m, values, dst, nd); break;
            case 6: pack_to_image<6, FULL>(m, values, dst, nd); break;
            case 7: pack_to_image<7, FULL>(m, values, dst, nd); break;
            default: pack_to_image<8, FULL>(m, values, dst, nd); break;
        }
    }

    // ---- what lies before the group, a word per thread at a time, the lowest first
    uint32_t ew = 0, ec = 0, bad = 0, spins = 0;
    const uint32_t u0 = u & ~(kDirectBlock - 1u), none = tag << 30;
    uint64_t base = (uint64_t)none << 32;
    if (u0 && wv == 0) base = prefix_load(pre + u0 + opaque_zero());
    for (uint32_t j0 = u0; j0 < u && !bad; j0 += 64u * W) {
        const uint32_t j = j0 + tid;
        uint32_t w = j < u ? word_load(sizes + j) : none;
        while (__builtin_amdgcn_ballot_w64((w >> 30) != tag) != 0) {
            if (!keep_waiting(spins, p.spin_limit, error_flag)) { bad = 1; break; }
            if ((w >> 30) != tag) w = word_load(sizes + j);
        }
        ew += (w >> 16) & 0x3FFFu;
        ec += w & 0xFFFFu;
    }
    if (wv == 0) {
        while ((uint32_t)(base >> 62) != tag && !bad) {
            if (!keep_waiting(spins, p.spin_limit, error_flag)) bad = 1;
            else base = prefix_load(pre + u0 + opaque_zero());
        }
        if (lane == 0) {
            ew += (uint32_t)(base >> 32) & 0x3FFFFFFFu;
            ec += (uint32_t)base;
        }
    }
    ew = wave_sum_u32(ew);
    ec = wave_sum_u32(ec);
    uint32_t *sums = exchange + 3u * W;
    if (lane == 0) { sums[wv] = ew; sums[W + wv] = ec; sums[2u * W + wv] = bad; }
    lds_barrier();
    ew = wave_sum_u32(lane < W ? sums[lane] : 0u);
    ec = wave_sum_u32(lane < W ? sums[W + lane] : 0u);
    bad = __builtin_amdgcn_ballot_w64(lane < W && sums[2u * W + lane] != 0) != 0 ? 1u : 0u;

    const uint32_t payload_words = (uint32_t)(p.payload_capacity >> 2), outlier_capacity = (uint32_t)p.outlier_capacity;
    if ((uint64_t)ew + group_words > (uint64_t)payload_words) bad = 1;     // never leaves the section, whatever the tables said
    if (bad) {
        if (lane == 0) {
            raise_error(error_flag);
            store_status(blob, kStatusInternal);
        }
    } else {
        if (tid == 0 && ((u + 1u) & (kDirectBlock - 1u)) == 0)
            prefix_store(pre + u + 1u, prefix_word(tag, ew + group_words, ec + group_outliers));
        const uint32_t my_word = ew + words_before;
        if (have && lane == 0 && part == 0) {
            reinterpret_cast<uint64_t *>(blob + p.off_pay_off)[t] = (uint64_t)my_word << 2;
            reinterpret_cast<uint64_t *>(blob + p.off_row_ptr)[t] = ec + token_first;
        }
        // ---- T_above of the lane's run, in column order
        if (nl && (uint64_t)(ec + token_first) + token_outliers <= (uint64_t)outlier_capacity) {
            uint32_t pos = ec + outliers_before + upto - nl;
            uint16_t *col = reinterpret_cast<uint16_t *>(blob + p.off_out_col), *val = reinterpret_cast<uint16_t *>(blob + p.off_out_val);
            for (uint32_t rest = omask; rest; rest &= rest - 1u) {
                const uint32_t j = (uint32_t)__builtin_ctz(rest);
                col[pos] = (uint16_t)(run * kRun + j);
                val[pos] = raw_element_sw(lrow, run, j);
                ++pos;
            }
        }
        // ---- the codes to their place in the blob, 16 bytes per lane and step
        {
            const uint32_t first = 64u * part * c.width;                  // the wave's first word of the row
            const uint32_t n = words > first ? (words - first < 64u * c.width ? words - first : 64u * c.width) : 0u;
            const uint32_t *img = image + part * (64u * 8u);
            uint8_t *dst = blob + p.off_payload + 4ull * (my_word + first);
            const uint32_t quads = n >> 2, rest = n & 3u;
            const __amdgpu_buffer_rsrc_t window = raw_window(dst, n << 2);
#pragma unroll
            for (uint32_t k = 0; k < 2; ++k) {
                const uint32_t i = lane + 64u * k;
                if (i < quads) store_quad_through(window, 16u * i, *reinterpret_cast<const u32x4 *>(img + 4u * i));
            }
            if (lane < rest) *reinterpret_cast<uint32_t *>(dst + 4u * (4u * quads + lane)) = img[4u * quads + lane];
        }
    }
    if (last && wv == 0) close_blob(p, blob, tickets, error_flag, epoch, bad, ew + group_words, (uint64_t)ec + group_outliers, raised);
}

// ---------------------------------------------------------------- launcher

typedef void (*DirectKernel)(const Params, const uint16_t *, uint8_t *, uint8_t *);

template <int DT, bool FULL>
static DirectKernel direct_kernel_for(uint32_t nw) {
    switch (nw) {
        case 1: return k_direct<DT, 1, FULL>;
        case 2: return k_direct<DT, 2, FULL>;
        case 3: return k_direct<DT, 3, FULL>;
        case 4: return k_direct<DT, 4, FULL>;
        case 8: return k_direct<DT, 8, FULL>;
        default: return k_direct<DT, 16, FULL>;
    }
}
static DirectKernel direct_kernel(uint32_t dtype, uint32_t nw, bool full) {
    if (dtype == (uint32_t)kF16) return full ? direct_kernel_for<kF16, true>(nw) : direct_kernel_for<kF16, false>(nw);
    return full ? direct_kernel_for<kBF16, true>(nw) : direct_kernel_for<kBF16, false>(nw);
}

template <int DT, bool FULL>
static DirectKernel group_kernel_for(uint32_t nw) {
    switch (nw) {
        case 1: return k_direct_group<DT, 1, FULL>;
        default: return k_direct_group<DT, 2, FULL>;
    }
}
static DirectKernel group_kernel(uint32_t dtype, uint32_t nw, bool full) {
    if (dtype == (uint32_t)kF16) return full ? group_kernel_for<kF16, true>(nw) : group_kernel_for<kF16, false>(nw);
    return full ? group_kernel_for<kBF16, true>(nw) : group_kernel_for<kBF16, false>(nw);
}

static uint32_t direct_lds_bytes(uint32_t runs) { return (runs * 24u + (runs > 64u ? kDirectRing : 0u)) * 4u; }

int prepare_direct_kernels() {
    const int big = (int)direct_lds_bytes(kMaxHidden / kRun);
    static const uint32_t sizes[] = {1, 2, 3, 4, 8, 16};
    for (uint32_t dt = 0; dt < 2; ++dt)
        for (uint32_t nw : sizes)
            for (int full = 0; full < 2; ++full) {
                const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(direct_kernel(dt, nw, full != 0)),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, big);
                if (e != hipSuccess) return (int)e;
            }
    return 0;
}

// Rows of one wave: eight tokens a workgroup from this number of tokens on.  Fewer do not fill the device with workgroups of
// eight: 500 x 768 f16 6.0 us with a token per workgroup against 6.5, 1000 x 2048 bf16 7.9 / 7.7, 2000 x 768 9.3 / 6.8.
// Rows of two waves, two tokens: 700 x 4096 f16 8.7 / 8.6, 1024 x 4096 8.5 / 8.0, 1100 x 4096 bf16 9.8 / 8.9, and with six
// widths and the LSB criterion 1237 x 4096 bf16 10.2 / 10.0, 3000 x 4096 14.8 / 14.3.
// Rows that do not fill their two waves gain nothing while pairs give a compute unit more tokens than it had (256 compute
// units: 6 against 5 up to 1280 tokens): 1024 x 2304 bf16, LSB, six widths 9.1 / 9.7, 1237 x 2856 10.3 / 10.6; a fifth of the
// elements outliers 1280 x 2856 f16 11.2 / 12.1.  Beyond: 1350 x 2856 bf16, LSB 10.2 / 9.4, 1500 x 3400 f16 10.4 / 9.6,
// 3000 x 2856 15.2 / 13.7; slower only now and then: bf16, LSB, six widths 3000 x 3400 14.7 / 15.4 (2000 x 3400 12.9 / 12.8),
// and a fifth of the elements outliers 2000 x 2856 f16 14.0 / 15.1 (3000 x 2856 20.9 / 19.0).
// A launch counts its threads in 32 bits, those of a last group's missing tokens included: the seven token counts of rows of
// one wave (2^26 - 7 .. 2^26 - 1) whose groups would be 2^32 threads take a workgroup per token, which is 64 a token.
constexpr uint32_t kGroupFrom = 1024, kRaggedPairsFrom = 5u * 256u + 1u;
uint32_t direct_group_log2(const Params &p, const Geometry &g) {
    const bool ragged_pairs = g.waves == 2 && p.hidden != 4096u;
    if (g.waves > 2 || p.tokens < (ragged_pairs ? kRaggedPairsFrom : kGroupFrom)) return 0u;
    const uint32_t log2 = g.waves == 1 ? 3u : 1u;
    const uint64_t groups = ((uint64_t)p.tokens + (1u << log2) - 1u) >> log2;
    return (groups * 64u * g.waves) << log2 < (1ull << 32) ? log2 : 0u;
}
DirectLaunch direct_launch(const Params &p, const Geometry &g) {
    const uint32_t log2 = direct_group_log2(p, g), G = 1u << log2;
    if (log2 == 0) return {1u, p.tokens, 64u * g.waves, direct_lds_bytes(p.runs)};
    return {G, (p.tokens + G - 1u) >> log2, 64u * g.waves * G,
            (G * p.runs * 24u + kGroupExchange + (g.waves > 1 ? kGroupRing : 0u)) * 4u};
}
int launch_direct(const Params &p, const Geometry &g, const void *d_in, void *d_blob, void *d_ws, void *stream) {
    const bool full = p.hidden == 2048u * g.waves;
    const DirectLaunch l = direct_launch(p, g);
    const DirectKernel kernel = l.tokens > 1 ? group_kernel(p.dtype, g.waves, full) : direct_kernel(p.dtype, g.waves, full);
    hipLaunchKernelGGL(kernel, dim3(l.workgroups), dim3(l.threads), l.lds_bytes, reinterpret_cast<hipStream_t>(stream), p,
                       static_cast<const uint16_t *>(d_in), static_cast<uint8_t *>(d_blob), static_cast<uint8_t *>(d_ws));
    return (int)hipGetLastError();
}

}  // namespace tsq
