// tkv_quantize_append: quantise newly written bf16 K/V at a per-token width
// (INT2 / INT4) and pack codes, fp16 scales and fp16 zero-points into the
// paged pool (paper Sec. 3.2.1 for the quantisation scheme, Sec. 3.2.2-3.2.3
// for the two pools and the per-token bitwidth array).
//
// Two workgroups of 256 threads per (destination page, kv head) record, one for its K planes and one for its V planes.
// Thread (slot = tid/4, group = tid%4) quantises one group of 32 channels of the token bound for that slot; a group
// is 64 contiguous bytes of the input, so min/max need no cross-lane step.
//
// What bounds it: HBM for whole pages (512 B read and 96 / 160 B written per token and head), the chain of dependent
// loads (arguments -> slots -> rows -> result) for a few tokens.  Hence
//  - the rows go straight to LDS, whole 128-byte lines per instruction, without a register, and all that can be asked
//    for at once is: the slots, then tags, rows and the V words that may have to be merged;
//  - K and V apart: a workgroup holds 16 KiB of LDS and eight are resident per compute unit, each in a phase of its
//    own.  65 536 tokens x 8 heads, inputs not in any cache: 67.2 us with both in one workgroup and 64-byte runs per thread
//    through registers, 63.1 with rows through LDS (32 KiB, five resident), 59.1 apart (with ordinary stores 60.7);
//    per-channel keys 69.4 -> 60.1; one token for each of 32 sequences 6.0 -> 4.4.  What one wait per level of the chain of
//    loads adds to that stands where it is made (tkv_append_kernel).  The launcher says which loads and
//    which order of the workgroups are taken.
//
// K words go straight to HBM (a wavefront's stores for one word index are 256 contiguous bytes, written with
// non-temporal stores).  V codes are transposed through LDS, because the V plane packs tokens, not channels, into a
// word; for a page that arrives whole, the V words and the two V metadata planes, which are adjacent in the record,
// are put together in LDS and leave in 16-byte non-temporal stores, one KiB per instruction of a wavefront.
//
// Arithmetic is IEEE binary32 without fused multiply-add so that the codes,
// scales and zero-points match a scalar CPU evaluation bit for bit:
//   zero = fp16(min), scale = fp16((max - min) / (2^b - 1)),
//   code = clamp(rint((x - zero) * (1 / scale)), 0, 2^b - 1), 0 if scale == 0.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <type_traits>

#include "tkv_internal.h"
#include "tkv_layout.h"

#pragma clang fp contract(off)

namespace {

using namespace tkv;

struct GroupQ {
    uint32_t words[4];   // packed codes: INT4 uses 4 words (8 channels each), INT2 2 words (16 each)
    uint32_t bytes[8];   // the same 32 codes, one per byte (for the V transpose)
    uint16_t scale, zero;
};

// One quantisation group of 32 values: the channels of a group of one token, or (per-channel keys) the 32
// tokens of a block for one channel.
template <int BITS>
__device__ __forceinline__ GroupQ quantize_values(const float (&f)[32])
{
    constexpr int L = (1 << BITS) - 1;
    // Inputs are finite, so min / max instructions give the value a chain of comparisons gives; only the sign
    // of a zero can differ.  A zero minimum is stored as +0 anyway; a zero maximum takes the sign the scalar
    // definition gives it (the first element that is not below its predecessors' maximum), settled below.
    float mn = f[0], mx = f[0];
#pragma unroll
    for (int i = 1; i < 32; ++i) {
        mn = fminf(mn, f[i]);
        mx = fmaxf(mx, f[i]);
    }
    if (mn == 0.0f) mn = 0.0f;   // -0 -> +0
    if (__builtin_expect(mx == 0.0f, 0)) {
        mx = f[0];
#pragma unroll
        for (int i = 1; i < 32; ++i) mx = f[i] > mx ? f[i] : mx;
    }
    const float r = __fsub_rn(mx, mn);
    const float s32 = __fdiv_rn(r, (float)L);
    const __half sh = __float2half_rn(s32), zh = __float2half_rn(mn);
    const float s = __half2float(sh), z = __half2float(zh);
    GroupQ out;
    out.scale = __half_as_ushort(sh);
    out.zero = __half_as_ushort(zh);
    const float inv = s == 0.0f ? 0.0f : __fdiv_rn(1.0f, s);   // a zero scale gives t = 0 and code 0 for every element
    // clamp, then round by adding 1.5 * 2^23: the sum is rounded to an integer (nearest, ties to even, the
    // same result as rounding first and clamping after) and its bit pattern is kBias + code
    constexpr float kMagic = 12582912.0f;
    constexpr uint32_t kBias = 0x4b400000u;
    uint32_t c[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const float t = __builtin_amdgcn_fmed3f(__fmul_rn(__fsub_rn(f[i], z), inv), 0.0f, (float)L);
        c[i] = __float_as_uint(__fadd_rn(t, kMagic));
    }
    // packed by shift-and-add; what the biases add up to (modulo 2^32) is one constant per word
    constexpr int per_word = 32 / BITS;
    uint32_t bias_word = 0, bias_byte = 0;
#pragma unroll
    for (int i = 0; i < per_word; ++i) bias_word += kBias << (BITS * i);
#pragma unroll
    for (int k = 0; k < 4; ++k) bias_byte += kBias << (8 * k);
#pragma unroll
    for (int w = 0; w < 4; ++w) out.words[w] = 0u - bias_word;
#pragma unroll
    for (int i = 0; i < 32; ++i) out.words[i / per_word] += c[i] << (BITS * (i % per_word));
#pragma unroll
    for (int w = 0; w < 8; ++w)
        out.bytes[w] = c[4 * w] + (c[4 * w + 1] << 8) + (c[4 * w + 2] << 16) + (c[4 * w + 3] << 24) - bias_byte;
    return out;
}

constexpr int kRowBytes = kHeadDim * 2, kRowPieces = kRowBytes / 16;   // a row: one token of one kv head, of K or of V
// The rows are fetched by the wavefront that uses them (wavefront w: slots 16 w .. 16 w + 15), straight into LDS: one
// instruction moves four rows, sixteen lanes to a row, 1 KiB that is contiguous in LDS.  A thread then reads four
// consecutive 16-byte pieces of its row; piece p of row r sits at place p ^ (r & 3), so that the lanes of neighbouring
// rows read from different banks.
template <bool ONCE> __device__ __forceinline__ void fetch_row_pieces(uint4 *lds_wave, int i, const uint16_t *__restrict__ row, int lane)
{
    const uint4 *src = reinterpret_cast<const uint4 *>(row) + ((lane & 15) ^ (lane >> 4));
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)(lds_wave + 64 * i), 16, 0, ONCE ? 2 : 0 /* nt */);
}
__device__ __forceinline__ int piece_at(int slot, int p) { return slot * kRowPieces + (p ^ (slot & 3)); }

template <int BITS>
__device__ __forceinline__ GroupQ quantize_group(const uint4 *rows, int slot, int g)
{
    float f[32];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint4 v = rows[piece_at(slot, 4 * g + i)];
        const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            f[8 * i + 2 * k] = __uint_as_float(u[k] << 16);
            f[8 * i + 2 * k + 1] = __uint_as_float(u[k] & 0xffff0000u);
        }
    }
    return quantize_values<BITS>(f);
}

// V codes of the page, one per byte: row of slot s, where the K rows of the same wavefront were.  144-byte rows: the four
// quads that one instruction of the transpose reads lie four rows apart and must not meet on the same banks.
__device__ __forceinline__ int code_row(int slot) { return (slot >> 4) * 16 * kRowBytes + (slot & 15) * 144; }
// 16-byte piece c of the V words and V metadata planes of a whole page, on their way out: the 112 pieces behind the
// code rows in each wavefront's part of the row area.
__device__ __forceinline__ int out_piece(int c)
{
    const int part = (c >= 112 ? 1 : 0) + (c >= 224 ? 1 : 0);
    return part * 16 * kRowPieces + 144 + (c - 112 * part);
}
static_assert((Rec<4>::kCodeBytes + 2 * kMetaBytes) / 16 <= 3 * 112, "the pieces of an INT4 page fit behind the code rows of three wavefronts");
// Token (slot) of code position p in a V word of (block of 32 tokens, quad); INT2 words hold both blocks.
template <int BITS> __device__ __forceinline__ constexpr int v_token(int blk, int quad, int p)
{
    const int j = BITS == 4 ? 2 * (p & 3) + (p >> 2) : 2 * (p & 3) + (p >> 3);
    return 32 * (BITS == 4 ? blk : (p & 7) >> 2) + 16 * (j >> 2) + 4 * quad + (j & 3);
}

// The K planes of a record.  `mask`: the slots that receive a token, the same in all four wavefronts.
// KC: keys per channel over each block of 32 slots (INT2 pages only); the mask then holds whole blocks.
template <int BITS, bool KC>
__device__ __forceinline__ void append_k(uint8_t *rec, uint64_t mask, uint4 *rows)
{
    using R = Rec<BITS>;
    const int tid = threadIdx.x, slot = tid >> 2, g = tid & 3;
    const int tile = slot >> 4, row = slot & 15;
    const bool valid = (mask >> slot) & 1;
    uint32_t *kc = reinterpret_cast<uint32_t *>(rec + R::kKCodes);
    constexpr int words = BITS;   // 32-bit words of codes per group: 4 (INT4) or 2 (INT2)
    if constexpr (KC) {
        __syncthreads();   // every row is there
        // thread (block, channel): the block's 32 token values of one channel are one quantisation group
        const int blk = tid >> 7, c = tid & 127;
        const bool there = (mask >> (32 * blk)) & 1;
        GroupQ kq;
        if (there) {
            float f[32];
            const uint16_t *kt = reinterpret_cast<const uint16_t *>(rows);
#pragma unroll
            for (int i = 0; i < 32; ++i) f[i] = __uint_as_float((uint32_t)kt[8 * piece_at(32 * blk + i, c >> 3) + (c & 7)] << 16);
            kq = quantize_values<BITS>(f);
            const int mi = kcmeta_index(blk, c);
            reinterpret_cast<uint16_t *>(rec + R::kKScale)[mi] = kq.scale;
            reinterpret_cast<uint16_t *>(rec + R::kKZero)[mi] = kq.zero;
        }
        __syncthreads();   // every row is read; their place takes the codes, one per byte [slot][channel]
        uint8_t *kcodes = reinterpret_cast<uint8_t *>(rows);
        if (there)
#pragma unroll
            for (int i = 0; i < 32; ++i) kcodes[(32 * blk + i) * kHeadDim + c] = (uint8_t)(kq.bytes[i >> 2] >> (8 * (i & 3)));
        __syncthreads();
        // thread (slot, group) again: its token's 32 codes of the group, packed as in the per-token layout
        if (valid) {
            const uint4 *cb = reinterpret_cast<const uint4 *>(kcodes + slot * kHeadDim + g * kGroup);
            constexpr int per_word = 32 / BITS;
            uint32_t wv[4] = {0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint4 v = cb[q];
                const uint32_t b4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int i = 16 * q + 4 * j + k;   // channel of the group
                        wv[i / per_word] |= ((b4[j] >> (8 * k)) & 0xffu) << (BITS * (i % per_word));
                    }
            }
#pragma unroll
            for (int w = 0; w < words; ++w) store_once(&kc[((tile * words + w) * 16 + row) * 4 + g], wv[w]);
        }
    } else if (valid) {
        const GroupQ kq = quantize_group<BITS>(rows, slot, g);
        // these stores of a wavefront fill whole lines (256 contiguous bytes per word index, 128 per plane)
#pragma unroll
        for (int w = 0; w < words; ++w) store_once(&kc[((tile * words + w) * 16 + row) * 4 + g], kq.words[w]);
        store_once(&reinterpret_cast<uint16_t *>(rec + R::kKScale)[slot * 4 + g], kq.scale);
        store_once(&reinterpret_cast<uint16_t *>(rec + R::kKZero)[slot * 4 + g], kq.zero);
    }
}

// The V planes.  `old`: this thread's V words as they are, if the page does not arrive whole.
template <int BITS>
__device__ __forceinline__ void append_v(uint8_t *rec, uint64_t mask, const uint32_t (&old)[4], uint4 *rows)
{
    using R = Rec<BITS>;
    const int tid = threadIdx.x, slot = tid >> 2, g = tid & 3;
    const bool valid = (mask >> slot) & 1;
    uint8_t *codes = reinterpret_cast<uint8_t *>(rows);
    uint16_t v_scale = 0, v_zero = 0;
    if (valid) {
        const GroupQ vq = quantize_group<BITS>(rows, slot, g);
        v_scale = vq.scale;
        v_zero = vq.zero;
        uint4 *dst = reinterpret_cast<uint4 *>(codes + code_row(slot) + g * kGroup);
        dst[0] = make_uint4(vq.bytes[0], vq.bytes[1], vq.bytes[2], vq.bytes[3]);
        dst[1] = make_uint4(vq.bytes[4], vq.bytes[5], vq.bytes[6], vq.bytes[7]);
    }
    __syncthreads();   // all V codes are there, all V rows read
    const int mi = vmeta_index(slot, g);
    constexpr int n_words = R::kCodeBytes / 4;
    if (mask == ~0ull) {
        // Whole page: a thread transposes four adjacent channels x the (8 | 16) tokens of one word with 32-bit
        // LDS reads (a row of the byte tile holds the token's codes in channel order), merges 2 | 4 tokens per
        // byte and finishes with a 4 x 4 byte transpose; no read-modify-write.  The V words and the two V metadata
        // planes are put together behind the code rows.
        reinterpret_cast<uint16_t *>(rows + out_piece(R::kCodeBytes / 16 + (mi >> 3)))[mi & 7] = v_scale;
        reinterpret_cast<uint16_t *>(rows + out_piece((R::kCodeBytes + kMetaBytes) / 16 + (mi >> 3)))[mi & 7] = v_zero;
        constexpr int n_units = n_words / 4;   // 256 (INT4) / 128 (INT2)
        if (tid < n_units) {
            const int k = tid & 3, n4 = (tid >> 2) & 3, quad = (tid >> 4) & 3, h = (tid >> 6) & 1;
            const int blk = tid >> 7;   // INT4 only (0 for INT2)
            const int c0 = 64 * h + 16 * k + 4 * n4;
            uint32_t m[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                m[b] = 0;
#pragma unroll
                for (int e = 0; e < 8 / BITS; ++e)
                    m[b] |= *reinterpret_cast<const uint32_t *>(codes + code_row(v_token<BITS>(blk, quad, (8 / BITS) * b + e)) + c0) << (BITS * e);
            }
            // byte i of m[b] = byte b of the word of channel c0 + i
            const uint32_t t01 = __builtin_amdgcn_perm(m[1], m[0], 0x05010400u), u01 = __builtin_amdgcn_perm(m[1], m[0], 0x07030602u);
            const uint32_t t23 = __builtin_amdgcn_perm(m[3], m[2], 0x05010400u), u23 = __builtin_amdgcn_perm(m[3], m[2], 0x07030602u);
            const uint32_t wv[4] = {__builtin_amdgcn_perm(t23, t01, 0x05040100u), __builtin_amdgcn_perm(t23, t01, 0x07060302u),
                                    __builtin_amdgcn_perm(u23, u01, 0x05040100u), __builtin_amdgcn_perm(u23, u01, 0x07060302u)};
            const int first = (((BITS == 4 ? blk * 2 : 0) + h) * 4 + quad) * 16 + 4 * n4;
#pragma unroll
            for (int i = 0; i < 4; ++i) reinterpret_cast<uint32_t *>(rows + out_piece(first + i))[k] = wv[i];
        }
        __syncthreads();
        // one run of 16-byte stores, every instruction of a wavefront a whole KiB, written once
        constexpr int n_chunks = (R::kCodeBytes + 2 * kMetaBytes) / 16;   // 192 (INT2) / 320 (INT4)
        uint4 *dst = reinterpret_cast<uint4 *>(rec + R::kVCodes);
#pragma unroll
        for (int c = tid; c < n_chunks; c += 256) store_once(dst + c, rows[out_piece(c)]);
        return;
    }
    // A page that arrives in parts: a thread's words change in the fields of the tokens that arrive.  The tokens of a
    // word share the quad, which is the number of the wavefront: wavefronts without any have nothing to do.
    if (valid) {
        reinterpret_cast<uint16_t *>(rec + R::kVScale)[mi] = v_scale;
        reinterpret_cast<uint16_t *>(rec + R::kVZero)[mi] = v_zero;
    }
    uint32_t *vc = reinterpret_cast<uint32_t *>(rec + R::kVCodes);
    const int quad = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int i = 0; i < n_words / 256; ++i) {
        const int widx = tid + 256 * i;
        const int jl = widx & 3, n = (widx >> 2) & 15, jh = i & 1, blk = i >> 1;
        const int c = (jh * 4 + jl) * 16 + n;
        uint32_t field = 0;   // the bits of the word that change
#pragma unroll
        for (int p = 0; p < 32 / BITS; ++p)
            if ((mask >> v_token<BITS>(blk, quad, p)) & 1) field |= ((1u << BITS) - 1u) << (BITS * p);
        if (field == 0) continue;
        uint32_t val = 0;
#pragma unroll
        for (int p = 0; p < 32 / BITS; ++p)   // (the rows of other tokens hold anything)
            val |= ((uint32_t)codes[code_row(v_token<BITS>(blk, quad, p)) + c] & ((1u << BITS) - 1u)) << (BITS * p);
        vc[widx] = (old[i] & ~field) | (val & field);
    }
}

// One argument instead of fourteen: the runtime looks every pointer argument up on the way to a launch (one token for each of 32
// sequences, where the launch is what a call waits for, 4.04 -> 3.76 us; chunks of a few hundred tokens 7.9 -> 7.7).
struct AppendArgs {
    uint8_t *pool;
    uint8_t *bit_map;
    const uint16_t *K;
    const uint16_t *V;
    const uint8_t *tag_bits;
    int n_tokens;
    const int32_t *work_pages;
    const int32_t *work_src;
    int n_work;
    int first_head;
    int n_kv_heads;
    int n_pages_int2;
    int n_pages_int4;
    int32_t *status;
};
// K_ONCE: the K rows are read with non-temporal loads (see the launcher).
template <bool KC, bool K_ONCE>
__global__ __launch_bounds__(256) void tkv_append_kernel(AppendArgs args)
{
    uint8_t *__restrict__ pool = args.pool;
    uint8_t *__restrict__ bit_map = args.bit_map;
    const uint16_t *__restrict__ K = args.K;
    const uint16_t *__restrict__ V = args.V;
    const uint8_t *__restrict__ tag_bits = args.tag_bits;
    const int n_tokens = args.n_tokens;
    const int32_t *__restrict__ work_pages = args.work_pages;
    const int32_t *__restrict__ work_src = args.work_src;
    const int n_work = args.n_work;
    const int first_head = args.first_head;
    const int n_kv_heads = args.n_kv_heads;
    const int n_pages_int2 = args.n_pages_int2;
    const int n_pages_int4 = args.n_pages_int4;
    int32_t *status = args.status;

    __shared__ uint4 rows[kPageTokens * kRowPieces];
    const int w = blockIdx.z * 8 + blockIdx.x, head = first_head + (blockIdx.y >> 1);   // grid (8, 2 * heads, blocks of eight pages): see the launcher
    const bool is_v = blockIdx.y & 1;
    // A launch of a few tokens is a chain of loads: arguments -> page and slots -> tags, rows and words to merge.  All of
    // a level at once: an argument fetched where it is first used, a wait for the tag ahead of the rows, or for a slot between
    // two rows, is a round trip more.  (12288 tokens x 8 heads 13.4 -> 12.7 us, 65536 59.6 -> 58.7, per-channel keys 61.6 -> 59.2,
    // six ragged chunks 10.85 -> 10.15, four-layer step 78.1 -> 76.8.)
    asm volatile("" :: "s"(pool), "s"(bit_map), "s"(K), "s"(V), "s"(tag_bits), "s"(n_tokens), "s"(work_pages), "s"(work_src), "s"(n_work),
                 "s"(n_kv_heads), "s"(n_pages_int2), "s"(n_pages_int4), "s"(status));
    if (w >= n_work) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t *__restrict__ srcs = work_src + (size_t)w * kPageTokens;
    const int src = srcs[lane];   // every wavefront looks at all 64 slots
    int row_src[4];               // and fetches pieces of four rows per lane
#pragma unroll
    for (int i = 0; i < 4; ++i) row_src[i] = srcs[16 * wave + 4 * i + (lane >> 4)];
    const int page = ((const __attribute__((address_space(4))) int32_t *)work_pages)[w];
    asm volatile("" :: "s"(page), "v"(src), "v"(row_src[0]), "v"(row_src[1]), "v"(row_src[2]), "v"(row_src[3]));
    if (page < 0 || page >= n_pages_int2 + n_pages_int4) {
        if (status && tid == 0) atomicOr(status, TKV_STATUS_PAGE_RANGE);
        return;
    }
    const int bits = page < n_pages_int2 ? 2 : 4;
    uint8_t *rec = pool + record_offset(page, head, n_kv_heads, n_pages_int2);
    const bool in = src >= 0 && src < n_tokens;
    // the tag of this lane's slot; slots without a source lie outside the buffer and read 0
    const uint8_t tag = __builtin_amdgcn_raw_buffer_load_b8(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(tag_bits), 0, n_tokens, 0x00027000), src, 0, 0);
    const size_t stride = (size_t)n_kv_heads * kHeadDim;
    const uint16_t *from = (is_v ? V : K) + head * kHeadDim;
    auto fetch_rows = [&](auto once) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (row_src[i] >= 0 && row_src[i] < n_tokens)
                fetch_row_pieces<decltype(once)::value>(rows + 16 * wave * kRowPieces, i, from + (size_t)row_src[i] * stride, lane);
    };
    if (K_ONCE && !is_v) fetch_rows(std::true_type());
    else fetch_rows(std::false_type());
    // the V words of a page that does not arrive whole, in case they change
    uint32_t old[4] = {0, 0, 0, 0};
    auto fetch_old = [&]() {
        const uint32_t *vc = reinterpret_cast<const uint32_t *>(rec + (bits == 2 ? Rec<2>::kVCodes : Rec<4>::kVCodes)) + tid;
        old[0] = vc[0];
        old[1] = vc[256];
        if (bits == 4) {
            old[2] = vc[512];
            old[3] = vc[768];
        }
    };
    const bool in_parts = is_v && __ballot(in) != ~0ull;
    if (in_parts) fetch_old();
    const bool fits = in && tag == bits;
    uint64_t mask = __ballot(fits);
    if (in && !fits && status && wave == 0) atomicOr(status, TKV_STATUS_TAG_MISMATCH);
    if (is_v && mask != ~0ull && !in_parts) fetch_old();   // only where tags contradict the page
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the rows this wavefront fetched are in LDS
    if (KC && bits == 2) {
        // a block of 32 slots is quantised in one piece: it takes part whole or not at all
        uint64_t whole = 0;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const uint32_t half = (uint32_t)(mask >> (32 * b));
            if (half == 0xffffffffu) whole |= 0xffffffffull << (32 * b);
            else if (half != 0 && status && tid == 0) atomicOr(status, TKV_STATUS_BLOCK_PARTIAL);
        }
        mask = whole;
    }
    if (is_v) {
        if (bits == 2) append_v<2>(rec, mask, old, rows);
        else append_v<4>(rec, mask, old, rows);
    } else {
        if (bits == 2) append_k<2, KC>(rec, mask, rows);
        else append_k<4, false>(rec, mask, rows);
    }
    if (head == 0 && !is_v && tid == 0 && mask != 0) bit_map[page] = (uint8_t)bits;
}

} // namespace

int tkv_launch_append(const tkv_desc *desc, void *pool, uint8_t *bit_map, const void *K, const void *V,
                      const uint8_t *tag_bits, int32_t n_tokens, const int32_t *work_pages,
                      const int32_t *work_src, int32_t n_work, int32_t *status, void *stream)
{
    const bool kc = desc->int2_key_axis == TKV_KEYS_PER_CHANNEL;
    // How much of the input leaves the 256 MiB Infinity Cache alone.  Up to 64 MiB of rows are still there from whoever
    // computed them, and ordinary loads find them; larger inputs push each other out, and with the K rows read past the
    // cache the V rows stay in it.  us per call, ordinary / K past the cache / both, same rows again and again | rows not read
    // for three calls: 12288 tokens x 8 heads 11.7 / 11.5 / - | 12.1 / 12.3 / -; 20001 16.6 / 16.5 / 17.7 | 19.1 / 17.3 / 19.3;
    // 65536 45.6 / 46.9 / 55.9 | 61.0 / 58.4 / 57.9; 131072 (eight workgroups per CU) 120 / 89 / 113 | 121 / 116 / 115.
    const int64_t row_bytes = (int64_t)n_tokens * desc->n_kv_heads * (2 * kRowBytes);
    const bool k_once = row_bytes > (64 << 20);
    // Eight workgroups of 16 KiB are resident per compute unit.  From 320 MiB of rows on six (by idle LDS): eight ask for more
    // at once than the memory takes in.  us, eight / six, rows not read for three calls | same rows again and again, 8 heads:
    // 65536 tokens 59.2 / 58.0 | 46.3 / 48.3; 81920 73.9 / 72.4 | 56.5 / 58.7; 98304 88.7 / 86.3 | 66.5 / 69.4; 131072 117.5 /
    // 113.8 | 87 / 91; 163840 146 / 142 | 147 / 140; 262144 235 / 229.  Where a tag held up the rows (one wait more in the
    // chain of loads), eight took 74.0 | 59.8 at 81920, 87.7 | 70.3 at 98304, 115 | 92 at 131072, 171.5 (196608; six 170.4, eight
    // 176.3), 229: the line lies where eight become slower than that on rows that no cache holds.  (1 and 2 heads, and per-channel
    // keys: six are nowhere slower than that either.)
    const unsigned idle_lds = row_bytes > ((int64_t)320 << 20) ? 10200 : 0;
    auto kernel = kc ? (k_once ? tkv_append_kernel<true, true> : tkv_append_kernel<true, false>)
                     : (k_once ? tkv_append_kernel<false, true> : tkv_append_kernel<false, false>);
    // Workgroups are dealt to the eight XCDs in turn: the first grid dimension is the XCD, which reads the rows of all heads
    // of a page one behind the other (2 KiB per token at eight heads).  65 536 tokens x 8 heads, K and V both read past
    // the cache: 57.5 us against 59.2 with the heads of a page spread over the XCDs; K before V, as the gather does it,
    // makes no difference here.
    constexpr int kMaxPages = 8 * 65535, kMaxHeads = 65535 / 2;   // of one launch, by the limits of the grid
    for (int page = 0; page < n_work; page += kMaxPages)
        for (int head = 0; head < desc->n_kv_heads; head += kMaxHeads) {
            const int n = n_work - page < kMaxPages ? n_work - page : kMaxPages;
            const int h = desc->n_kv_heads - head < kMaxHeads ? desc->n_kv_heads - head : kMaxHeads;
            const AppendArgs args = {(uint8_t *)pool, bit_map, (const uint16_t *)K, (const uint16_t *)V, tag_bits, n_tokens, work_pages + page,
                                     work_src + (size_t)page * kPageTokens, n, head, desc->n_kv_heads, desc->n_pages_int2, desc->n_pages_int4,
                                     status};
            hipLaunchKernelGGL(kernel, dim3(8, 2 * (unsigned)h, (unsigned)((n + 7) / 8)), dim3(256), idle_lds, (hipStream_t)stream, args);
        }
    return hipGetLastError() == hipSuccess ? TKV_OK : TKV_ERR_HIP;
}
