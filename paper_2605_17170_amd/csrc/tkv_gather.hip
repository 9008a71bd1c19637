// tkv_gather_dequant: the prefill gather (paper Sec. 3.2.3 "Prefill"): reads the
// pages of a matched prefix from the mixed-precision pool, unpacks every
// listed slot, dequantises it into FP16 and writes dense K / V rows in the
// caller's token order, ready for an FP16 prefill attention kernel.
//
// Two workgroups of 256 threads per (page, kv head) record, the mirror image of the append kernel: one writes the K
// rows, one the V rows.  Thread (slot = tid/4, part = tid%4) produces channels 32*i + 8*part .. +7 of its token for
// the four groups i.  For K one 16-byte load fetches the codes of all four groups, and nothing goes through LDS.  V
// is stored channel-major (a word holds several tokens of one channel), so the V words are expanded into an LDS byte
// tile first and each thread reads its token's codes back.  A thread's four 16-byte pieces of a row would each fill a
// quarter of a line; mirror-image threads of two neighbouring slots trade pieces instead, so that eight lanes write
// one whole 128-byte line per store instruction, and the stores are non-temporal (the output is written once).
//
// Bound by the HBM write stream (82 % of its bytes).  One record per workgroup with everything it reads requested at
// once, eight workgroups to a compute unit, and an order of the workgroups that keeps the writes together (see the
// launcher): 65 536 tokens x 8 heads 61.2 -> 53.7 us, per-channel keys 68.9 -> 54.2, against three looping workgroups
// per compute unit that staged the next record in registers.
//
// Value: binary16 nearest-even of the exact code * scale + zero.  The fp16
// fused multiply-add gives exactly that: code, scale and zero are fp16
// numbers and the FMA rounds once.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include "tkv_internal.h"
#include "tkv_layout.h"

namespace {

using namespace tkv;

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

// A code under the bit pattern 0x6400 is the fp16 number 1024 + code (the fp16 spacing there is 1), and subtracting 1024
// is exact: two codes in bits 0.. and 16.. of x, the rest of which is masked away, as a pair of fp16 numbers.
template <int BITS> __device__ __forceinline__ half2_t code_pair(uint32_t x)
{
    constexpr uint32_t m = ((1u << BITS) - 1u) * 0x00010001u;
    const half2_t k = {(_Float16)1024.0f, (_Float16)1024.0f};
    return __builtin_bit_cast(half2_t, (x & m) | 0x64006400u) - k;
}
__device__ __forceinline__ uint32_t fma2(half2_t c, uint32_t s, uint32_t z)   // c * s + z, one rounding
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(c, __builtin_bit_cast(half2_t, s), __builtin_bit_cast(half2_t, z)));
}
// Low halves of a and b, high halves of a and b.
__device__ __forceinline__ uint32_t lows(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t highs(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
// Eight codes, 0..3 packed from bit 0 and 4..7 from bit 16 of x, to fp16 values.  s, z: the fp16 pairs (scale, zero) of
// codes (k, k + 4), k = 0..3.
template <int BITS> __device__ __forceinline__ uint4 dequant8(uint32_t x, const uint32_t (&s)[4], const uint32_t (&z)[4])
{
    uint32_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = fma2(code_pair<BITS>(x >> (BITS * k)), s[k], z[k]);
    return make_uint4(lows(v[0], v[1]), lows(v[2], v[3]), highs(v[0], v[1]), highs(v[2], v[3]));
}
template <int BITS> __device__ __forceinline__ uint4 dequant8(uint32_t x, uint32_t s, uint32_t z)   // the same pair for all
{
    const uint32_t sv[4] = {s, s, s, s}, zv[4] = {z, z, z, z};
    return dequant8<BITS>(x, sv, zv);
}
// Half i & 1 of the 16-bit halves of v, twice.
__device__ __forceinline__ uint32_t twice(uint32_t v, int i) { return __builtin_amdgcn_perm(v, v, (i & 1) ? 0x07060706u : 0x05040504u); }

// Value of the lane that mirrors this one within its group of eight lanes (lane ^ 7).
__device__ __forceinline__ uint32_t half_mirror(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true);
}
__device__ __forceinline__ uint4 half_mirror(uint4 v)
{
    return make_uint4(half_mirror(v.x), half_mirror(v.y), half_mirror(v.z), half_mirror(v.w));
}
__device__ __forceinline__ uint4 pick(bool c, uint4 a, uint4 b) { return c ? a : b; }
// Stores the four 16-byte pieces v[i] (channels 32 i + 8 part .. + 7) of this thread's token row so that every
// store instruction of a wavefront writes whole 128-byte lines: thread (slot, part) and thread (slot ^ 1, 3 - part),
// mirror images within eight lanes, trade one piece per line, and the eight lanes write first the line of the even
// slot's row, then that of the odd slot's.
__device__ __forceinline__ void store_row(uint16_t *__restrict__ out, int dst, bool valid, const uint4 (&v)[4], int slot, int part,
                                          int head, int n_kv_heads)
{
    const bool odd = slot & 1;
    const int dst_other = (int)half_mirror((uint32_t)dst);
    const bool valid_other = half_mirror((uint32_t)valid) != 0;
    const bool valid_even = odd ? valid_other : valid, valid_odd = odd ? valid : valid_other;
    // (a row that is not written gets the address of row 0: no pointer is formed from an index that was never checked)
    const size_t dst_even = valid_even ? (size_t)(odd ? dst_other : dst) : 0, dst_odd = valid_odd ? (size_t)(odd ? dst : dst_other) : 0;
    uint4 *row_even = reinterpret_cast<uint4 *>(out + (dst_even * n_kv_heads + head) * kHeadDim);
    uint4 *row_odd = reinterpret_cast<uint4 *>(out + (dst_odd * n_kv_heads + head) * kHeadDim);
    // Through the L2: what a short launch leaves dirty there holds up the next one (three prefixes of 701 to 9001 tokens, 8 heads,
    // 7.8 -> 7.0 us, 65536 tokens on one head 8.45 -> 8.15; 35 shapes from one page to 262144 tokens x 8 heads .985 to 1.09 times as
    // fast, the smallest by no more than their spread; without nt 65536 tokens x 8 heads would take 66 us, not 54).
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint4 recv = half_mirror(pick(odd, v[2 * h], v[2 * h + 1]));
        if (valid_even) store_once_through(row_even + 8 * h + (odd ? 7 - part : part), pick(odd, recv, v[2 * h]));
        if (valid_odd) store_once_through(row_odd + 8 * h + (odd ? 4 + part : 3 - part), pick(odd, v[2 * h + 1], recv));
    }
}

// KC: the keys of an INT2 record are quantised per channel over blocks of 32 slots.
template <int BITS, bool KC>
__device__ __forceinline__ void gather_k(const uint8_t *__restrict__ rec, uint16_t *__restrict__ K_out, int dst, bool valid, int head,
                                         int n_kv_heads, uint4 *lds)
{
    using R = Rec<BITS>;
    const int tid = threadIdx.x, slot = tid >> 2, part = tid & 3;
    const int tile = slot >> 4, row = slot & 15;
    // INT4: chunk (tile*4 + part)*16 + row = word `part` (8 channels) of the four groups
    // INT2: chunk (tile*2 + part/2)*16 + row = word part/2 (16 channels); this thread takes half part%2
    // read once, and an instruction of a wavefront covers 1 KiB (INT4) or 512 B (INT2) of whole lines
    const uint4 kw = load_once(reinterpret_cast<const uint4 *>(rec + R::kKCodes) +
                               (BITS == 4 ? (tile * 4 + part) * 16 + row : (tile * 2 + (part >> 1)) * 16 + row));
    const uint32_t w[4] = {kw.x, kw.y, kw.z, kw.w};
    // INT4: nibbles 0..3 and 4..7 already lie in the two halves of the word.  INT2: the bytes of this thread's half move there.
    auto spread = [&](uint32_t x) { return BITS == 4 ? x : __builtin_amdgcn_perm(x, x, (part & 1) ? 0x0c070c06u : 0x0c050c04u); };
    uint4 kv[4];
    if constexpr (!KC) {
        const uint2 ksc = reinterpret_cast<const uint2 *>(rec + R::kKScale)[slot], kzc = reinterpret_cast<const uint2 *>(rec + R::kKZero)[slot];
#pragma unroll
        for (int i = 0; i < 4; ++i) kv[i] = dequant8<BITS>(spread(w[i]), twice(i < 2 ? ksc.x : ksc.y, i), twice(i < 2 ? kzc.x : kzc.y, i));
    } else {
        if (tid < 64) lds[tid] = reinterpret_cast<const uint4 *>(rec + R::kKScale)[tid];   // 512 B scale, 512 B zero
        __syncthreads();
        // channels 32*i + 8*part + j: chunks (block, group i, quarter 2*(part/2) + j/4) of the planes, fp16
        // half part%2 of word j%4
        const uint4 *sp4 = lds + (slot >> 5) * 16 + 2 * (part >> 1);
        const uint4 *zp4 = sp4 + 32;
        const uint32_t sel = (part & 1) ? 0x07060302u : 0x05040100u;   // v_perm: the chosen halves of (second, first)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 s0 = sp4[4 * i], s1 = sp4[4 * i + 1], z0 = zp4[4 * i], z1 = zp4[4 * i + 1];
            const uint32_t sp[4] = {__builtin_amdgcn_perm(s1.x, s0.x, sel), __builtin_amdgcn_perm(s1.y, s0.y, sel),
                                    __builtin_amdgcn_perm(s1.z, s0.z, sel), __builtin_amdgcn_perm(s1.w, s0.w, sel)};
            const uint32_t zp[4] = {__builtin_amdgcn_perm(z1.x, z0.x, sel), __builtin_amdgcn_perm(z1.y, z0.y, sel),
                                    __builtin_amdgcn_perm(z1.z, z0.z, sel), __builtin_amdgcn_perm(z1.w, z0.w, sel)};
            kv[i] = dequant8<BITS>(spread(w[i]), sp, zp);
        }
    }
    store_row(K_out, dst, valid, kv, slot, part, head, n_kv_heads);
}

// V codes of the page, one per byte, in LDS: 144-byte rows, because the four quads that one instruction writes lie four
// rows apart and must not meet on the same banks; then the V scale plane and the V zero plane as stored.
constexpr int kCodeRow = 144;
struct VLds {
    alignas(16) uint8_t codes[kPageTokens * kCodeRow];
    alignas(16) uint16_t meta[2 * kPageTokens * kGroups];
};

template <int BITS>
__device__ __forceinline__ void gather_v(const uint8_t *__restrict__ rec, uint16_t *__restrict__ V_out, int dst, bool valid, int head,
                                         int n_kv_heads, VLds &lds)
{
    using R = Rec<BITS>;
    const int tid = threadIdx.x, slot = tid >> 2, part = tid & 3;
    constexpr int n_quads = R::kCodeBytes / 16;   // 256 (INT4) / 128 (INT2)
    if (tid < n_quads) {
        // four words of four adjacent channels c0 .. c0 + 3, so that a token's four codes go out as one 32-bit write
        const uint32_t *vc = reinterpret_cast<const uint32_t *>(rec + R::kVCodes);
        const int jl = tid & 3, nq = (tid >> 2) & 3, quad = (tid >> 4) & 3, jh = (tid >> 6) & 1;
        const int blk = tid >> 7;   // INT4 only (0 for INT2)
        const int widx = jl + 16 * nq + 64 * quad + 256 * jh + 512 * blk;   // word of channel c0; c0 + k is 4*k words on
        const int c0 = (jh * 4 + jl) * 16 + 4 * nq;
        const uint32_t w[4] = {vc[widx], vc[widx + 4], vc[widx + 8], vc[widx + 12]};
        // byte b of a word holds 8 / BITS positions; position e of every byte, then the 4 x 4 bytes transposed
#pragma unroll
        for (int e = 0; e < 8 / BITS; ++e) {
            constexpr uint32_t m = ((1u << BITS) - 1u) * 0x01010101u;
            uint32_t x[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k] = (w[k] >> (BITS * e)) & m;
            const uint32_t t01 = __builtin_amdgcn_perm(x[1], x[0], 0x05010400u), u01 = __builtin_amdgcn_perm(x[1], x[0], 0x07030602u);
            const uint32_t t23 = __builtin_amdgcn_perm(x[3], x[2], 0x05010400u), u23 = __builtin_amdgcn_perm(x[3], x[2], 0x07030602u);
            const uint32_t four[4] = {lows(t01, t23), highs(t01, t23), lows(u01, u23), highs(u01, u23)};
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int p = (8 / BITS) * b + e;   // position of the token in the word
                const int j = BITS == 4 ? 2 * (p & 3) + (p >> 2) : 2 * (p & 3) + (p >> 3);
                const int t = 32 * (BITS == 4 ? blk : (p & 7) >> 2) + 16 * (j >> 2) + 4 * quad + (j & 3);
                *reinterpret_cast<uint32_t *>(&lds.codes[t * kCodeRow + c0]) = four[b];
            }
        }
    }
    if (tid < 128) reinterpret_cast<uint2 *>(lds.meta)[tid] = reinterpret_cast<const uint2 *>(rec + R::kVScale)[tid];   // 512 B scale, 512 B zero
    __syncthreads();
    uint4 vv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int mi = vmeta_index(slot, i);
        const uint2 cb = *reinterpret_cast<const uint2 *>(&lds.codes[slot * kCodeRow + 32 * i + 8 * part]);
        // codes 0..3 and 4..7 one per byte; code_pair wants (k, k + 4) in the halves of a word
        const uint32_t s = lds.meta[mi] * 0x00010001u, z = lds.meta[kPageTokens * kGroups + mi] * 0x00010001u;
        uint32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t sel = 0x0c000c04u + k * 0x00010001u;   // byte k of lo, zero, byte k of hi, zero
            v[k] = fma2(code_pair<BITS>(__builtin_amdgcn_perm(cb.x, cb.y, sel)), s, z);
        }
        vv[i] = make_uint4(lows(v[0], v[1]), lows(v[2], v[3]), highs(v[0], v[1]), highs(v[2], v[3]));
    }
    store_row(V_out, dst, valid, vv, slot, part, head, n_kv_heads);
}

// One argument instead of thirteen, as in the other kernels: a launch costs the host less (prefixes of a few hundred tokens 1 to 5 %).
struct GatherArgs {
    const uint8_t *pool;
    const uint8_t *bit_map;
    const int32_t *work_pages;
    const int32_t *work_dst;
    int n_work;
    int first_head;
    int n_kv_heads;
    int n_pages_int2;
    int n_pages_int4;
    uint16_t *K_out;
    uint16_t *V_out;
    int n_tokens;
    int32_t *status;
};
template <bool KC>
__device__ __forceinline__ void gather_record(
    const uint8_t *__restrict__ pool, const uint8_t *__restrict__ bit_map, const int32_t *__restrict__ work_pages,
    const int32_t *__restrict__ work_dst, int n_work, int first_head, int n_kv_heads, int n_pages_int2, int n_pages_int4,
    uint16_t *__restrict__ K_out, uint16_t *__restrict__ V_out, int n_tokens, int32_t *status)
{
    __shared__ VLds lds;
    // grid (8, heads, 2 * blocks of eight pages): see the launcher
    const int n_blocks = gridDim.z >> 1;
    const bool is_v = blockIdx.z >= n_blocks;
    const int w = (blockIdx.z - (is_v ? n_blocks : 0)) * 8 + blockIdx.x, head = first_head + blockIdx.y;
    if (w >= n_work) return;
    const int page = work_pages[w];
    const int dst = work_dst[(size_t)w * kPageTokens + (threadIdx.x >> 2)];
    if (page < 0 || page >= n_pages_int2 + n_pages_int4) {
        if (status && threadIdx.x == 0) atomicOr(status, TKV_STATUS_PAGE_RANGE);
        return;
    }
    const int bits = page < n_pages_int2 ? 2 : 4;
    const uint8_t *rec = pool + record_offset(page, head, n_kv_heads, n_pages_int2);
    // a page that was never written, or written at another width, is read (its address is valid) and nothing of it
    // is stored
    const bool written = bit_map[page] == bits;
    if (!written && status && threadIdx.x == 0) atomicOr(status, TKV_STATUS_BITMAP_MISMATCH);
    const bool valid = written && dst >= 0 && dst < n_tokens;
    if (written && dst >= n_tokens && status && (threadIdx.x & 3) == 0) atomicOr(status, TKV_STATUS_DST_RANGE);
    if (is_v) {
        if (bits == 2) gather_v<2>(rec, V_out, dst, valid, head, n_kv_heads, lds);
        else gather_v<4>(rec, V_out, dst, valid, head, n_kv_heads, lds);
    } else {
        if (bits == 2) gather_k<2, KC>(rec, K_out, dst, valid, head, n_kv_heads, reinterpret_cast<uint4 *>(&lds));
        else gather_k<4, false>(rec, K_out, dst, valid, head, n_kv_heads, reinterpret_cast<uint4 *>(&lds));
    }
}
template <bool KC>
__global__ __launch_bounds__(256) void tkv_gather_kernel(GatherArgs a)
{
    gather_record<KC>(a.pool, a.bit_map, a.work_pages, a.work_dst, a.n_work, a.first_head, a.n_kv_heads, a.n_pages_int2, a.n_pages_int4,
                      a.K_out, a.V_out, a.n_tokens, a.status);
}

} // namespace

int tkv_launch_gather(const tkv_desc *desc, const void *pool, const uint8_t *bit_map, const int32_t *work_pages,
                      const int32_t *work_dst, int32_t n_work, void *K_out, void *V_out, int32_t n_tokens,
                      int32_t *status, void *stream)
{
    const bool kc = desc->int2_key_axis == TKV_KEYS_PER_CHANNEL;
    auto kernel = kc ? tkv_gather_kernel<true> : tkv_gather_kernel<false>;
    // Which workgroup does what, and when: workgroups are dealt to the eight XCDs in turn, so the first grid dimension is
    // the XCD: it writes the rows of all heads of a page one behind the other (2 KiB per token at eight heads), and
    // all K rows are written before the V rows.  65 536 tokens x 8 heads: 53.7 us (6.1 TB/s; a plain 1 : 4 stream reaches
    // 6.2) against 61.2 with K and V of a record side by side, 54.5 with the heads of a page spread over the XCDs and
    // 69.9 with both: two write streams at a time cost more than anything else here.
    constexpr int kMaxPages = 8 * (65535 / 2), kMaxHeads = 65535;   // of one launch, by the limits of the grid
    for (int page = 0; page < n_work; page += kMaxPages)
        for (int head = 0; head < desc->n_kv_heads; head += kMaxHeads) {
            const int n = n_work - page < kMaxPages ? n_work - page : kMaxPages;
            const int h = desc->n_kv_heads - head < kMaxHeads ? desc->n_kv_heads - head : kMaxHeads;
            const GatherArgs args = {(const uint8_t *)pool, bit_map, work_pages + page, work_dst + (size_t)page * kPageTokens, n, head,
                                     desc->n_kv_heads, desc->n_pages_int2, desc->n_pages_int4, (uint16_t *)K_out, (uint16_t *)V_out, n_tokens,
                                     status};
            hipLaunchKernelGGL(kernel, dim3(8, (unsigned)h, 2 * (unsigned)((n + 7) / 8)), dim3(256), 0, (hipStream_t)stream, args);
        }
    return hipGetLastError() == hipSuccess ? TKV_OK : TKV_ERR_HIP;
}
