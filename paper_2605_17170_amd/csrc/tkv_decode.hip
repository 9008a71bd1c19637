// tkv_decode_attention: split-K flash-decoding over the paged INT2 / INT4 KV
// pool with in-register dequantisation, and the cross-split reduction
// (paper Sec. 3.2.3 "Decode").
//
// One wavefront owns one (work item, kv head): a contiguous range of one
// sequence's page list.  All query heads that share the kv head (up to 8)
// are processed together so the packed KV bytes are read from HBM once; the
// partials (m, l, acc) of the items are merged by tkv_merge_kernel or tkv_reduce_rows_kernel.
//
// Matrix cores do both contractions (v_mfma_f32_16x16x32_f16), fp32 accumulate,
// and the packed codes are never expanded by arithmetic: a masked 16-bit field
// with a code in its low ten bits *is* the fp16 subnormal code * 2^(pos-24), so
// unpacking is one AND per two codes, for K and for V.
//
//   QK^T  D[token, head] = sum_c code[token, c] * q[head, c].  q is converted to fp16
//         once, scaled by a power of two common to the heads and by 2^-pos per slot
//         (exact above the subnormals of fp16, see build_q_operand); the K scale
//         (fp32, times the compensating power of two) multiplies the MFMA result.  The
//         eight heads fill half of the 16 columns, so the columns carry two token sets:
//         row r of a 32-token block is token r in columns 0..7 and token 16 + r in
//         columns 8..15; an MFMA contracts half a group (16 channels) of both, the B
//         operand holding q in the k-slots of the column's own set and zeros in the
//         others.  Scale, exponential and weight pieces are then formed once per
//         (token, head).  The zero-point term sum_g zero[token,g] * sum_{c in g} q[head,c]
//         is one more MFMA per block whose A operand is the stored fp16 zero plane; the
//         sums of q are fp32, in three fp16 pieces.
//         (Per-channel INT2 keys use the columns differently, see compute_page.)
//   PV    D[(piece, head), channel] = sum_token a[piece, head, token, g] * code[token, channel],
//         a = W * scale[token, g] in two pieces, W the softmax weight: the V scale multiplies the
//         weights, not the codes.  Rows 0..7 carry the leading pieces of the heads, rows 8..15 the
//         second pieces, and the two are added once, in the epilogue: every row and column
//         of every MFMA counts.  (With rows 8..15 for other groups than rows 0..7 and an MFMA
//         for each piece, half of every result was never read: 32 MFMAs a page instead of 16.
//         MFMAs and other vector instructions of the three wavefronts of a SIMD hardly overlap:
//         16 of these MFMAs alone take 85 ns, 64 FMAs 68 ns, both together 123 to 133 ns.
//         With cache-resident pages an INT2 page takes 0.77 us of its SIMD instead of 0.84, an
//         INT4 page 0.81 instead of 0.86.)
//         The weights must be good to about 2^-17: a group with outlier channels has
//         |code * scale| and |zero| of tens that cancel, and the tolerance near zero is
//         2e-3.  W is therefore carried in two fp16 pieces (the leading 11 bits, then the
//         next 11), and a in two pieces as well: a_hi = fp16(W_hi * s), a_lo = W_lo * s +
//         the exact remainder of the hi product (packed fp16 FMAs).  The zero-point term
//         sum_t W * zero[t, g] and the softmax denominator sum_t W come from one more
//         pair of MFMAs per 32 tokens against the stored zero plane and a column of ones.  (As
//         one MFMA with the pieces in separate rows it would round less, but not as the code
//         term does, which it cancels: error of 32 contexts of 4K to 128K 6.6e-6 -> 7.0e-6,
//         as a pair 5.7e-6.)
//
// Every product the MFMAs see is exact; the roundings are fp32 accumulation (the sums of
// q among it), the fp32 K-scale multiply, the 22-bit softmax weight (common to numerator and denominator),
// the two-piece a, and those of channels of q far below the largest of the kv head's heads (build_q_operand).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <mutex>
#include <type_traits>

#include "tkv_internal.h"
#include "tkv_layout.h"

namespace {

using namespace tkv;

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

typedef const __attribute__((address_space(4))) int32_t *ConstWords;   // words that stay as they are during a launch: scalar loads

constexpr float kTau = 4.0f;   // rescale when a logit exceeds the reference maximum by this much (log2 units)
// Softmax weights are carried in fp16 as W = P * 2^kPExp (P <= 2^kTau), so that small weights stay clear
// of the fp16 subnormal grid; numerator and denominator share the factor.
constexpr int kPExp = 8;
// The V scale is staged as scale * 2^(kVExp - pos), pos = bit position of the code's field in its fp16 half; undone once in the epilogue.
constexpr int kVExp = -1;
// W * staged scale must stay finite in fp16: the staged scale is clamped to 65504 / 2^(kTau + kPExp)
constexpr uint32_t kVsClamp = 0x4bff4bffu;   // fp16 15.99 twice
// Per-channel INT2 keys: q'' (q normalised, times its slot factor) stays below 2^6 and is multiplied by the K scale in fp16; the scale saturates at 1023.
constexpr uint32_t kKcClamp = 0x63fe63feu;   // fp16 1023 twice
constexpr int kKcQExp = 9;   // the first slot factor is 2^-3, so q'' stays below 2^6

__device__ __forceinline__ half8 as_half8(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    uint4v v = {a, b, c, d};
    return __builtin_bit_cast(half8, v);
}
__device__ __forceinline__ uint32_t pk_mul(uint32_t x, uint32_t y)
{
    const half2_t r = __builtin_bit_cast(half2_t, x) * __builtin_bit_cast(half2_t, y);
    return __builtin_bit_cast(uint32_t, r);
}
__device__ __forceinline__ uint32_t pk_rem(uint32_t x, uint32_t y, uint32_t h)   // x * y - h per fp16 half, one rounding
{
    const half2_t r = __builtin_elementwise_fma(__builtin_bit_cast(half2_t, x), __builtin_bit_cast(half2_t, y),
                                                -__builtin_bit_cast(half2_t, h));
    return __builtin_bit_cast(uint32_t, r);
}
__device__ __forceinline__ uint32_t pk_min(uint32_t x, uint32_t y)
{
    const half2_t r = __builtin_elementwise_min(__builtin_bit_cast(half2_t, x), __builtin_bit_cast(half2_t, y));
    return __builtin_bit_cast(uint32_t, r);
}
// p - k * t where t is the fp16 value in the low (HALF = 0) or high (HALF = 1) half of `t2`
template <int HALF> __device__ __forceinline__ float residual(uint32_t t2, float negk, float p)
{
    float r;
    if (HALF == 0) asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(t2), "v"(negk), "v"(p));
    else asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(t2), "v"(negk), "v"(p));
    return r;
}
__device__ __forceinline__ uint32_t pk_fma(uint32_t x, uint32_t y, uint32_t z)   // x * y + z per fp16 half, one rounding
{
    const half2_t r = __builtin_elementwise_fma(__builtin_bit_cast(half2_t, x), __builtin_bit_cast(half2_t, y),
                                                __builtin_bit_cast(half2_t, z));
    return __builtin_bit_cast(uint32_t, r);
}
__device__ __forceinline__ uint32_t pack_h2(float a, float b)
{
    const half2_t v = {(_Float16)a, (_Float16)b};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ floatx4 mfma(half8 a, half8 b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
// The value of the lane eight columns on in the same row of 16 lanes.  (In all DPP moves here every lane has a source;
// `bound_ctrl` says so to the compiler, which otherwise presets the destination register with a move of its own.)
__device__ __forceinline__ float row_ror8(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128 /* row_ror:8 */, 0xf, 0xf, true));
}
// The A operand of a PV MFMA from the two pieces (hi, lo) that every lane has made for its own four tokens (two fp16 pairs
// each): row r < 8 is the leading piece of head r, row r + 8 the second, and the k-slot octet of both lists the four tokens
// of the lanes of columns 0..7, then those of columns 8..15.  A lane keeps the piece its row wants and takes the other four
// tokens from the lane eight columns on: one select with a DPP operand per register.  (DPP moves into a preset register
// need a copy of one of the pieces as well, 25 moves a page.)  Two wait states are due between the write of a register
// and its DPP read, and between the write and the read by an MFMA; the compiler does not see the instructions in here.
__device__ __forceinline__ half8 piece_rows(const uint32_t (&hi)[2], const uint32_t (&lo)[2])
{
    uint32_t r0, r1, r2, r3;
    asm("s_nop 0\n\t"
        "s_mov_b64 vcc, %8\n\t"
        "v_cndmask_b32_dpp %0, %6, %4, vcc row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %1, %7, %5, vcc row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "s_not_b64 vcc, vcc\n\t"
        "v_cndmask_b32_dpp %2, %4, %6, vcc row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %3, %5, %7, vcc row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1"
        : "=&v"(r0), "=&v"(r1), "=&v"(r2), "=&v"(r3)
        : "v"(hi[0]), "v"(hi[1]), "v"(lo[0]), "v"(lo[1]), "s"(0x00ff00ff00ff00ffull /* columns 0..7 */)
        : "vcc", "scc");
    return as_half8(r0, r1, r2, r3);
}
__device__ __forceinline__ uint32_t ror8_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128 /* row_ror:8 */, 0xf, 0xf, true);
}
// x and y hold the sums of the two pieces of the weights in lanes 0..31 and 32..63: adds the pieces, x in lanes 0..31, y in
// lanes 32..63.
__device__ __forceinline__ float add_pieces(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y), false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
// The larger of the two results of a swap of a register with itself (lane i has the values of lanes i and i ^ 16 or i ^ 32).
template <class Pair> __device__ __forceinline__ float swap_max(Pair r) { return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])); }
// The value of another lane of the same row of 16 lanes: CTRL is a DPP pattern under which every lane has a source.
template <int CTRL> __device__ __forceinline__ int row_dpp(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true); }
template <int CTRL> __device__ __forceinline__ float row_dpp(float v) { return __builtin_bit_cast(float, row_dpp<CTRL>(__builtin_bit_cast(int, v))); }
// Maximum over a row of 16 lanes, in every lane of the row: neighbours, pairs, quads, halves
// (quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror, row_mirror).
__device__ __forceinline__ int row_max(int v)
{
    v = max(v, row_dpp<0xB1>(v));
    v = max(v, row_dpp<0x4E>(v));
    v = max(v, row_dpp<0x141>(v));
    return max(v, row_dpp<0x140>(v));
}
__device__ __forceinline__ int wave_max(int v)
{
    v = row_max(v);
    const int r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
    const int r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
    const int a = r0 > r1 ? r0 : r1, b = r2 > r3 ? r2 : r3;
    return a > b ? a : b;
}
// Orders this wavefront's LDS writes before its later LDS reads.  The workgroup is one wavefront
// and LDS operations of a wavefront execute in order, so no wait and no barrier instruction is needed.
__device__ __forceinline__ void lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct WaveState {
    // PV accumulators.  Lane (c = lane % 16, q4 = lane / 16) holds rows 4*q4 + i: head 4*(q4 & 1) + i, leading piece of the
    // weights (q4 < 2) or second piece; acc[half][comp] is channel 64*half + 16*comp + c.
    floatx4 acc[2][4];
    floatx4 zp;         // rows 0..7: sum_t W * zero[t, g] in columns 0..3 (groups), sum_t W in column 4
    uint32_t sat;       // non-zero once a staged scale was clamped (reported in the status word at the end)
    float m_ref;        // reference maximum of this lane's head column, log2 units, -inf before the first page
};

// q operands of the QK^T MFMAs with two token sets: per (group, half group) 16 entries (sub*8 + head) and two entries of
// zeros.  The 16 lanes that a 16-byte LDS read serves together hold eight lanes that read their own entries
// sub*8 .. sub*8+7 (32 consecutive banks) and eight that read zeros: the zero entry they use lies in the other 32
// banks (entry 16 for sub = 1, entry 24 for sub = 0; entries 17..23 are padding).
constexpr int kQyStride = 25, kQyZero0 = 24, kQyZero1 = 16;
constexpr int kPvZ = 0, kPvS = 32, kPvZero = 64, kPvOne = 65, kPvChunks = 66;

// Entries of the q operand tables: 16 bytes for (group, half group, channel octet sub, head).  With per-channel INT2 keys
// they lie densely; lane (r16, q4) of an MFMA reads entry (g, q4 >> 1, q4 & 1, r16 & 7).
constexpr int kQcEntries = kGroups * 32;
// What only the kernel for per-channel INT2 keys keeps in LDS: the second q operand.
template <bool KC> struct LdsExtra {};
template <> struct LdsExtra<true> {
    alignas(16) uint4 qp[kQcEntries];                    // q * 2^E in the slot order of qo, without the slot factors
};
template <bool KC> struct alignas(16) Lds : LdsExtra<KC> {
    // Per-channel INT2 keys reuse ks while INT2 pages run: the K scale plane (512 B) and the K zero plane (512 B) of
    // the page as stored (the INT4 pages, which come later in an item, overwrite them with their own staging).
    alignas(16) float ks[kPageTokens * kGroups];         // K scale * F, fp32 [token][group]
    // Operands of the PV phase, 16-byte chunks of eight fp16 (the tokens of one k-slot octet), one array so that
    // a lane-dependent index can choose between staged data and the constants:
    //   kPvZ + (blk*4 + quad)*4 + g   V zero, as stored
    //   kPvS + (blk*4 + quad)*4 + g   V scale * 2^(kVExp - pos)
    //   kPvZero   zeros;   kPvOne   ones
    alignas(16) uint4 pv[kPvChunks];
    // B operands of the QK^T MFMAs (build_q_operand): 8 x (16 entries + zeros), or, per-channel INT2 keys, kQcEntries
    alignas(16) uint4 qo[8 * kQyStride];
    static_assert(8 * kQyStride >= kQcEntries, "either table");
    // group sums of q (prologue: per head 12 fp16, the pieces of the four sums); zero-point sums of the groups and the
    // denominator (epilogue: per head 5 floats)
    alignas(16) float zl[8][8];
    alignas(16) float alpha[16];
    __device__ __forceinline__ uint4 *kc_scale() { return reinterpret_cast<uint4 *>(ks); }
    __device__ __forceinline__ uint4 *kc_zero() { return reinterpret_cast<uint4 *>(ks) + 32; }
};

// q of one work item: lane (head = lane / 8, c = lane % 8) holds channels 8 c .. 8 c + 7 and 64 + 8 c .. of its head, two
// loads of whole lines.  Channel octet c of half j lies in group 2 j + c / 4, half group (c / 2) % 2, octet c % 2.
// (Staged in LDS as rows and read back in operand order, q cost 24 LDS instructions more, a round trip and, with a row sum of
// four DPP steps per head, four times the additions.)
struct QRegs { uint4 x[2]; };
__device__ __forceinline__ void load_q(QRegs &qr, const uint16_t *__restrict__ q_head /* this lane's head */, int lane)
{
#pragma unroll
    for (int j = 0; j < 2; ++j) qr.x[j] = reinterpret_cast<const uint4 *>(q_head)[8 * j + (lane & 7)];
}
__device__ __forceinline__ float bf16_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }

// B operands of the QK^T MFMAs for one width, kept in LDS: entries of eight fp16 holding q' = q * 2^E * 2^-pos in the slot
// order the unpack produces.  INT4 words list the eight channels of an octet, register k holds channels k and k + 4; INT2
// words list the sixteen of a half group, an entry has channels 4 sub + k and 8 + 4 sub + k: the lanes of the two octets
// trade four channels.
//  - per-channel INT2 keys: dense entries, plus the copy without slot factors;
//  - otherwise (two token sets, see compute_page): per (group, half group) one entry per (channel octet sub,
//    head) and an entry of zeros, which the lanes whose k-slots belong to the other token set read.
// The slot factors are powers of two and q * 2^E has 8 significant bits: the fp16 products are exact unless they
// fall below the grid of the subnormals, 2^-24.  With a slot factor of 2^-p that spares every q down to 2^(p-31) of the largest
// |q| of the heads, 2^(p-25) in the kernel for per-channel INT2 keys, whose q * 2^E stays below 2^kKcQExp: INT2 (p up to 9)
// down to 2^-22 and 2^-16, INT4 (p = 0 or 4) down to 2^-27 and 2^-21, the copy without slot factors down to 2^-25.  What is
// smaller rounds once, by at most 2^(p-39) of the largest |q| (2^(p-33)); for per-channel INT2 keys twice, first by 2^-33
// on the way to the copy.
template <int BITS, bool KC>
__device__ __forceinline__ void build_q_operand(const QRegs &qr, float two_e, int lane, Lds<KC> &lds)
{
    const int head = lane >> 3, sub = lane & 1, hg = (lane >> 1) & 1;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int g = 2 * j + ((lane >> 2) & 1);
        uint32_t x[2] = {qr.x[j].x, qr.x[j].y}, y[2] = {qr.x[j].z, qr.x[j].w};
        if (BITS == 2) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t other = (uint32_t)row_dpp<0xB1>((int)(sub ? x[i] : y[i]));
                x[i] = sub ? other : x[i];
                y[i] = sub ? y[i] : other;
            }
        }
        auto pair = [&](int k, float f) {   // channels k of x and y, times f
            return (k & 1) ? pack_h2(bf16_hi(x[k >> 1]) * f, bf16_hi(y[k >> 1]) * f) : pack_h2(bf16_lo(x[k >> 1]) * f, bf16_lo(y[k >> 1]) * f);
        };
        uint32_t r[4];
        if constexpr (KC && BITS == 2) {
            // the unpack leaves the field of slot k at bit 2k + 3 (see compute_page)
            constexpr uint32_t kSlot2[4] = {0x30003000u, 0x28002800u, 0x20002000u, 0x18001800u};   // fp16 2^-3, 2^-5, 2^-7, 2^-9 twice
#pragma unroll
            for (int k = 0; k < 4; ++k) r[k] = pair(k, two_e);
            const int e = g * 32 + hg * 16 + sub * 8 + head;
            lds.qp[e] = make_uint4(r[0], r[1], r[2], r[3]);
            lds.qo[e] = make_uint4(pk_mul(r[0], kSlot2[0]), pk_mul(r[1], kSlot2[1]), pk_mul(r[2], kSlot2[2]), pk_mul(r[3], kSlot2[3]));
        } else {
            // INT4: fields at bits 0 and 4 of a half, in turn; INT2: at bit 2k + 3
#pragma unroll
            for (int k = 0; k < 4; ++k) r[k] = pair(k, two_e * (BITS == 4 ? ((k & 1) ? 0.0625f : 1.0f) : 0.125f / (float)(1 << (2 * k))));
            lds.qo[(g * 2 + hg) * kQyStride + sub * 8 + head] = make_uint4(r[0], r[1], r[2], r[3]);
        }
    }
    if constexpr (!(KC && BITS == 2)) {
        if (lane < 16) lds.qo[(lane & 7) * kQyStride + (lane < 8 ? kQyZero0 : kQyZero1)] = make_uint4(0u, 0u, 0u, 0u);
    }
}

// Everything one wavefront loads for one (page, kv head) record.
template <int BITS> struct PageRegs {
    uint4 kw[4];          // K codes, 16-byte chunks of four group words: [blk*2 + half group] of this lane's token (two token
                          // sets), or one per 16-token tile (per-channel INT2 keys)
    uint4 vw[BITS];       // V codes: 16-byte chunks, one word per 16-channel tile; [blk*2 + channel half] (INT4), [channel half] (INT2)
    uint2 ksc, vsc, vzc;  // this lane's four entries of the K scale / V scale / V zero planes
    uint2 kzc;            // K zero of token `lane`, four groups
};

// A record as a buffer: base address and size in scalar registers, so that a load needs one 32-bit lane offset.  Size 0
// makes every load of it return zeros without touching memory: that is how a wavefront runs past its last page
// without a branch around the loads (a branch would make the compiler wait for all of them in every iteration).  A
// wavefront that asked for its last record again instead, as it used to, read 9 % more than the cache holds at eleven
// pages per wavefront (8 sequences of 32768 tokens: step 51.3 -> 49.1 us) and twice as much at one.
typedef __amdgpu_buffer_rsrc_t Record;
template <int BITS> __device__ __forceinline__ Record record_at(const uint8_t *__restrict__ rec, bool wanted)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(rec), 0, wanted ? Rec<BITS>::kBytes : 0, 0x00027000);
}
__device__ __forceinline__ uint2 buffer_load8(Record r, int lane_offset, int plane)
{
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(r, lane_offset, plane, 0);
    return make_uint2(v.x, v.y);
}
// (whole offsets in the vector register: with part of it in a scalar one the range check is not of the sum)
__device__ __forceinline__ uint2 buffer_load8_once(Record r, uint32_t offset)
{
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)offset, 0, 2 /* nt */);
    return make_uint2(v.x, v.y);
}
__device__ __forceinline__ uint32_t buffer_load4_once(Record r, uint32_t offset) { return __builtin_amdgcn_raw_buffer_load_b32(r, (int)offset, 0, 2 /* nt */); }
__device__ __forceinline__ uint4 buffer_load16_once(Record r, int lane_offset, int plane)   // non-temporal, as load_once
{
    const uint4v v = __builtin_amdgcn_raw_buffer_load_b128(r, lane_offset, plane, 2 /* nt */);
    return make_uint4(v.x, v.y, v.z, v.w);
}
// Index (16-byte chunks) of part 0 of this lane's K codes in the record's code plane, and how far on part i is.
template <int BITS, bool KC> __device__ __forceinline__ int kcode_chunk(int lane)
{
    const int r16 = lane & 15, q4 = lane >> 4;
    if constexpr (KC && BITS == 2) return (q4 >> 1) * 16 + r16;
    // k-slots 0..15 of an MFMA are the first token set (tile 2*blk), 16..31 the second (tile 2*blk + 1); a lane
    // holds eight channels: octet q4 & 1 of half group hg; i = blk*2 + hg
    return BITS == 4 ? (q4 >> 1) * 64 + (q4 & 1) * 16 + r16 : (q4 >> 1) * 32 + r16;
}
template <int BITS, bool KC> constexpr int kcode_part(int i)
{
    if (KC && BITS == 2) return i * 32;   // tile i
    return BITS == 4 ? (i >> 1) * 128 + (i & 1) * 32 : (i >> 1) * 64 + (i & 1) * 16;
}
// The loads of one record come in two parts, so that each can be issued as soon as the registers it lands in are
// free: the metadata planes and the K codes, and the V codes.
template <int BITS, bool KC> __device__ __forceinline__ void load_page_k(PageRegs<BITS> &pr, Record rec, int lane)
{
    using R = Rec<BITS>;
    pr.ksc = buffer_load8(rec, lane * 8, R::kKScale);
    pr.vsc = buffer_load8(rec, lane * 8, R::kVScale);
    pr.vzc = buffer_load8(rec, lane * 8, R::kVZero);
    pr.kzc = buffer_load8(rec, lane * 8, R::kKZero);
    const int at = kcode_chunk<BITS, KC>(lane) * 16;
#pragma unroll
    for (int i = 0; i < 4; ++i) pr.kw[i] = buffer_load16_once(rec, at, R::kKCodes + 16 * kcode_part<BITS, KC>(i));
}
template <int BITS> __device__ __forceinline__ void load_page_v(PageRegs<BITS> &pr, Record rec, int lane)
{
    using R = Rec<BITS>;
#pragma unroll
    for (int i = 0; i < BITS; ++i) pr.vw[i] = buffer_load16_once(rec, lane * 16, R::kVCodes + 1024 * i);   // chunk 64 i + lane
}
// Lane constants of the page loop.
struct LaneConst {
    float F;              // 2^(24 - E): undoes the subnormal position and the power-of-two normalisation of q
    float kappa;          // sm_scale * log2(e)
    uint32_t vmul01, vmul23;   // fp16 pairs of the staging factor of the V scale, 2^(kVExp - pos)
    int zp_idx[2];        // chunk of Lds::pv with this lane's B operand of the zero-point MFMA, per 32-token block
    int vs_idx;           // 8-byte half chunk of Lds::pv with the staged V scales of (block 0, group 0) of this lane's four tokens
    int tok0;             // two token sets: first token of this lane's four within a 32-token block
    int qy_ent;           // ... entry of this lane in a q operand of the QK^T MFMAs (or one of the two zero entries)
    int qc_ent;           // per-channel INT2 keys: entry of this lane among those of a group
    float zmul;           // per-channel INT2 keys: 2^-24 in head columns 0..7, 0 in columns 8..15
};

// One page.  `after_qk` runs once the K codes, K zeros and metadata registers of `pr` are dead, `after_pv`
// once the V codes are: the caller reloads them there for the next page.
template <int BITS, bool KC, class AfterQK, class AfterPV>
__device__ __forceinline__ void compute_page(const PageRegs<BITS> &pr, int n_valid, int lane,
                                             half8 qz, const LaneConst &lc, WaveState &st, Lds<KC> &lds,
                                             AfterQK after_qk, AfterPV after_pv)
{
    constexpr bool kPerChannel = KC && BITS == 2;   // INT2 keys quantised per channel over 32-token blocks
    const int r16 = lane & 15, q4 = lane >> 4;
    const bool partial = n_valid < kPageTokens;   // wave-uniform: only the last page of a width can be partly filled

    // ---- stage metadata in LDS --------------------------------------------
    uint2 kzv[2] = {{0u, 0u}, {0u, 0u}};   // K zeros of this lane's MFMA row per 32-token block (two token sets)
    (void)kzv;
    {
        uint2 vsc = pr.vsc, vzc = pr.vzc;
        if (partial) {
            // Tokens at or beyond n_valid (never-written slots) are masked by count, never by content:
            // their logits become -inf below (so P = 0) and their V scale and V zero become 0 here, so
            // the products with P = 0 cannot be NaN.
            // this lane holds plane entries 4*lane .. 4*lane+3: chunk lane/2, slots 4*(lane&1) + 0..3
            const int chunk = lane >> 1, blk = chunk >> 4, quad = (chunk >> 2) & 3, jb = 4 * (lane & 1);
            const int t0 = 32 * blk + 16 * (jb >> 2) + 4 * quad;   // tokens t0 .. t0+3
            const uint32_t m01 = (t0 < n_valid ? 0xffffu : 0u) | (t0 + 1 < n_valid ? 0xffff0000u : 0u);
            const uint32_t m23 = (t0 + 2 < n_valid ? 0xffffu : 0u) | (t0 + 3 < n_valid ? 0xffff0000u : 0u);
            vsc.x &= m01; vsc.y &= m23; vzc.x &= m01; vzc.y &= m23;
        }
        if constexpr (kPerChannel) {
            // the two key metadata planes as stored: fp16 [block][128 channel positions]; lanes 0..31 hold block 0.
            // A block that was never written (a half-filled page) is masked by count like everything else: whatever
            // its planes hold is neither used nor reported as a saturated scale.
            const bool dead = partial && 32 * (lane >> 5) >= n_valid;
            const uint2 ks = dead ? make_uint2(0u, 0u) : pr.ksc, kz = dead ? make_uint2(0u, 0u) : pr.kzc;
            const uint32_t k01 = pk_min(ks.x, kKcClamp), k23 = pk_min(ks.y, kKcClamp);
            st.sat |= (k01 ^ ks.x) | (k23 ^ ks.y);
            reinterpret_cast<uint2 *>(lds.kc_scale())[lane] = make_uint2(k01, k23);
            reinterpret_cast<uint2 *>(lds.kc_zero())[lane] = kz;
        } else {
            const half2_t a = __builtin_bit_cast(half2_t, pr.ksc.x), b = __builtin_bit_cast(half2_t, pr.ksc.y);
            // K scale * F as fp32 [block][group][token of the block]: a lane reads the scales of its four tokens for
            // one group with one 16-byte read
            {
                float *kst = lds.ks + (lane >> 5) * 128 + (lane & 31);
                kst[0] = fmaf((float)a[0], lc.F, 0.0f);   // (one mixed-precision FMA converts and scales)
                kst[32] = fmaf((float)a[1], lc.F, 0.0f);
                kst[64] = fmaf((float)b[0], lc.F, 0.0f);
                kst[96] = fmaf((float)b[1], lc.F, 0.0f);
            }
            // K zeros: lane (r, q4) takes those of token 32*blk + 16*(q4 >> 1) + r, which lane number that token holds.
            // An MFMA row holds a token of either set: a never-written token's zero-point (any bit pattern) would
            // meet the zeros of the other set's columns in the same row and could make them NaN.
            const uint2 kzm = partial && lane >= n_valid ? make_uint2(0u, 0u) : pr.kzc;
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                const int src = 4 * (32 * blk + 16 * (q4 >> 1) + r16);
                kzv[blk] = make_uint2((uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)kzm.x),
                                      (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)kzm.y));
            }
        }
        // V side, this lane's four (token, group) entries: the staged scale and the zero plane as stored
        {
            const uint32_t m01 = pk_mul(vsc.x, lc.vmul01), m23 = pk_mul(vsc.y, lc.vmul23);
            const uint32_t s01 = pk_min(m01, kVsClamp), s23 = pk_min(m23, kVsClamp);
            st.sat |= (s01 ^ m01) | (s23 ^ m23);
            reinterpret_cast<uint2 *>(lds.pv)[2 * kPvS + lane] = make_uint2(s01, s23);
            reinterpret_cast<uint2 *>(lds.pv)[2 * kPvZ + lane] = vzc;
        }
    }
    lds_order();

    // ---- QK^T: S[blk][i] = q . k_hat (unscaled) of token 32*blk + 16*(r16 >> 3) + 4*q4 + i for the head of column
    // r16 (two token sets); the per-channel path works on the four 16-token tiles first and folds them at its end
    floatx4 S[4];
    if constexpr (kPerChannel) {
        // score = sum_c (q_c s_c) code + sum_c q_c z_c with s, z of the token's block.  q s is formed per block
        // in two fp16 pieces, exactly (q has 8 significant bits, s 11) above the subnormals' grid: head columns 0..7 take
        // fp16(q s), columns 8..15 the remainder q s - fp16(q s); the columns of a head are added after the
        // MFMAs.  What is subtracted is formed from a q that is zero in the hi columns.
        const uint32_t lo_cols = r16 >= 8 ? 0xffffffffu : 0u;
        const uint32_t rot = (q4 & 1) ? 5u : 29u;   // this lane's 16 codes of a word are its upper / lower half
        // Zero term, sum_c q_c z_c of the two blocks: rows 0..7 of the A operand are block 0, rows 8..15 block 1.
        // Group by group, the LDS reads of the next group under way while a group is computed; four accumulation chains
        // (one per 16-token tile) and that of the zero term.
        struct Operands { uint4 qp, qo, zc, sc[2]; } op;
        auto fetch = [&](int g) {
            op.qo = lds.qo[g * 32 + lc.qc_ent];
            op.sc[0] = lds.kc_scale()[g * 4 + q4];
            op.sc[1] = lds.kc_scale()[(4 + g) * 4 + q4];
            op.qp = lds.qp[g * 32 + lc.qc_ent];
            op.zc = lds.kc_zero()[((r16 >> 3) * 4 + g) * 4 + q4];
        };
        floatx4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) S[e] = floatx4{0.f, 0.f, 0.f, 0.f};
        fetch(0);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            half8 b[2];
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                const uint4 sc = op.sc[blk], qo = op.qo;
                b[blk] = as_half8(pk_rem(qo.x, sc.x, pk_mul(qo.x & lo_cols, sc.x)), pk_rem(qo.y, sc.y, pk_mul(qo.y & lo_cols, sc.y)),
                                  pk_rem(qo.z, sc.z, pk_mul(qo.z & lo_cols, sc.z)), pk_rem(qo.w, sc.w, pk_mul(qo.w & lo_cols, sc.w)));
            }
            z = mfma(as_half8(op.zc.x, op.zc.y, op.zc.z, op.zc.w), as_half8(op.qp.x, op.qp.y, op.qp.z, op.qp.w), z);
            if (g < 3) fetch(g + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t wg = g == 0 ? pr.kw[e].x : g == 1 ? pr.kw[e].y : g == 2 ? pr.kw[e].z : pr.kw[e].w;
                // fields at bits 4:3, 6:5, 8:7, 10:9 of each half: q s spans more binades than q, and
                // the matrix core drops product bits that fall below its alignment window
                const uint32_t ws = __builtin_amdgcn_alignbit(wg, wg, rot);   // w >> 5 or w << 3, stray bits fall outside the masks
                const half8 a = as_half8(ws & 0x00180018u, ws & 0x00600060u, ws & 0x01800180u, ws & 0x06000600u);
                S[e] = mfma(a, b[e >> 1], S[e]);
            }
        }
        // every row of a block's half holds the same sum; lanes 0..31 hold that of block 0, lanes 32..63 that of block 1
        const float zmine = z[0] * lc.zmul;   // to the unit of the code products, hi columns only
        const float zother = __shfl_xor(zmine, 32);
        const float zb[2] = {lane < 32 ? zmine : zother, lane < 32 ? zother : zmine};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i) S[e][i] += zb[e >> 1];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int i = 0; i < 4; ++i) S[e][i] += row_ror8(S[e][i]);   // the two pieces of q s: columns h and h + 8
            asm volatile("" : "+v"(S[e]));
        }
        // Both column halves now hold the logits of all four tiles.  From here on the page is treated as with
        // per-token keys: columns 0..7 go on with tile 2*blk, columns 8..15 with tile 2*blk + 1 (two token sets), so
        // that exponentials and weight pieces are formed once per (token, head).
        if (r16 >= 8) { S[0] = S[1]; S[2] = S[3]; }
        S[1] = S[2];
        __builtin_amdgcn_sched_barrier(0);
    } else {
        // Per-token groups.  The eight heads fill only half of the 16 MFMA columns, so the columns carry two
        // token sets: rows r of a 32-token block are token 32*blk + r in columns 0..7 and token 32*blk + 16 + r in
        // columns 8..15.  An MFMA contracts 16 channels (half a group) of both sets: k-slots 0..15 hold the
        // codes of the first token, 16..31 those of the second, and the B operand holds q in the matching half
        // of its k-slots and zeros in the other.  All that follows the MFMAs (K scale, exponentials, weight
        // pieces) is then done once per (token, head).
        const uint4 *qy = lds.qo;
        floatx4 s[2];
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            const half8 za = as_half8(kzv[blk].x, kzv[blk].y, kzv[blk].x, kzv[blk].y);
            s[blk] = mfma(za, qz, floatx4{0.f, 0.f, 0.f, 0.f});   // zero-point term
        }
        // group by group, both 32-token blocks against one read of the q operand: two independent MFMA chains
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            floatx4 p[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int hg = 0; hg < 2; ++hg) {
                const uint4 qb4 = qy[(g * 2 + hg) * kQyStride + lc.qy_ent];
                const half8 qb = as_half8(qb4.x, qb4.y, qb4.z, qb4.w);
#pragma unroll
                for (int blk = 0; blk < 2; ++blk) {
                    const uint4 kw = pr.kw[blk * 2 + hg];
                    const uint32_t w = g == 0 ? kw.x : g == 1 ? kw.y : g == 2 ? kw.z : kw.w;
                    half8 a;
                    if (BITS == 4) {
                        const uint32_t w8 = w >> 8;
                        a = as_half8(w & 0x000f000fu, w & 0x00f000f0u, w8 & 0x000f000fu, w8 & 0x00f000f0u);
                    } else {
                        // this lane's 8 codes of the word are its upper or lower half; the rotate leaves the fields at bits
                        // 4:3, 6:5, 8:7, 10:9 of each half (towards the top of the fp16 mantissa, as for V: the matrix core
                        // drops product bits below its alignment window), stray bits fall outside the masks
                        const uint32_t ws = __builtin_amdgcn_alignbit(w, w, (q4 & 1) ? 5u : 29u);
                        a = as_half8(ws & 0x00180018u, ws & 0x00600060u, ws & 0x01800180u, ws & 0x06000600u);
                    }
                    p[blk] = mfma(a, qb, p[blk]);
                }
            }
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                const float4 sc = reinterpret_cast<const float4 *>(lds.ks)[(blk * 4 + g) * 8 + (lc.tok0 >> 2)];
                s[blk][0] = fmaf(sc.x, p[blk][0], s[blk][0]);
                s[blk][1] = fmaf(sc.y, p[blk][1], s[blk][1]);
                s[blk][2] = fmaf(sc.z, p[blk][2], s[blk][2]);
                s[blk][3] = fmaf(sc.w, p[blk][3], s[blk][3]);
            }
        }
        S[0] = s[0];
        S[1] = s[1];
        asm volatile("" : "+v"(S[0]), "+v"(S[1]));   // the scaled sums are formed here, not sunk next to their first use
        __builtin_amdgcn_sched_barrier(0);
    }
    // What the PV phase reads from LDS, requested ahead of the softmax: columns 0..3 of the zero-point MFMA are the V zeros of
    // the groups, column 4 ones; the staged V scales of this lane's own tokens.
    uint4 v_zero[2];
    uint2 v_scale[2][4];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        v_zero[blk] = lds.pv[lc.zp_idx[blk]];
#pragma unroll
        for (int g = 0; g < 4; ++g) v_scale[blk][g] = reinterpret_cast<const uint2 *>(lds.pv)[lc.vs_idx + 32 * blk + 2 * g];
    }
    after_qk();
    constexpr int kS = 2;   // logit registers of this lane: its eight tokens of the page
    if (partial) {
#pragma unroll
        for (int e = 0; e < kS; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int t = 32 * e + lc.tok0 + i;
                S[e][i] = t < n_valid ? S[e][i] : -INFINITY;
            }
    }

    // ---- online softmax with a lazily updated reference maximum ------------
    // The cheap test looks only at this lane's own logits; the column maximum is formed across
    // lanes only when some lane needs a new reference.
    float mx = fmaxf(fmaxf(S[0][0], S[0][1]), fmaxf(S[0][2], S[0][3]));
#pragma unroll
    for (int e = 1; e < kS; ++e) mx = fmaxf(fmaxf(mx, S[e][0]), fmaxf(fmaxf(S[e][1], S[e][2]), S[e][3]));
    if (__any(mx * lc.kappa > st.m_ref + kTau)) {
        // the other token set of the head, then the other rows of 16 lanes (every item comes here on its first page; through
        // LDS, two round trips and 14 instructions more, 16 contexts of 97 to 6011 tokens took 14.1 us, now 13.85, 8 contexts of
        // 2000 to 16000 19.2, now 18.75)
        mx = fmaxf(mx, row_ror8(mx));
        mx = swap_max(__builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false));
        mx = swap_max(__builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false));
        const float m_new = fmaxf(st.m_ref, mx * lc.kappa);
        const float alpha = m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(st.m_ref - m_new);
        st.m_ref = m_new;
        if (q4 == 0) lds.alpha[r16] = alpha;   // columns r16 and r16 ^ 8 hold the same head
        lds_order();
        const float4 al = reinterpret_cast<const float4 *>(lds.alpha)[q4 & 1];   // rows 4*q4 .. 4*q4+3 -> heads (4*q4 + i) & 7
        const floatx4 av = {al.x, al.y, al.z, al.w};
#pragma unroll
        for (int j = 0; j < 8; ++j) st.acc[j >> 2][j & 3] *= av;
        st.zp *= av;
    }
    const float nmref = (float)kPExp - (st.m_ref == -INFINITY ? 0.0f : st.m_ref);
    // W = P * 2^kPExp in two fp16 pieces (leading 11 bits truncated, then the next 11), for this lane's own four tokens of
    // each 32-token block (two token sets: tile 2*blk in columns 0..7, 2*blk + 1 in columns 8..15)
    uint32_t wh[2][2], wl[2][2];
#pragma unroll
    for (int e = 0; e < kS; ++e) {
        float pv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) pv[i] = __builtin_amdgcn_exp2f(fmaf(S[e][i], lc.kappa, nmref));
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            wh[e][k] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(pv[2 * k], pv[2 * k + 1]));
            wl[e][k] = __builtin_bit_cast(
                uint32_t, __builtin_amdgcn_cvt_pkrtz(residual<0>(wh[e][k], -1.0f, pv[2 * k]), residual<1>(wh[e][k], -1.0f, pv[2 * k + 1])));
        }
    }

    // ---- PV ------------------------------------------------------------------
    auto weights = [&](int blk, int g) {
        // a = W * scale in two fp16 pieces: hi = fp16(W_hi s), lo = W_lo s + the exact remainder of the hi product
        const uint32_t vsr[2] = {v_scale[blk][g].x, v_scale[blk][g].y};
        uint32_t ah[2], al[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) ah[k] = pk_mul(wh[blk][k], vsr[k]);
#pragma unroll
        for (int k = 0; k < 2; ++k) al[k] = pk_rem(wh[blk][k], vsr[k], ah[k]);
#pragma unroll
        for (int k = 0; k < 2; ++k) al[k] = pk_fma(wl[blk][k], vsr[k], al[k]);
        return piece_rows(ah, al);
    };
    // Codes as fp16 subnormals, fields shifted towards the top of the mantissa (INT2: bits 4:3, 6:5, 8:7, 10:9 of each half;
    // INT4: bits 6:3 and 10:7): the matrix core aligns the products of a lane's eight k-slots to the largest exponent
    // *field* and drops what falls below a fixed window, so leading zeros of a subnormal cost precision.  Bit 10 is the
    // lowest exponent bit: fp16 is linear through the first binade, so a field may reach it.  The slot's power of two is
    // undone in the staged V scale.  Bits of the other half that a shift brings in fall outside the masks.
    auto codes = [&](int blk, int half, int comp) {
        const uint4 v = BITS == 4 ? pr.vw[blk * 2 + half] : pr.vw[half];
        const uint32_t w = comp == 0 ? v.x : comp == 1 ? v.y : comp == 2 ? v.z : v.w;
        if (BITS == 4) {
            const uint32_t wa = w << 3, wb = w >> 5;
            return as_half8(wa & 0x00780078u, wa & 0x07800780u, wb & 0x00780078u, wb & 0x07800780u);
        } else {
            const uint32_t ws = blk ? (w >> 5) : (w << 3);
            return as_half8(ws & 0x00180018u, ws & 0x00600060u, ws & 0x01800180u, ws & 0x06000600u);
        }
    };
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        // zero-point term and denominator, both pieces into rows 0..7 (rows 8..15 are never read)
        const half8 vz = as_half8(v_zero[blk].x, v_zero[blk].y, v_zero[blk].z, v_zero[blk].w);
        st.zp = mfma(as_half8(wh[blk][0], wh[blk][1], ror8_u32(wh[blk][0]), ror8_u32(wh[blk][1])), vz, st.zp);
        st.zp = mfma(as_half8(wl[blk][0], wl[blk][1], ror8_u32(wl[blk][0]), ror8_u32(wl[blk][1])), vz, st.zp);
    }
    // (block, group) by (block, group), the weights of the next one made ahead of the MFMAs of this one
    half8 a = weights(0, 0);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const int blk = t >> 2, g = t & 3, half = g >> 1, comp = 2 * (g & 1);
        const half8 b0 = codes(blk, half, comp), b1 = codes(blk, half, comp + 1);
        const half8 next = t < 7 ? weights((t + 1) >> 2, (t + 1) & 3) : a;
        st.acc[half][comp] = mfma(a, b0, st.acc[half][comp]);
        st.acc[half][comp + 1] = mfma(a, b1, st.acc[half][comp + 1]);
        a = next;
    }
    after_pv();
}

// What stays the same for every page of a work item.
struct ItemCtx {
    const uint8_t *__restrict__ pool;
    const uint8_t *__restrict__ bit_map;
    const int32_t *__restrict__ pages;   // the sequence's page list
    int pb, pe;                          // the item's range of it
    int np2, np4;                        // pages of the sequence: the INT2 pages come first
    int last2, last4;                    // valid tokens of the last page of either width
    int kvh, n_kv_heads, n_pages_int2, n_pages_total, lane;
    int32_t *status;
};
// The pages of an item, 64 at a time in registers: lane l holds list position base + l.  The page id, the check against
// its pool, the bit_map entry, the address arithmetic and the token count of a page cost one lane each, once, instead
// of two loads and some thirty scalar instructions on the way from page to page.
struct PageBatch {
    int base;
    uint32_t at;   // where this wavefront's record of the page starts in the pool, in units of kRecordUnit
    int nv;        // number of valid tokens; 0: the page is run with every token masked
    uint32_t bm;
};
constexpr int kRecordUnitLog2 = 11;   // record sizes and arena sizes are multiples of it
static_assert(Rec<2>::kBytes % (1 << kRecordUnitLog2) == 0 && Rec<4>::kBytes % (1 << kRecordUnitLog2) == 0, "record unit");
// Requests the ids of positions base .. base + 63.
__device__ __forceinline__ int batch_ids(const ItemCtx &cx, PageBatch &pb, int base)
{
    pb.base = base;
    return cx.pages[base + cx.lane < cx.pe ? base + cx.lane : cx.pe - 1];
}
// Checks the ids.  A page id outside its pool cannot be addressed: it is flagged, a valid page is read instead and
// none of its tokens count.  Requests the bit_map entries.
__device__ __forceinline__ void batch_check(const ItemCtx &cx, PageBatch &pb, int page)
{
    const int pi = pb.base + cx.lane;
    const bool is2 = pi < cx.np2;
    const int lo = is2 ? 0 : cx.n_pages_int2, hi = is2 ? cx.n_pages_int2 : cx.n_pages_total;
    const bool ok = page >= lo && page < hi;
    if (!ok && pi < cx.pe && cx.status)
        atomicOr(cx.status, page < 0 || page >= cx.n_pages_total ? TKV_STATUS_PAGE_RANGE : TKV_STATUS_BITMAP_MISMATCH);
    pb.nv = ok ? (pi == cx.np2 - 1 ? cx.last2 : pi == cx.np2 + cx.np4 - 1 ? cx.last4 : kPageTokens) : 0;
    // (lanes beyond the item repeat its last page, whose width need not be theirs; they are never used)
    const int at = ok ? page : (lo < cx.n_pages_total ? lo : 0);
    // (pools below 8 TB: 32 bits)
    const uint32_t rec = (uint32_t)(at < cx.n_pages_int2 ? at : at - cx.n_pages_int2) * (uint32_t)cx.n_kv_heads + (uint32_t)cx.kvh;
    constexpr uint32_t kUnits2 = Rec<2>::kBytes >> kRecordUnitLog2, kUnits4 = Rec<4>::kBytes >> kRecordUnitLog2;
    pb.at = at < cx.n_pages_int2 ? rec * kUnits2 : (uint32_t)cx.n_pages_int2 * (uint32_t)cx.n_kv_heads * kUnits2 + rec * kUnits4;
    pb.bm = cx.bit_map[at];
}
// A page that was never written, or written at the other width, counts no tokens.
__device__ __forceinline__ void batch_finish(const ItemCtx &cx, PageBatch &pb)
{
    const int pi = pb.base + cx.lane;
    const bool written = pb.bm == (pi < cx.np2 ? 2u : 4u);
    if (!written && pb.nv > 0 && pi < cx.pe && cx.status) atomicOr(cx.status, TKV_STATUS_BITMAP_MISMATCH);
    pb.nv = written ? pb.nv : 0;
}
__device__ __forceinline__ void batch_seek(const ItemCtx &cx, PageBatch &pb, int pi)
{
    if (__builtin_expect(pi - pb.base >= 64, 0)) {
        const int page = batch_ids(cx, pb, pi);
        batch_check(cx, pb, page);
        batch_finish(cx, pb);
    }
}
__device__ __forceinline__ int batch_valid(const PageBatch &pb, int pi) { return __builtin_amdgcn_readlane(pb.nv, pi - pb.base); }
template <int BITS> __device__ __forceinline__ Record batch_record(const ItemCtx &cx, const PageBatch &pb, int pi, bool wanted)
{
    const uint64_t at = (uint32_t)__builtin_amdgcn_readlane((int)pb.at, pi - pb.base);
    return record_at<BITS>(cx.pool + (at << kRecordUnitLog2), wanted);
}

// The pages [pi, pe) of one width.  `pr` holds (or has requested) the record of page pi.
template <int BITS, bool KC>
__device__ __forceinline__ void run_pages(const ItemCtx &cx, PageBatch &batch, int pi, int pe, PageRegs<BITS> &pr, half8 qz, LaneConst lc,
                                          WaveState &st, Lds<KC> &lds)
{
    const int lane = cx.lane;
    // A V code enters the MFMA as code * 2^(pos - 24), pos = lowest bit of its field after the unpack shift; the
    // staged scale of the slot carries 2^(kVExp - pos).  This lane stages plane entries 4*lane .. 4*lane+3 =
    // k-slots 4*(lane&1) + 0..3, i.e. operand registers 2*(lane&1) (first pair) and 2*(lane&1) + 1 (second pair).
    {
        const int k0 = 2 * (lane & 1);
        const int p01 = BITS == 4 ? 3 : 3 + 2 * k0, p23 = BITS == 4 ? 7 : 5 + 2 * k0;
        const uint32_t h01 = (uint32_t)(15 + kVExp - p01) << 10, h23 = (uint32_t)(15 + kVExp - p23) << 10;
        lc.vmul01 = h01 | (h01 << 16);
        lc.vmul23 = h23 | (h23 << 16);
    }
    // One register set: every part of the next record is requested as soon as the registers it lands in
    // are dead, so about one page per wavefront is in flight while the current one is computed.
    int nv = batch_valid(batch, pi);
    int prio_end = 0;   // list position at which the priority changes next
    const int item_pages = cx.pe - cx.pb;
    for (; pi < pe; ++pi) {
        // Wavefronts that share a SIMD are served oldest first; left alone, the oldest finishes long before
        // the others and the SIMD ends its work with one wavefront.  The priority follows the share of the
        // item still to do (three quarters and more, a half, a quarter, less), so the wavefronts of a SIMD advance together.
        if (__builtin_expect(pi >= prio_end, 0)) {
            const int left4 = 4 * (cx.pe - pi) - 1;
            int q;
            if (left4 >= 3 * item_pages) { q = 3; __builtin_amdgcn_s_setprio(3); }
            else if (left4 >= 2 * item_pages) { q = 2; __builtin_amdgcn_s_setprio(2); }
            else if (left4 >= item_pages) { q = 1; __builtin_amdgcn_s_setprio(1); }
            else { q = 0; __builtin_amdgcn_s_setprio(0); }
            // the first position with 4 * (pe - position) - 1 < q * item_pages
            prio_end = cx.pe - ((q * item_pages) >> 2);
        }
        // The last page asks for nothing (an empty record).
        const bool wanted = pi + 1 < pe;
        const int next = wanted ? pi + 1 : pi;
        batch_seek(cx, batch, next);
        const Record rec = batch_record<BITS>(cx, batch, next, wanted);
        const int nv_next = batch_valid(batch, next);
        auto after_qk = [&]() {
            __builtin_amdgcn_sched_barrier(0);   // keep the reloads below the last use of the registers they overwrite
            load_page_k<BITS, KC>(pr, rec, lane);
        };
        auto after_pv = [&]() {
            __builtin_amdgcn_sched_barrier(0);
            load_page_v<BITS>(pr, rec, lane);
        };
        // a page with no valid token still runs (every token masked by count): no second path through the loop
        compute_page<BITS, KC>(pr, nv, lane, qz, lc, st, lds, after_qk, after_pv);
        nv = nv_next;
    }
}

// The rows of a partial: accumulators and (m, l) pairs of the R heads that follow head h0 in a slot.  Stores beyond them are dropped.
// Written through the L2: with the partials left dirty there, the merge began that much later.  Before | now, us a call: 16 contexts of
// 97 to 6011 tokens 12.45 | 11.95, 4 x 102400 on one head 18.1 | 17.5, four-layer step 74.7 | 67.8, of 23 more shapes five of 9 to 100 us
// 1.08 to 1.11 times as fast, the others .99 to 1.03; 36 shapes of about as many wavefronts as run at once and eight query heads each,
// 20 to 193 us, .997 to 1.05.  (Non-temporal stores .97 to 1.05 of it, .88 on some; both at once .88 to 1.06.)
struct PartialRows {
    Record acc, ml;
    __device__ __forceinline__ PartialRows(float *acc_ws, float *ml_ws, int slot, int n_q_heads, int h0, int R)
    {
        const size_t row = (size_t)slot * n_q_heads + h0;
        acc = __builtin_amdgcn_make_buffer_rsrc(acc_ws + row * kHeadDim, 0, R * kHeadDim * 4, 0x00027000);
        ml = __builtin_amdgcn_make_buffer_rsrc(ml_ws + row * 2, 0, R * 8, 0x00027000);
    }
    __device__ __forceinline__ void put(int head, int c4, float4 v) const { store_through(acc, head * (kHeadDim * 4) + c4 * 16, v); }
    __device__ __forceinline__ void put(int head, float2 v) const { store_through(ml, head * 8, v); }
};
// The kernels take their arguments as one struct: the runtime looks every pointer argument up on the way to a launch, and small calls
// wait for their two launches (eighteen arguments 2.7 us, a struct of them 2.4, on a slower host 3.8 and 3.3; step of five layers over
// 19 pages 64 -> 57 us, tiny calls 1 to 7 %).  The bodies are functions with parameters of their own, which the compiler then
// knows apart: with the members read where they are used two registers were spilled (four-layer step 75.2 -> 76.2).
struct DecodeArgs {
    const uint8_t *pool;
    const uint8_t *bit_map;
    const uint16_t *q;
    const int32_t *page_indptr;
    const int32_t *page_ids;
    const int32_t *n_tok_int2;
    const int32_t *n_tok_int4;
    const int32_t *items;
    int n_items;
    int batch;
    int n_kv_heads;
    int log2_r;
    int n_pages_int2;
    int n_pages_int4;
    float kappa;
    float *acc_ws;
    float *ml_ws;
    int32_t *status;
};
// KC: the INT2 keys of the pool are quantised per channel over 32-token blocks (Sec. 3.2.1).
// The grid is (kv heads, items): the workgroups of an item are launched one behind the other, without a division to
// find the item.
template <bool KC>
__device__ __forceinline__ void decode_item(
    const uint8_t *__restrict__ pool, const uint8_t *__restrict__ bit_map, const uint16_t *__restrict__ q,
    const int32_t *__restrict__ page_indptr, const int32_t *__restrict__ page_ids,
    const int32_t *__restrict__ n_tok_int2, const int32_t *__restrict__ n_tok_int4,
    const int32_t *__restrict__ items, int n_items, int batch, int n_kv_heads, int log2_r, int n_pages_int2, int n_pages_int4,
    float kappa, float *__restrict__ acc_ws, float *__restrict__ ml_ws, int32_t *status)
{
    __shared__ Lds<KC> lds;
    const int lane = threadIdx.x, r16 = lane & 15, q4 = lane >> 4;
    // Everything of a level of the chain arguments -> item -> counts -> page ids at once: fetched where each is first used,
    // the arguments and counts alone are six round trips in a row.  (16 contexts of 97 to 6011 tokens 14.45 -> 14.1 us, 4 x
    // 102400 on one head 18.5 -> 18.2, 8 contexts of 2000 to 16000 20.1 -> 19.3, four-layer step 79.5 -> 78.1.)
    asm volatile("" :: "s"(pool), "s"(bit_map), "s"(q), "s"(page_indptr), "s"(page_ids), "s"(n_tok_int2), "s"(n_tok_int4), "s"(items),
                 "s"(n_items), "s"(batch), "s"(n_kv_heads), "s"(log2_r), "s"(n_pages_int2), "s"(n_pages_int4), "s"(acc_ws), "s"(ml_ws), "s"(status),
                 "s"(gridDim.y));
    const int item = blockIdx.y + blockIdx.z * gridDim.y, kvh = blockIdx.x;
    if (item >= n_items) return;
    const int R = 1 << log2_r, n_q_heads = n_kv_heads << log2_r;
    // The partial of this item goes to slot items[4*item + 3] of the workspace: items are listed in launch order,
    // the slots of a sequence are contiguous (the merge reads them by sequence).
    const ConstWords words = (ConstWords)(items + 4 * (size_t)item);
    const int seq = words[0], item_pb = words[1], item_pe = words[2], slot = words[3];
    asm volatile("" :: "s"(seq), "s"(item_pb), "s"(item_pe), "s"(slot));
    const bool slot_ok = slot >= 0 && slot < n_items, seq_ok = seq >= 0 && seq < batch;
    const int sq = __builtin_amdgcn_readfirstlane((uint32_t)seq < (uint32_t)batch ? seq : 0);
    const int n2 = ((ConstWords)n_tok_int2)[sq], n4 = ((ConstWords)n_tok_int4)[sq], list0 = ((ConstWords)page_indptr)[sq], list1 = ((ConstWords)page_indptr)[sq + 1];
    asm volatile("" :: "s"(n2), "s"(n4), "s"(list0), "s"(list1));
    auto write_empty = [&]() {
        for (int h = 0; h < R; ++h) {
            const size_t ph = (size_t)slot * n_q_heads + kvh * R + h;
            reinterpret_cast<float2 *>(acc_ws + ph * kHeadDim)[lane] = make_float2(0.0f, 0.0f);
            if (lane == 0) reinterpret_cast<float2 *>(ml_ws)[ph] = make_float2(-INFINITY, 0.0f);
        }
    };
    if (!seq_ok || !slot_ok) {
        // malformed item: an empty partial (m = -inf, l = 0), which the merge ignores, and a status bit; with a slot
        // outside the workspace nothing can be written, and whoever owns the slot it should have named reads what
        // the workspace held before
        if (slot_ok) write_empty();
        if (status && lane == 0) atomicOr(status, TKV_STATUS_BAD_ITEM);
        return;
    }
    const int np2 = (n2 + kPageTokens - 1) / kPageTokens, np4 = (n4 + kPageTokens - 1) / kPageTokens;
    const int seq_pages = list1 - list0;
    const int np_all = np2 + np4 < seq_pages ? np2 + np4 : seq_pages;
    const int pb = item_pb > 0 ? item_pb : 0;
    const int pe = item_pe < np_all ? item_pe : np_all;
    const int32_t *pages = page_ids + list0;
    const int n_pages_total = n_pages_int2 + n_pages_int4;
    // INT2 pages of the range, then INT4 pages: each page runs one dequantisation path
    const int e2 = pe < np2 ? pe : np2, b4 = pb > np2 ? pb : np2;
    bool has2 = pb < e2, has4 = b4 < pe;
    // tokens of a width whose pool has no pages at all: nothing to read
    if ((has2 && n_pages_int2 == 0) || (has4 && n_pages_int4 == 0)) {
        int bits = TKV_STATUS_PAGE_RANGE;
        // (pages of the other pool among the first 64 are flagged as such, as they are where the pool has pages)
        if (has4 && n_pages_int4 > 0 && pb + lane < b4 && (uint32_t)pages[pb + lane] < (uint32_t)n_pages_total) bits |= TKV_STATUS_BITMAP_MISMATCH;
        if (status) atomicOr(status, bits);
        has2 = has2 && n_pages_int2 > 0;
        has4 = has4 && n_pages_int4 > 0;
    }
    const int first = has2 ? pb : b4;   // the first list position that is read: more than pb where there is no INT2 pool
    if (!(has2 || has4)) {   // an item without pages
        write_empty();
        return;
    }
    const ItemCtx cx = {pool, bit_map, pages, pb, pe, np2, np4, n2 - (np2 - 1) * kPageTokens, n4 - (np4 - 1) * kPageTokens,
                        kvh, n_kv_heads, n_pages_int2, n_pages_total, lane, status};
    PageBatch list = {first, 0, 0, 0};
    PageRegs<2> s2;
    PageRegs<4> s4;

    // What a wavefront of few pages does is a chain of loads (arguments -> item -> counts -> page ids and q -> record) and the
    // preparation of q.  The vector loads of a compute unit return in the order in which they were asked for: records that the
    // first wavefronts ask for early stand in front of the q and the page ids of the others.  So the first record is requested
    // when the exponents and sums of q are known, ahead of the operand tables (16 contexts of 97 to 6011 tokens, one page to a
    // wavefront, 15.4 us asked with the page ids, 14.7 here, 14.9 behind the tables; four-layer step 84.1, 81.8, 83.8), and its V
    // codes, which are needed last, behind them (step 75.8 -> 75.2, 4 x 102400 on one head 18.5 -> 18.3, 20 shapes of 1500 to
    // 9000 records .94 to 1.00, mean .985; with the first K metadata 76.3 and 18.5).  The tables for per-channel keys take longer
    // (.98 to 1.04): K and V together there.
    const int first_ids = batch_ids(cx, list, first);
    const uint16_t *q_head = q + ((size_t)seq * n_q_heads + kvh * R + ((lane >> 3) & (R - 1))) * kHeadDim;   // columns beyond R repeat heads
    QRegs qr;
    load_q(qr, q_head, lane);
    batch_check(cx, list, first_ids);

    float two_e;
    LaneConst lc;
    half8 qz;
    WaveState st;
    // ---- q: common power-of-two normalisation, group sums (no branches that depend on the lane, no 64-bit arithmetic) ----
    // (Called in the branch of the item's first width: in front of the branches, its registers live through both page loops
    // and are spilled, 16 short contexts 14.7 -> 15.2 us.)
    auto prepare_q = [&]() {
        const uint32_t d[8] = {qr.x[0].x, qr.x[0].y, qr.x[0].z, qr.x[0].w, qr.x[1].x, qr.x[1].y, qr.x[1].z, qr.x[1].w};
        // Largest exponent of the heads, from the bf16 bits: |x| as an integer, plus one in the exponent, which makes NaN and
        // infinities negative: they do not count (a head that holds one must not spoil the others)
        typedef short short2_t __attribute__((ext_vector_type(2)));
        short2_t big = {0, 0};
#pragma unroll
        for (int i = 0; i < 8; ++i) big = __builtin_elementwise_max(big, __builtin_bit_cast(short2_t, ((d[i] & 0x7fff7fffu) + 0x00800080u)));
        const int top = wave_max(big[0] > big[1] ? big[0] : big[1]);   // 0x80 where all are zero
        // 2^E with max|q| * 2^E in [2^14, 2^15) ([2^8, 2^9) with per-channel INT2 keys); E clamped so every factor stays a normal fp32
        int E = (KC ? kKcQExp : 15) - ((top >> 7) - 127);   // max|q| = m * 2^(exponent - 126), m in [0.5, 1)
        E = E > 100 ? 100 : (E < -100 ? -100 : E);
        if (top <= 0x80) E = 0;
        two_e = ldexpf(1.0f, E);
        lc.F = ldexpf(1.0f, 24 - E);
        lc.kappa = kappa;
        lc.vmul01 = lc.vmul23 = 0;
        lc.zmul = r16 >= 8 ? 0.0f : 0x1p-24f;
        lc.vs_idx = 2 * (kPvS + q4 * 4) + (r16 >> 3);
        lc.tok0 = 16 * (r16 >> 3) + 4 * q4;
        static_assert(kQyZero0 == 24 && kQyZero1 == 16, "entry 24 - 8 * sub holds the zeros of the lanes of octet sub");
        const int other_set = -(int)((r16 >> 3) != (q4 >> 1));
        lc.qy_ent = (((q4 & 1) * 8 + (r16 & 7)) & ~other_set) | ((kQyZero0 - 8 * (q4 & 1)) & other_set);
        lc.qc_ent = q4 * 8 + (r16 & 7);
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            lc.zp_idx[blk] = r16 < 4 ? kPvZ + (blk * 4 + q4) * 4 + r16 : (r16 == 4 ? kPvOne : kPvZero);
        }
        if (lane < 2) {
            const uint32_t c = lane == 1 ? 0x3c003c00u : 0u;
            lds.pv[kPvZero + lane] = make_uint4(c, c, c, c);
        }
        // The sums of q over this lane's two groups, in 32 bits: they meet zero-points of tens.  (From the staged q on the
        // matrix core, numbers far below the largest of their group or of the heads lose bits, and it is no faster.)  As
        // three fp16 pieces to LDS, [head][hi of the four groups, mid, lo], one by each of three lanes of a quad.  (A sum beyond
        // 65504 has no such pieces: NaN.)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float sum = ((bf16_lo(d[4 * j]) + bf16_hi(d[4 * j])) + (bf16_lo(d[4 * j + 1]) + bf16_hi(d[4 * j + 1]))) +
                        ((bf16_lo(d[4 * j + 2]) + bf16_hi(d[4 * j + 2])) + (bf16_lo(d[4 * j + 3]) + bf16_hi(d[4 * j + 3])));
            sum += row_dpp<0xB1>(sum);
            sum += row_dpp<0x4E>(sum);
            const _Float16 hi = (_Float16)sum;
            const float r1 = sum - (float)hi;
            const _Float16 mid = (_Float16)r1, lo = (_Float16)(r1 - (float)mid);
            const int piece = lane & 3;
            if (piece < 3) reinterpret_cast<_Float16 *>(lds.zl[lane >> 3])[4 * piece + 2 * j + ((lane >> 2) & 1)] = piece == 0 ? hi : (piece == 1 ? mid : lo);
        }
        lds_order();
        // Z-term B operand (two token sets: the k-slots of a column's own set carry the pieces, the others zeros):
        // slots 0..3 / 4..7 of the first octet = hi / mid pieces of the four group sums, slots 0..3 of the second
        // octet = lo pieces.  Masks and no branches.
        const uint4 z4 = reinterpret_cast<const uint4 *>(lds.zl[r16 & 7])[q4 & 1];
        const uint32_t own = (r16 >> 3) == (q4 >> 1) ? 0xffffffffu : 0u, first = (q4 & 1) ? 0u : own;
        qz = as_half8(z4.x & own, z4.y & own, z4.z & first, z4.w & first);
#pragma unroll
        for (int j = 0; j < 8; ++j) st.acc[j >> 2][j & 3] = floatx4{0.f, 0.f, 0.f, 0.f};
        st.zp = floatx4{0.f, 0.f, 0.f, 0.f};
        st.m_ref = -INFINITY;
        st.sat = 0;
    };

    if (has2) {
        prepare_q();
        __builtin_amdgcn_sched_barrier(0);
        const Record rec = batch_record<2>(cx, list, pb, true);
        load_page_k<2, KC>(s2, rec, lane);
        if constexpr (KC) load_page_v<2>(s2, rec, lane);
        __builtin_amdgcn_sched_barrier(0);
        build_q_operand<2, KC>(qr, two_e, lane, lds);
        if constexpr (!KC) {
            __builtin_amdgcn_sched_barrier(0);
            load_page_v<2>(s2, rec, lane);
            __builtin_amdgcn_sched_barrier(0);
        }
        batch_finish(cx, list);
        LaneConst lc2 = lc;
        if constexpr (KC) {
            lc2.kappa = lc.kappa * lc.F;   // the power of two that the K scale carries otherwise
        }
        lds_order();
        run_pages<2, KC>(cx, list, pb, e2, s2, qz, lc2, st, lds);
    }
    if (has4) {
        if (has2) {
            batch_seek(cx, list, b4);
            load_q(qr, q_head, lane);   // (not kept through the INT2 pages)
        } else {
            prepare_q();
            batch_finish(cx, list);
        }
        __builtin_amdgcn_sched_barrier(0);
        const Record rec = batch_record<4>(cx, list, b4, true);
        load_page_k<4, KC>(s4, rec, lane);
        if constexpr (KC) load_page_v<4>(s4, rec, lane);
        __builtin_amdgcn_sched_barrier(0);
        build_q_operand<4, KC>(qr, two_e, lane, lds);
        if constexpr (!KC) {
            __builtin_amdgcn_sched_barrier(0);
            load_page_v<4>(s4, rec, lane);
            __builtin_amdgcn_sched_barrier(0);
        }
        lds_order();
        run_pages<4, KC>(cx, list, b4, pe, s4, qz, lc, st, lds);
    }

    // ---- write the partial (m, l, acc) of this item ------------------------------
    if (status && __any(st.sat != 0) && lane == 0) atomicOr(status, TKV_STATUS_SCALE_SATURATED);
    // per head: columns 0..3 of zl = zero-point sums of the groups, 4 = denominator
    lds_order();
    if (q4 < 2 && r16 < 5)
#pragma unroll
        for (int i = 0; i < 4; ++i) lds.zl[4 * q4 + i][r16] = st.zp[i];
    if (q4 == 0 && r16 < 8) lds.alpha[r16] = st.m_ref;
    lds_order();
    const float unscale = ldexpf(1.0f, 24 - kVExp);
    // The accumulators go through an LDS tile [head][channel] so that every lane stores 16 bytes and a store
    // instruction covers two whole heads (a lane holds single channels of four heads).  The tile takes the start of
    // the LDS, which holds nothing the epilogue needs (page staging, q operands); rows are 16 bytes longer than a
    // head so that heads h and h + 4, written by the same instruction, fall on different banks.
    constexpr int kOutRow = kHeadDim + 4;
    static_assert(sizeof(lds.ks) + sizeof(lds.pv) + sizeof(lds.qo) >= 8 * kOutRow * sizeof(float), "the output tile must fit in what precedes zl and alpha in Lds");
    float *tile = reinterpret_cast<float *>(&lds);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int head = 4 * (q4 & 1) + i, half = q4 >> 1;   // lanes 0..31 go on with the lower channels, 32..63 with the upper
        const float2 zsum = *reinterpret_cast<const float2 *>(&lds.zl[head][2 * half]);
#pragma unroll
        for (int comp = 0; comp < 4; ++comp)
            tile[head * kOutRow + 64 * half + 16 * comp + r16] = fmaf(add_pieces(st.acc[0][comp][i], st.acc[1][comp][i]), unscale, comp < 2 ? zsum.x : zsum.y);
    }
    const PartialRows partial(acc_ws, ml_ws, slot, n_q_heads, kvh * R, R);
    if (lane < 8) partial.put(lane, make_float2(lds.alpha[lane], lds.zl[lane][4]));
    lds_order();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int head = 2 * k + (lane >> 5), c4 = lane & 31;
        partial.put(head, c4, reinterpret_cast<const float4 *>(tile + head * kOutRow)[c4]);
    }
}
template <bool KC>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 3))) void tkv_decode_kernel(DecodeArgs a)
{
    decode_item<KC>(a.pool, a.bit_map, a.q, a.page_indptr, a.page_ids, a.n_tok_int2, a.n_tok_int4, a.items, a.n_items, a.batch,
                    a.n_kv_heads, a.log2_r, a.n_pages_int2, a.n_pages_int4, a.kappa, a.acc_ws, a.ml_ws, a.status);
}

// D7: out = sum_i 2^(m_i - M) acc_i / sum_i 2^(m_i - M) l_i over the items of a sequence (Sec. 3.2.3: the
// splits are merged by online log-sum-exp).
// Two kernels: this one for batches of up to 128 items per sequence on average, the next for more.
//
// A workgroup of four wavefronts per (sequence, query head, 2 / VEC halves of the channels), a lane owns VEC channels.  Each
// wavefront takes a quarter of the items; lane l weighs item l, and an item's accumulators are one load of whole lines.
// What bounds it is latency (bytes alone would take 1 to 2 us): the chain is item list -> (m, l) pairs and accumulators of 32
// items at once -> weights -> sum -> one exchange through LDS, which a sequence of few items does without.
// Against a kernel of the next one's kind that it replaced (a running maximum per item, 8 items in flight per workgroup), us
// alone, 64 heads, sequences x items each: 8 x 4 2.6 -> 2.25, 32 x 12 4.6 -> 4.4, 8 x 24 4.4 -> 3.4, 8 x 48 5.1 -> 4.6, 4 x 96
// 4.9 -> 4.2; behind the split kernel, 16 short contexts 14.7 -> 14.45, four-layer step 83.4 -> 79.5.
constexpr int kMergeWaves = 4, kMergeBatch = 32;
constexpr int kMergeAlone = 24;   // up to that many items the first wavefront does the work alone
__device__ __forceinline__ float wave_sum(float v)   // four DPP steps in the rows of 16 lanes, then the four rows
{
    v += row_dpp<0xB1>(v);
    v += row_dpp<0x4E>(v);
    v += row_dpp<0x141>(v);
    v += row_dpp<0x140>(v);
    const int i = __float_as_int(v);
    return (__int_as_float(__builtin_amdgcn_readlane(i, 0)) + __int_as_float(__builtin_amdgcn_readlane(i, 16))) +
           (__int_as_float(__builtin_amdgcn_readlane(i, 32)) + __int_as_float(__builtin_amdgcn_readlane(i, 48)));
}
__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, row_dpp<0xB1>(v));
    v = fmaxf(v, row_dpp<0x4E>(v));
    v = fmaxf(v, row_dpp<0x141>(v));
    v = fmaxf(v, row_dpp<0x140>(v));
    const int i = __float_as_int(v);
    return fmaxf(fmaxf(__int_as_float(__builtin_amdgcn_readlane(i, 0)), __int_as_float(__builtin_amdgcn_readlane(i, 16))),
                 fmaxf(__int_as_float(__builtin_amdgcn_readlane(i, 32)), __int_as_float(__builtin_amdgcn_readlane(i, 48))));
}
// 2^(m - M), and 0 for m = -inf: an item without tokens has m = -inf, l = 0 and weighs nothing
__device__ __forceinline__ float merge_weight(float m, float M) { return m == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m - M); }

struct MergeArgs {
    const float *acc_ws;
    const float *ml_ws;
    const int32_t *seq_item_indptr;
    int batch;
    int n_q_heads;
    float *out;
};
template <int VEC>
__device__ __forceinline__ void merge_sequence(
    const float *__restrict__ acc_ws, const float *__restrict__ ml_ws, const int32_t *__restrict__ seq_item_indptr,
    int batch, int n_q_heads, float *__restrict__ out)
{
    constexpr int kParts = 2 / VEC;
    __shared__ float num_s[kMergeWaves][64 * VEC];
    __shared__ float2 ml_s[kMergeWaves];
    asm volatile("" :: "s"(acc_ws), "s"(ml_ws), "s"(seq_item_indptr), "s"(batch), "s"(n_q_heads), "s"(out), "s"(gridDim.y));   // all arguments at once
    const int b = blockIdx.y + blockIdx.z * gridDim.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (b >= batch) return;
    const int h = blockIdx.x / kParts, c0 = (blockIdx.x % kParts) * 64 + lane * VEC;   // this lane's first channel
    int i0 = ((ConstWords)seq_item_indptr)[b], i1 = ((ConstWords)seq_item_indptr)[b + 1];
    const bool alone = i1 - i0 <= kMergeAlone;
    if (!alone) {
        const int per = (i1 - i0 + kMergeWaves - 1) / kMergeWaves;
        i0 += wave * per;
        i1 = i0 + per < i1 ? i0 + per : i1;
    } else if (wave > 0) {
        return;
    }
    const uint32_t stride = (uint32_t)n_q_heads * (kHeadDim * 4);
    float M = -INFINITY, den = 0.0f;
    float num[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) num[v] = 0.0f;
    for (int i = i0; i < i1; i += kMergeBatch) {
        const int n = i1 - i < kMergeBatch ? i1 - i : kMergeBatch;
        // item i + k of the head at k * stride; those behind the last one lie outside the buffer: zeros, no memory access
        const float *base = acc_ws + ((size_t)i * n_q_heads + h) * kHeadDim;
        const Record rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, (uint32_t)(n - 1) * stride + kHeadDim * 4, 0x00027000);
        float2 ml = make_float2(-INFINITY, 0.0f);
        if (lane < n) ml = reinterpret_cast<const float2 *>(ml_ws)[(size_t)(i + lane) * n_q_heads + h];
        float a[kMergeBatch][VEC];
        uint32_t at = (uint32_t)c0 * 4;
        asm volatile("" : "+v"(at));   // (the offsets are not all made in front of the first load)
#pragma unroll
        for (int g = 0; g < kMergeBatch; g += 8) {
            if (g > 0 && n <= g) break;
#pragma unroll
            for (int k = g; k < g + 8; ++k, at += stride) {
                if constexpr (VEC == 2) {
                    const uint2 t = buffer_load8_once(rows, at);
                    a[k][0] = __uint_as_float(t.x);
                    a[k][VEC - 1] = __uint_as_float(t.y);
                } else {
                    a[k][0] = __uint_as_float(buffer_load4_once(rows, at));
                }
            }
        }
        const float Mn = fmaxf(M, wave_max(ml.x));
        const float so = merge_weight(M, Mn), w = merge_weight(ml.x, Mn);
        den = den * so + wave_sum(w * ml.y);
#pragma unroll
        for (int v = 0; v < VEC; ++v) num[v] *= so;
#pragma unroll
        for (int g = 0; g < kMergeBatch; g += 8) {
            if (g > 0 && n <= g) break;
#pragma unroll
            for (int k = g; k < g + 8; ++k) {
                const float wk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), k));
#pragma unroll
                for (int v = 0; v < VEC; ++v) num[v] = fmaf(wk, a[k][v], num[v]);
            }
        }
        M = Mn;
    }
    if (!alone) {
        if (wave > 0) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) num_s[wave][lane * VEC + v] = num[v];
            if (lane == 0) ml_s[wave] = make_float2(M, den);
        }
        __syncthreads();
        if (wave > 0) return;
        float2 o[kMergeWaves];
        float Mg = M;
#pragma unroll
        for (int k = 1; k < kMergeWaves; ++k) {
            o[k] = ml_s[k];
            Mg = fmaxf(Mg, o[k].x);
        }
        const float w0 = merge_weight(M, Mg);
        den *= w0;
#pragma unroll
        for (int v = 0; v < VEC; ++v) num[v] *= w0;
#pragma unroll
        for (int k = 1; k < kMergeWaves; ++k) {
            const float wk = merge_weight(o[k].x, Mg);
            den += wk * o[k].y;
#pragma unroll
            for (int v = 0; v < VEC; ++v) num[v] += wk * num_s[k][lane * VEC + v];
        }
    }
    const float r = den > 0.0f ? 1.0f / den : 0.0f;
    float *dst = out + ((size_t)b * n_q_heads + h) * kHeadDim + c0;
    if constexpr (VEC == 2) *reinterpret_cast<float2 *>(dst) = make_float2(num[0] * r, num[VEC - 1] * r);
    else dst[0] = num[0] * r;
}
template <int VEC>
__global__ __launch_bounds__(64 * kMergeWaves) void tkv_merge_kernel(MergeArgs a)
{
    merge_sequence<VEC>(a.acc_ws, a.ml_ws, a.seq_item_indptr, a.batch, a.n_q_heads, a.out);
}

// Sequences of hundreds of items, as a single long sequence with one kv head has them.  One workgroup of TH threads per
// (sequence, query head, one of SL channel slices).  32 / SL lanes own an item at a time: their 16-byte loads are the item's
// accumulators of the slice, so every partial is read once with 128-bit loads and TH * SL / 32 items are in flight per
// workgroup round.  Each such lane group keeps a running (M, l, acc); the groups are merged through LDS by the first wavefront.
constexpr int SL = 4, TH = 512;   // four workgroups per head, 64 item slots each
constexpr uint32_t kRowsGridX = 1u << 22;   // workgroups are folded there: a grid dimension ends at 2^32 threads
__device__ __forceinline__ void reduce_rows(
    const float *__restrict__ acc_ws, const float *__restrict__ ml_ws, const int32_t *__restrict__ seq_item_indptr,
    int n_rows /* sequences x query heads */, int n_q_heads, float *__restrict__ out)
{
    constexpr int kLanes = 32 / SL;       // lanes per item: 16 bytes each
    constexpr int kSlots = TH / kLanes;   // items in flight
    constexpr int kSubsets = 64 / kLanes; // the first wavefront merges the slots in this many interleaved subsets
    __shared__ float4 num_s[kSlots][kLanes];
    __shared__ float2 ml_s[kSlots];
    const int bh = blockIdx.y * (kRowsGridX / SL) + blockIdx.x / SL, slice = blockIdx.x % SL;
    if (bh >= n_rows) return;
    const int b = bh / n_q_heads, h = bh % n_q_heads, tid = threadIdx.x;
    const int slot = tid / kLanes, ln = tid % kLanes, cq = slice * kLanes + ln;   // cq: which float4 of the 32 of a row
    const int i0 = seq_item_indptr[b], i1 = seq_item_indptr[b + 1];
    float M = -INFINITY, den = 0.0f;
    float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
    for (int i = i0 + slot; i < i1; i += kSlots) {
        const size_t ph = (size_t)i * n_q_heads + h;
        const float2 ml = reinterpret_cast<const float2 *>(ml_ws)[ph];
        // a partial is read once, 512 contiguous bytes per item
        const uint4 au = load_once(reinterpret_cast<const uint4 *>(acc_ws + ph * kHeadDim) + cq);
        const float4 a = make_float4(__uint_as_float(au.x), __uint_as_float(au.y), __uint_as_float(au.z), __uint_as_float(au.w));
        // an item without tokens has m = -inf, l = 0 and weighs nothing; no branch, so the loads of several
        // rounds are in flight together
        const float Mn = fmaxf(M, ml.x);
        const float so = M == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(M - Mn);
        const float sn = ml.x == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ml.x - Mn);
        den = den * so + sn * ml.y;
        num.x = num.x * so + sn * a.x;
        num.y = num.y * so + sn * a.y;
        num.z = num.z * so + sn * a.z;
        num.w = num.w * so + sn * a.w;
        M = Mn;
    }
    num_s[slot][ln] = num;
    if (ln == 0) ml_s[slot] = make_float2(M, den);
    __syncthreads();
    if (tid < 64) {
        // lane (subset, ln) of the first wavefront merges slots subset, subset + kSubsets, ...
        float Mg = -INFINITY;
#pragma unroll
        for (int k = slot; k < kSlots; k += kSubsets) Mg = fmaxf(Mg, ml_s[k].x);
#pragma unroll
        for (int o = kLanes; o < 64; o <<= 1) Mg = fmaxf(Mg, __shfl_xor(Mg, o));
        float4 n = make_float4(0.f, 0.f, 0.f, 0.f);
        float d = 0.0f;
#pragma unroll
        for (int k = slot; k < kSlots; k += kSubsets) {
            const float2 ml = ml_s[k];
            const float wk = ml.x == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ml.x - Mg);
            const float4 a = num_s[k][ln];
            d += wk * ml.y;
            n.x += wk * a.x;
            n.y += wk * a.y;
            n.z += wk * a.z;
            n.w += wk * a.w;
        }
#pragma unroll
        for (int o = kLanes; o < 64; o <<= 1) {
            d += __shfl_xor(d, o);
            n.x += __shfl_xor(n.x, o);
            n.y += __shfl_xor(n.y, o);
            n.z += __shfl_xor(n.z, o);
            n.w += __shfl_xor(n.w, o);
        }
        const float r = d > 0.0f ? 1.0f / d : 0.0f;
        if (tid < kLanes)
            reinterpret_cast<float4 *>(out + ((size_t)b * n_q_heads + h) * kHeadDim)[cq] = make_float4(n.x * r, n.y * r, n.z * r, n.w * r);
    }
}
__global__ __launch_bounds__(TH) void tkv_reduce_rows_kernel(MergeArgs a)
{
    reduce_rows(a.acc_ws, a.ml_ws, a.seq_item_indptr, a.batch * a.n_q_heads, a.n_q_heads, a.out);
}

} // namespace

int tkv_launch_decode_split(const tkv_desc *desc, const void *pool, const uint8_t *bit_map, const void *q,
                            const int32_t *page_indptr, const int32_t *page_ids, const int32_t *n_tok_int2,
                            const int32_t *n_tok_int4, const int32_t *items, int32_t n_items, int32_t batch,
                            int32_t n_q_heads, float sm_scale, void *workspace, int32_t *status, void *stream)
{
    if (n_items == 0) return TKV_OK;
    float *acc_ws = (float *)workspace;
    float *ml_ws = acc_ws + (size_t)n_items * n_q_heads * kHeadDim;
    const float kappa = sm_scale * 1.44269504088896340736f;
    auto kernel = desc->int2_key_axis == TKV_KEYS_PER_CHANNEL ? tkv_decode_kernel<true> : tkv_decode_kernel<false>;
    int log2_r = 0;   // 1, 2, 4 or 8 query heads per kv head
    while ((desc->n_kv_heads << log2_r) < n_q_heads) ++log2_r;
    constexpr int kMaxY = 65535;
    const dim3 grid((unsigned)desc->n_kv_heads, (unsigned)(n_items < kMaxY ? n_items : kMaxY), (unsigned)((n_items + kMaxY - 1) / kMaxY));
    const DecodeArgs args = {(const uint8_t *)pool, bit_map, (const uint16_t *)q, page_indptr, page_ids, n_tok_int2, n_tok_int4, items, n_items, batch,
                             desc->n_kv_heads, log2_r, desc->n_pages_int2, desc->n_pages_int4, kappa, acc_ws, ml_ws, status};
    hipLaunchKernelGGL(kernel, grid, dim3(64), 0, (hipStream_t)stream, args);
    return hipGetLastError() == hipSuccess ? TKV_OK : TKV_ERR_HIP;
}

int tkv_launch_decode_reduce(const tkv_desc *desc, const int32_t *seq_item_indptr, int32_t n_items, int32_t batch,
                             int32_t n_q_heads, float *out, const void *workspace, void *stream)
{
    (void)desc;
    const float *acc_ws = (const float *)workspace;
    const float *ml_ws = acc_ws + (size_t)n_items * n_q_heads * kHeadDim;
    const MergeArgs args = {acc_ws, ml_ws, seq_item_indptr, batch, n_q_heads, out};
    // The item counts are on the device; the average per sequence picks the kernel.  The longest sequence decides how long
    // either takes, and it may hold nearly all items.  Up to 128 on average the merge kernel is the faster one for equal
    // counts and for every skew (against a kernel of 8 item slots, which it has replaced; us alone, 64 heads: [250, 45, 45, 44] 8.8 ->
    // 6.6, [300, 7 x 12] 9.5 -> 7.6, [200, 56] 7.3 -> 5.0; 8 heads: 24 x 128 6.2 -> 4.9, [2049, 31 x 33] 45 -> 27).  Above, it
    // gains on equal counts and loses on skewed ones (64 slots / merge kernel, 64 heads: 16 x 161 21.5 / 16.6, 2 x 192 5.9 / 5.1,
    // [380, 4] 6.1 / 6.6, [700, 1, 1, 1] 8.4 / 12.5; 8 heads: 16 x 161 5.4 / 4.8, 4 x 256 4.6 / 4.9, 16 between 30 and 409 6.2 / 7.9,
    // [2049, 11 x 32] 11.3 / 18.7), and the host cannot tell them apart.  Two channels a lane where that gives 256 workgroups:
    // 64 heads, 8 x 48 4.6 against 4.9, 4 x 96 4.2 against 4.6; 8 heads, 4 x 96 3.0 against 2.8.  (32 items of one head are
    // addressed in 32 bits.)
    if ((int64_t)n_items <= 128 * (int64_t)batch && n_q_heads <= 1 << 17) {
        const bool two = (int64_t)batch * n_q_heads >= 256;
        constexpr int kMaxY = 65535;
        const dim3 grid((unsigned)n_q_heads * (two ? 1 : 2), (unsigned)(batch < kMaxY ? batch : kMaxY), (unsigned)((batch + kMaxY - 1) / kMaxY));
        hipLaunchKernelGGL(two ? tkv_merge_kernel<2> : tkv_merge_kernel<1>, grid, dim3(64 * kMergeWaves), 0, (hipStream_t)stream, args);
    } else {
        const uint64_t blocks = (uint64_t)batch * n_q_heads * SL;
        const dim3 grid((unsigned)(blocks < kRowsGridX ? blocks : kRowsGridX), (unsigned)((blocks + kRowsGridX - 1) / kRowsGridX));
        hipLaunchKernelGGL(tkv_reduce_rows_kernel, grid, dim3(TH), 0, (hipStream_t)stream, args);
    }
    return hipGetLastError() == hipSuccess ? TKV_OK : TKV_ERR_HIP;
}

// ---- tkv_decode_attention_static: the same two launches with the partials in a file-scope device array ----
// For callers that cannot allocate (HIP graph capture, tight serving loops).  `scratch` is a host-side
// stand-in for the device array: its device address is looked up once per device and only that address
// is handed to kernels.
static __device__ __align__(256) unsigned char scratch[TKV_DECODE_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each device, null until first use there

// Device address of this device's copy of `scratch` (the current device), or null on failure.
void *scratch_address()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}
} // namespace

extern "C" int tkv_decode_attention_static(const tkv_desc *desc, const void *pool, const uint8_t *bit_map,
                                           const void *q, const int32_t *page_indptr, const int32_t *page_ids,
                                           const int32_t *n_tok_int2, const int32_t *n_tok_int4,
                                           const int32_t *items, const int32_t *seq_item_indptr, int32_t n_items,
                                           int32_t batch, int32_t n_q_heads, float sm_scale, float *out,
                                           int32_t *status, void *stream)
{
    // the argument checks of tkv_decode_attention, with the fixed array as the workspace
    const size_t need = tkv_decode_workspace_bytes(desc, n_items, n_q_heads);
    if (desc && n_items > 0 && n_q_heads > 0 && need == 0) return TKV_ERR_BAD_SHAPE;
    if (need > (size_t)TKV_DECODE_STATIC_SCRATCH_BYTES) return TKV_ERR_WORKSPACE_TOO_SMALL;
    alignas(16) static const char placeholder[16] = {0};   // stands for the workspace in the host-side checks (non-null, aligned)
    if (int st = tkv_decode_check_args(desc, n_items, batch, n_q_heads, placeholder, TKV_DECODE_STATIC_SCRATCH_BYTES)) return st;
    if (batch == 0) return TKV_OK;
    if (!(sm_scale > 0.0f) || !(sm_scale < 3.0e38f)) return TKV_ERR_INVALID_ARG;
    if (!q || !out || !page_indptr || !n_tok_int2 || !n_tok_int4 || !seq_item_indptr) return TKV_ERR_INVALID_ARG;
    if (n_items > 0 && (!pool || !bit_map || !page_ids || !items)) return TKV_ERR_INVALID_ARG;
    if (((uintptr_t)pool & 255) || ((uintptr_t)q & 15) || ((uintptr_t)out & 15)) return TKV_ERR_INVALID_ARG;
    void *ws = scratch_address();
    if (!ws) return TKV_ERR_HIP;
    // every partial the reduction reads is written by the split kernel of this call: nothing to clear
    if (int st = tkv_launch_decode_split(desc, pool, bit_map, q, page_indptr, page_ids, n_tok_int2, n_tok_int4, items,
                                         n_items, batch, n_q_heads, sm_scale, ws, status, stream))
        return st;
    return tkv_launch_decode_reduce(desc, seq_item_indptr, n_items, batch, n_q_heads, out, ws, stream);
}
