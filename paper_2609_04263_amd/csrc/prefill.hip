// Chunked prefill attention over the packed cache (Sec. 3.1: evaluation
// runs chunk by chunk; the chunk's states are coded and appended, then its
// queries attend causally over the reconstruction of everything stored).
//
// A 32-token block enters the products as a "block image" (192 D bytes):
// k_hat in fp32 stored as fp16 hi + lo (~22 bits), v_hat as fp16, both in
// the order of the MFMA operand fragments, so a fragment is 1 KiB that the
// wave reads with one conflict-free 16-byte load per lane from one base
// address.  A block of per-token key groups whose tokens are all coded (a
// "code block") keeps the key codes instead, as exact fp16 values, with the
// groups' scales and offsets in place of the lo half.  A rotating format's
// keys and values are rotated back to the original basis (an fp32 FWHT per
// token in LDS) before they are rounded, so queries and outputs need no
// rotation.  dequant_kernel reconstructs every visible block of a unit once
// into the caller's workspace and attn_kernel streams the images through an
// LDS ring with global_load_lds_dwordx4.
//
// Each workgroup handles 256 query rows ((chunk token, head) pairs of a
// unit, token-major), each wave 32 QT of them, and per block:
//   - scores S^T = K Q^T with v_mfma_f32_32x32x16_f16 (keys as rows, query
//     rows as columns).  A bf16 query scaled by a power of two is exact in
//     fp16, so the products are K hi x q + K lo x q, or for a code block S =
//     sum_g s_g (c_g . q_g) + z'_g sum q_g with exact products c q, one fp32
//     scaling of each group's tile and the offset terms as fp32 MFMAs
//     (v_mfma_f32_32x32x2_f32: two groups each);
//   - softmax in base 2, online per column (the running maximum moves only
//     in steps of more than 2^8);
//   - O^T += V^T P^T in fp16.  A lane holds the score rows 8 j + 4 h + i of
//     its half wave h, which are the eight k-slots of its next two operands
//     when the image stores V^T in that key order, so probabilities never
//     cross lanes.
// Why 32 rows per wave: a wave reads every K and V fragment of a block from
// LDS once for all of its rows.  With 16 rows at D = 256 the eight waves read
// 256 KiB per block against 1024 cycles of MFMA work, and LDS, not the matrix
// cores, was the limit (3500 cycles per block of 128 rows; now 4070 per block
// of 256, 2320 of them MFMA); 32 rows halve that, and take 128 accumulator and
// 64 query registers, which fits two waves per SIMD only because fragment
// order needs no address arithmetic.  A chunk of 2048 tokens at the end of
// 8192 (B = 8, 16 query heads on 8, D = 256): 2570 -> 2170 us per call.
// Sink tokens (fp16 rows) come first as blocks of their own; fp16 window
// tokens past the coded ones are read from the ring.

#include <atomic>

#include "kvq_device.h"
#include "kvq_internal.h"

namespace kvq {
namespace pre {

constexpr int kDqThreads = 256;

// Waves per attention workgroup: eight (one workgroup per CU, two waves per
// SIMD), four at D = 64, where two workgroups share a CU (each SIMD holds
// one wave of each, with independent per-block barriers).
template <int D>
constexpr int waves()
{
    return D == 64 ? 4 : 8;
}

template <int D>
constexpr int threads()
{
    return 64 * waves<D>();
}

// 32-row query tiles per wave: 256 rows per workgroup at every head size
template <int D>
constexpr int qtiles()
{
    return D == 64 ? 2 : 1;
}

constexpr int kRows = 256;  // query rows per workgroup

// One reconstructed 32-token block, 192 D bytes: K hi, K lo (64 D bytes
// each), V (64 D bytes), all in fragment order.  K fragment s (channels 16 s
// .. + 15) is the 1 KiB at 1024 s: lane l's 16 bytes at 16 l are channels 16 s
// + 8 (l / 32) .. + 7 of token l % 32.  V fragment (t, u) is the 1 KiB at 1024
// (2 t + u): lane l holds channel 32 t + l % 32 of the tokens 16 u + 4 h + {0
// .. 3, 8 .. 11}, h = l / 32.
template <int D>
__host__ __device__ constexpr int image_bytes()
{
    return 192 * D;
}

// Byte offsets in an image of the K lo half (or a code block's scales and
// offsets) and of V.
template <int D>
__host__ __device__ constexpr int klo_at()
{
    return 64 * D;
}

template <int D>
__host__ __device__ constexpr int vt_at()
{
    return 128 * D;
}

// LDS ring depth (block images in flight) of the workspace path
template <int D>
constexpr int stages()
{
    return D == 128 ? 4 : 3;
}

// Query fragments per wave kept in LDS
template <int D>
__host__ __device__ constexpr int query_lds_fragments()
{
    return D == 256 ? 2 : 0;
}

// the ring, then the query fragments
template <int D>
constexpr size_t attn_lds_bytes()
{
    return (size_t)stages<D>() * image_bytes<D>() + (size_t)waves<D>() * query_lds_fragments<D>() * 1024;
}

__device__ __forceinline__ float dq(int mode, int bits, uint32_t c, float s, float z)
{
    return mode == KVQ_AFFINE ? (float)c * s + z : ((float)c - (float)(1 << (bits - 1))) * s;
}

// scale or offset i of a raw metadata range (fp32, or fp16 with meta16)
__device__ __forceinline__ float meta(const uint8_t* sec, size_t i, bool m16)
{
    return m16 ? f16_bits_to_f32(((const uint16_t*)sec)[i]) : ((const float*)sec)[i];
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// v_mfma_f32_32x32x16_f16: D[32x32] += A[32x16] B[16x32].  Lane l supplies
// A[l % 32][8 (l / 32) + e] and B[8 (l / 32) + e][l % 32], and receives
// D[8 (e / 4) + 4 (l / 32) + e % 4][l % 32] for e = 0..15.
__device__ __forceinline__ floatx16 mfma32(half8 a, half8 b, floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Eight codes of piece idx of a block's code range (8-bit: two u32; 4-bit:
// one u32; 2-bit: one u16), as the words holding codes 0..3 and 4..7 (the
// same word unless the codes are 8-bit).
struct Piece {
    uint32_t lo, hi;
};

template <bool W8>
__device__ __forceinline__ Piece piece(const uint8_t* sec, int idx, int bits)
{
    if constexpr (W8) {
        const u32x2 w = ((const u32x2*)sec)[idx];
        return Piece{w.x, w.y};
    }
    const uint32_t w = bits == 4 ? ((const uint32_t*)sec)[idx] : ((const uint16_t*)sec)[idx];
    return Piece{w, w};
}

// Code e (0..7) of a piece.
__device__ __forceinline__ uint32_t code_of(const Piece& w, int bits, int e)
{
    const uint32_t x = e < 4 ? w.lo : w.hi;
    return (x >> ((bits * e) & 31)) & ((1u << bits) - 1u);
}

// four consecutive scales or offsets from element i (a multiple of 4)
__device__ __forceinline__ void meta4(const uint8_t* sec, int i, bool m16, float* v)
{
    if (m16) {
        const uint2 h = *(const uint2*)(sec + 2 * i);
        v[0] = f16_bits_to_f32((uint16_t)h.x);
        v[1] = f16_bits_to_f32((uint16_t)(h.x >> 16));
        v[2] = f16_bits_to_f32((uint16_t)h.y);
        v[3] = f16_bits_to_f32((uint16_t)(h.y >> 16));
    } else {
        const floatx4 a = *(const floatx4*)(sec + 4 * i);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = a[e];
    }
}

__device__ __forceinline__ float half_bits(const uint16_t* row, size_t i)
{
    return f16_bits_to_f32(row[i]);
}

// Whether a block (sink block when sinkblk, else tail block blk) is a code
// block: per-token key groups, no rotation, every token of the block coded.
// Its image holds the key codes as exact fp16 values in place of k_hat's hi
// half, and the group scales and offsets in place of the lo half.  Groups of
// 32 at D = 256 (eight groups) keep hi + lo keys.
template <int D>
__device__ __forceinline__ bool code_block(const AttnParams& p, bool sinkblk, int blk)
{
    return p.k_axis == KVQ_PER_TOKEN && !p.rotate && !(D >= 256 && p.k_group == 32) && !sinkblk && 32 * blk + 31 < p.nq;
}

// One block's packed sections (codes, scales, offsets of K and V; offsets
// null for symmetric codes), in global memory or in LDS, and the byte lengths
// they have.
struct Sections {
    const uint8_t *kc, *ks, *kz, *vc, *vs, *vz;
};

struct SectionBytes {
    int kc, km, vc, vm;  // codes of K, scales (and offsets) of K, the same of V
};

template <int D, bool W8>
__device__ __forceinline__ SectionBytes section_bytes(const AttnParams& p)
{
    const int msz = p.meta16 ? 2 : 4;
    SectionBytes s;
    s.kc = 4 * D * (W8 ? 8 : p.k_bits);
    s.km = p.k_axis == KVQ_PER_TOKEN ? (D / p.k_group) * 32 * msz : D * msz;
    s.vc = 4 * D * (W8 ? 8 : p.v_bits);
    s.vm = (D / p.v_group) * 32 * msz;
    return s;
}

// Block i (unit * blocks + block) in the cache.
__device__ __forceinline__ Sections cache_sections(const AttnParams& p, const SectionBytes& n, size_t i)
{
    Sections s;
    s.kc = (const uint8_t*)p.kc + i * n.kc;
    s.ks = (const uint8_t*)p.ks + i * n.km;
    s.kz = p.k_mode == KVQ_AFFINE ? (const uint8_t*)p.kz + i * n.km : nullptr;
    s.vc = (const uint8_t*)p.vc + i * n.vc;
    s.vs = (const uint8_t*)p.vs + i * n.vm;
    s.vz = p.v_mode == KVQ_AFFINE ? (const uint8_t*)p.vz + i * n.vm : nullptr;
    return s;
}

// Rows of the rotation scratch: 32 tokens of D fp32, the pitch padded so that
// 16-byte reads of one channel chunk over consecutive rows hit distinct banks.
template <int D>
constexpr int scratch_pitch()
{
    return D + 4;
}

template <int D>
constexpr size_t scratch_bytes()
{
    return (size_t)32 * scratch_pitch<D>() * 4;
}

// In-place FWHT of the scratch's 32 rows (butterflies of half width 1, 2, ..,
// D / 2), then * c, by a workgroup of NTH threads: three half widths per pass
// in registers (1, 2, 4; 8, 16, 32; then 64 and 128).  Ends with a barrier.
template <int D, int NTH>
__device__ __forceinline__ void fwht_block(float* x, float c)
{
    constexpr int PT = scratch_pitch<D>();
    __syncthreads();
#pragma unroll
    for (int i = threadIdx.x; i < 32 * (D / 8); i += NTH) {
        float* r = x + (i & 31) * PT + 8 * (i >> 5);
        floatx4 a = *(const floatx4*)r, b = *(const floatx4*)(r + 4);
        float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
#pragma unroll
        for (int h = 1; h < 8; h <<= 1)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (!(e & h)) {
                    const float s = v[e], t = v[e + h];
                    v[e] = s + t;
                    v[e + h] = s - t;
                }
        *(floatx4*)r = floatx4{v[0], v[1], v[2], v[3]};
        *(floatx4*)(r + 4) = floatx4{v[4], v[5], v[6], v[7]};
    }
    __syncthreads();
#pragma unroll
    for (int i = threadIdx.x; i < 32 * (D / 8); i += NTH) {
        // lanes: eight channels of a 64-channel span, then spans, then rows
        float* r = x + (i / (D / 8)) * PT + 64 * ((i % (D / 8)) >> 3) + (i & 7);
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = r[8 * e];
#pragma unroll
        for (int h = 1; h < 8; h <<= 1)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (!(e & h)) {
                    const float s = v[e], t = v[e + h];
                    v[e] = s + t;
                    v[e + h] = s - t;
                }
#pragma unroll
        for (int e = 0; e < 8; ++e)
            r[8 * e] = D == 64 ? v[e] * c : v[e];
    }
    __syncthreads();
    if constexpr (D > 64) {
        constexpr int NV = D / 64;
#pragma unroll
        for (int i = threadIdx.x; i < 32 * 64; i += NTH) {
            float* r = x + (i >> 6) * PT + (i & 63);
            float v[NV];
#pragma unroll
            for (int e = 0; e < NV; ++e)
                v[e] = r[64 * e];
#pragma unroll
            for (int h = 1; h < NV; h <<= 1)
#pragma unroll
                for (int e = 0; e < NV; ++e)
                    if (!(e & h)) {
                        const float s = v[e], t = v[e + h];
                        v[e] = s + t;
                        v[e + h] = s - t;
                    }
#pragma unroll
            for (int e = 0; e < NV; ++e)
                r[64 * e] = v[e] * c;
        }
        __syncthreads();
    }
}

// Keys of a rotating format are kept at 2^-4 of their value: rotated back, an
// outlier channel can be sqrt(D) <= 16 times the largest stored magnitude,
// and binary16 must still hold it.
constexpr float kRotKeyScale = 0.0625f;

// The image of one block, by a workgroup of NTH threads: sink block sb when
// sb >= 0, else tail block blk.  CODED: every token is coded (and `s` may be
// in LDS).  Tokens past the end (sink rows beyond n_sink, tail tokens beyond
// n) are zeros: the causal mask removes them, and zero values keep 0 * v
// finite.  W8: both code widths are 8 bits.  ROT: through `scratch` (LDS),
// with barriers; otherwise none.
template <int D, bool W8, bool ROT, int NTH, bool CODED>
__device__ __forceinline__ void build_image(const AttnParams& p, int unit, int sb, int blk, const Sections& s, bool ck,
                                            uint8_t* img, float* scratch)
{
    const int kbits = W8 ? 8 : p.k_bits, vbits = W8 ? 8 : p.v_bits;
    const bool kaff = p.k_mode == KVQ_AFFINE, vaff = p.v_mode == KVQ_AFFINE;
    const bool m16 = p.meta16 != 0;
    const size_t sbase = (size_t)unit * p.sink;
    const size_t rbase = (size_t)unit * p.ring;
    constexpr int PT = scratch_pitch<D>();

    // K piece: token tau, channels 8 P .. 8 P + 7; 32 consecutive lanes write
    // 512 contiguous bytes
#pragma unroll
    for (int pc = threadIdx.x; pc < 4 * D; pc += NTH) {
        const int tau = pc & 31, P = pc >> 5;
        float x[8];
        const uint16_t* row = nullptr;  // fp16 source row (sink or window)
        bool coded = CODED;
        if constexpr (!CODED) {
            if (sb >= 0) {
                const int ts = 32 * sb + tau;
                if (ts < p.n_sink)
                    row = p.kq + (sbase + ts) * D;
            } else {
                const int t = 32 * blk + tau;
                if (t < p.nq)
                    coded = true;
                else if (t < p.n)
                    row = p.kr + (rbase + t % p.ring) * D;
            }
        }
        if (coded) {
            const int r = 4 * (tau >> 3) + (tau & 3), half = (tau >> 2) & 1;
            const int idx = (half * 64 + r + 16 * (P & 3)) * (D / 32) + (P >> 2);
            const Piece w = piece<W8>(s.kc, idx, kbits);
            if (!ROT && ck) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    x[e] = (float)code_of(w, kbits, e);
            } else if (p.k_axis == KVQ_PER_TOKEN) {
                const int mi = ((8 * P) / p.k_group) * 32 + tau;
                const float sc = meta(s.ks, mi, m16), z = kaff ? meta(s.kz, mi, m16) : 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    x[e] = dq(p.k_mode, kbits, code_of(w, kbits, e), sc, z);
            } else {
                // per-channel keys: the piece's eight channels' scales
                // (and offsets) are consecutive, two vector loads each
                float sc[8], zc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                meta4(s.ks, 8 * P, m16, sc);
                meta4(s.ks, 8 * P + 4, m16, sc + 4);
                if (kaff) {
                    meta4(s.kz, 8 * P, m16, zc);
                    meta4(s.kz, 8 * P + 4, m16, zc + 4);
                }
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    x[e] = dq(p.k_mode, kbits, code_of(w, kbits, e), sc[e], zc[e]);
            }
        } else if (row) {
            const u32x4 rw = *(const u32x4*)(row + 8 * P);
            const uint32_t w4[4] = {rw.x, rw.y, rw.z, rw.w};
#pragma unroll
            for (int e = 0; e < 8; ++e)
                x[e] = f16_bits_to_f32((uint16_t)(w4[e >> 1] >> (16 * (e & 1))));
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                x[e] = 0.0f;
        }
        if constexpr (ROT) {
            float* dst = scratch + tau * PT + 8 * P;
            *(floatx4*)dst = floatx4{x[0], x[1], x[2], x[3]};
            *(floatx4*)(dst + 4) = floatx4{x[4], x[5], x[6], x[7]};
        } else if (ck) {
            *(u32x4*)(img + 16 * pc) = __builtin_bit_cast(u32x4, pack_half8(x));
        } else {
            half8 h, l;
            split_half8(x, &h, &l);
            *(u32x4*)(img + 16 * pc) = __builtin_bit_cast(u32x4, h);
            *(u32x4*)(img + klo_at<D>() + 16 * pc) = __builtin_bit_cast(u32x4, l);
        }
    }
    if constexpr (ROT) {
        fwht_block<D, NTH>(scratch, p.rot_c * kRotKeyScale);
#pragma unroll
        for (int pc = threadIdx.x; pc < 4 * D; pc += NTH) {
            const float* src = scratch + (pc & 31) * PT + 8 * (pc >> 5);
            const floatx4 a = *(const floatx4*)src, b = *(const floatx4*)(src + 4);
            const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
            half8 h, l;
            split_half8(x, &h, &l);
            *(u32x4*)(img + 16 * pc) = __builtin_bit_cast(u32x4, h);
            *(u32x4*)(img + klo_at<D>() + 16 * pc) = __builtin_bit_cast(u32x4, l);
        }
        __syncthreads();  // the values follow through the same scratch
    }

    // V piece: channel d, fragment chunk c = 2 u + h (tokens 16 u + 4 h + {0
    // .. 3, 8 .. 11}: codes 4 h .. 4 h + 3 of octets 2 u and 2 u + 1)
#pragma unroll
    for (int pc = threadIdx.x; pc < 4 * D; pc += NTH) {
        const int d = (pc & 31) + 32 * (pc >> 7), c = (pc >> 5) & 3, u = c >> 1, h = c & 1;
        float x[8];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int tk0 = 16 * u + 8 * j + 4 * h;  // first of four tokens
            if (CODED || (sb < 0 && 32 * blk + tk0 < p.nq)) {
                const Piece w = piece<W8>(s.vc, (d % 16 + 16 * (2 * u + j)) * (D / 16) + d / 16, vbits);
                const int mi = (d / p.v_group) * 32 + tk0;
                float sc[4], zc[4] = {0.f, 0.f, 0.f, 0.f};
                meta4(s.vs, mi, m16, sc);
                if (vaff)
                    meta4(s.vz, mi, m16, zc);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float val = dq(p.v_mode, vbits, code_of(w, vbits, 4 * h + e), sc[e], zc[e]);
                    if constexpr (CODED) {
                        x[4 * j + e] = val;
                    } else {
                        const int t = 32 * blk + tk0 + e;
                        x[4 * j + e] = t < p.nq  ? val
                                       : t < p.n ? half_bits(p.vr, (rbase + t % p.ring) * D + d)
                                                 : 0.0f;
                    }
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int tk = tk0 + e;
                    float val = 0.0f;
                    if (sb >= 0) {
                        const int ts = 32 * sb + tk;
                        if (ts < p.n_sink)
                            val = half_bits(p.vq, (sbase + ts) * D + d);
                    } else {
                        const int t = 32 * blk + tk;
                        if (t < p.n)
                            val = half_bits(p.vr, (rbase + t % p.ring) * D + d);
                    }
                    x[4 * j + e] = val;
                }
            }
        }
        if constexpr (ROT) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                scratch[(16 * u + 4 * h + 8 * (e >> 2) + (e & 3)) * PT + d] = x[e];
        } else {
            *(u32x4*)(img + vt_at<D>() + 16 * pc) = __builtin_bit_cast(u32x4, pack_half8(x));
        }
    }
    if constexpr (ROT) {
        fwht_block<D, NTH>(scratch, p.rot_c);
#pragma unroll
        for (int pc = threadIdx.x; pc < 4 * D; pc += NTH) {
            const int d = (pc & 31) + 32 * (pc >> 7), c = (pc >> 5) & 3;
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                x[e] = scratch[(16 * (c >> 1) + 4 * (c & 1) + 8 * (e >> 2) + (e & 3)) * PT + d];
            *(u32x4*)(img + vt_at<D>() + 16 * pc) = __builtin_bit_cast(u32x4, pack_half8(x));
        }
    }
    // a code block's key scales and offsets z'[g][t] (fp32, in place of the
    // lo half), with k_hat = c s + z': z' = z for affine codes, -2^(bits-1) s
    // for symmetric ones.  The scales are kept as ratios s[g] / s[g + 1], the
    // last group's as it is: the score sum over groups is then one chain of
    // products, its running sum moved from one group's scale to the next
    // (scales are never zero: the code's floor is 1e-8, 2^-24 in fp16).
    if (!ROT && ck) {
        const int ng = D / p.k_group;
        float* ms = (float*)(img + klo_at<D>());
        for (int i = threadIdx.x; i < 32 * ng; i += NTH) {
            const float sc = meta(s.ks, i, m16);
            ms[i] = i + 32 < 32 * ng ? sc / meta(s.ks, i + 32, m16) : sc;
            ms[32 * ng + i] = kaff ? meta(s.kz, i, m16) : -(float)(1 << (kbits - 1)) * sc;
        }
    }
}

// ---------------------------------------------------------------------------
// 1. Workspace images.  Grid (blocks per unit, units of the group); workspace
// block v of a unit is sink block v for v < pf_nsb, else tail block v - pf_nsb.
template <int D, bool W8, bool ROT>
__global__ __launch_bounds__(kDqThreads) void dequant_kernel(AttnParams p)
{
    extern __shared__ __attribute__((aligned(16))) float dq_scratch[];
    const int v = blockIdx.x;
    const int unit = p.pf_u0 + blockIdx.y;
    uint8_t* img = p.pf_ws + ((size_t)blockIdx.y * p.pf_nvb + v) * (size_t)image_bytes<D>();
    const bool sinkblk = v < p.pf_nsb;
    const int blk = v - p.pf_nsb;
    const size_t i = (size_t)unit * (p.T >> 5) + (sinkblk ? 0 : blk);
    const Sections s = cache_sections(p, section_bytes<D, W8>(p), i);
    build_image<D, W8, ROT, kDqThreads, false>(p, unit, sinkblk ? v : -1, blk, s, code_block<D>(p, sinkblk, blk), img,
                                               dq_scratch);
}

// ---------------------------------------------------------------------------
// 2. Attention over block images in LDS.

// 16 bytes per lane from global memory to LDS address lds_addr + 16 lane
// (lds_addr wave-uniform, held in M0 while the copy issues).  Inline
// assembly, so that the compiler does not make LDS reads wait for every
// outstanding copy; the kernel's own vmcnt waits order them.
__device__ __forceinline__ void copy16(uint64_t base, uint32_t voff, uint32_t lds_addr)
{
    const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds_addr);
    // (the builtin returns int: widen both halves as unsigned, or a low
    // word with bit 31 set would be sign-extended into the high word)
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)base);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
    const uint64_t sb = ((uint64_t)hi << 32) | (uint64_t)lo;
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(m0v), "v"(voff), "s"(sb) : "memory");
}

// s_waitcnt vmcnt(n) for a wave-uniform n (expcnt and lgkmcnt not waited)
__device__ __forceinline__ void wait_vm(int n)
{
    switch (n) {
#define KVQ_WAIT_VM(k)                              \
    case k:                                         \
        __builtin_amdgcn_s_waitcnt(0x0F70 | (k)); \
        break;
        KVQ_WAIT_VM(1)
        KVQ_WAIT_VM(2)
        KVQ_WAIT_VM(3)
        KVQ_WAIT_VM(4)
        KVQ_WAIT_VM(5)
        KVQ_WAIT_VM(6)
        KVQ_WAIT_VM(7)
        KVQ_WAIT_VM(8)
        KVQ_WAIT_VM(9)
        KVQ_WAIT_VM(10)
        KVQ_WAIT_VM(11)
        KVQ_WAIT_VM(12)
#undef KVQ_WAIT_VM
    default:
        __builtin_amdgcn_s_waitcnt(0x0F70);
    }
}

// The copies of this wave that precede the newest `after` of its issued
// copies have landed, then every wave is past the same point.
__device__ __forceinline__ void ring_sync(int after)
{
    wait_vm(after);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Query rows of a workgroup: rows r0 .. r0 + 255 of a unit.  Positions are
// tail indices (token minus sink); sink tokens sit at -sink .. -1, so a chunk
// that starts in the sink has negative positions.
struct Tile {
    int unit, b, h;  // unit = b H + h
    int r0, rows;
    int nsb, nvis;   // sink blocks and all blocks that hold a visible token
};

__device__ __forceinline__ Tile make_tile(const AttnParams& p, int unit, int tile)
{
    Tile t;
    t.unit = unit;
    t.b = __builtin_amdgcn_readfirstlane(unit / p.H);
    t.h = unit - t.b * p.H;
    t.rows = p.C * p.G;
    t.r0 = tile * kRows;
    const int newest = __builtin_amdgcn_readfirstlane(p.n - p.C + (min(t.r0 + kRows, t.rows) - 1) / p.G);
    const int nkb = newest >= 0 ? newest / 32 + 1 : 0;  // coded-tail blocks
    t.nsb = min((p.n_sink + 31) >> 5, (newest + p.sink) / 32 + 1);
    t.nvis = t.nsb + nkb;
    return t;
}

constexpr int kNoRow = -(1 << 30);  // position of a query row past the end: every key masked

// One wave's state: 32 QT query rows (columns of the MFMAs: column l % 32 of
// tile q is row r0 + 32 (QT wave + q) + l % 32).  KG: key group size / 32 when
// the format's keys have per-token groups (code blocks then take exact code
// operands), 0 otherwise.
template <int D, int KG, int QT>
struct Wave {
    static constexpr int NK = D / 16, NT = D / 32;        // K fragments, 32-channel value tiles
    static constexpr int KS = KG > 0 ? 2 * KG : NK;       // K fragments per group
    static constexpr int NG = NK / KS, NZ = (NG + 1) / 2;  // groups, offset MFMAs per tile
    static constexpr int PF = D == 256 ? 3 : 4;  // fragments read ahead (LDS latency)
        // The last QL query fragments of a wave live in LDS (the 16 KiB that the
    // ring leaves free at D = 256, where the registers do not hold them all).
    static constexpr int QL = query_lds_fragments<D>();
    half8 q[QT][NK - QL];
    uint8_t* ql;
    float qz[QT][NZ];  // lane (col, h): the query's sum over group 2 j + h
    int qpos[QT];
    float sscale;      // scores times sscale are exponents (base 2)
    int first;         // position of the wave's oldest query when all its rows exist
    floatx16 acc[QT][NT];
    floatx16 s[QT];    // the scores of the block between scores() and update()
    float m[QT], lsum[QT];

    // `spare`: 1 KiB QL per wave of LDS that nothing else uses
    __device__ __forceinline__ void init(const AttnParams& p, const Tile& t, uint8_t* spare, int wave, int lane)
    {
        static_assert(QL == 0 || QT == 1, "one query tile per wave");
        ql = spare + 1024 * QL * wave + 16 * lane;
        const int col = lane & 31, hf = lane >> 5;
        // Queries are scaled by qscale, sm_scale log2(e) rounded down to a
        // power of two (exact in fp16 below 65504), and the scores take the
        // rest, sscale (qscale keeps the sign of the scale, so sscale > 0; a
        // zero or subnormal scale gives zero queries, zero scores, sscale 1)
        const float qscale = __uint_as_float(__float_as_uint(p.sm_log2) & 0xFF800000u);
        sscale = qscale == 0.0f ? 1.0f : p.sm_log2 / qscale;
        if (p.rotate)
            sscale *= 1.0f / kRotKeyScale;
        sscale = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(sscale)));  // a scalar register
        const int first_pos = p.n - p.C, wrow0 = t.r0 + 32 * QT * wave;
        first = __builtin_amdgcn_readfirstlane(wrow0 + 32 * QT <= t.rows ? first_pos + wrow0 / p.G : kNoRow);
#pragma unroll
        for (int c = 0; c < QT; ++c) {
            const int R = wrow0 + 32 * c + col;
            const int i = R / p.G, g = R % p.G;
            const uint16_t* src = p.q + (((size_t)t.b * p.C + i) * p.H_q + (size_t)t.h * p.G + g) * D + 8 * hf;
            float qsum[NG];
#pragma unroll
            for (int j = 0; j < NG; ++j)
                qsum[j] = 0.0f;
#pragma unroll
            for (int s = 0; s < NK; ++s) {
                u32x4 w = {0u, 0u, 0u, 0u};
                if (R < t.rows)
                    w = *(const u32x4*)(src + 16 * s);
                const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
                float v[8];
                float part = 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[e] = __uint_as_float((e & 1) ? (ww[e >> 1] & 0xFFFF0000u) : (ww[e >> 1] << 16)) * qscale;
                    part += v[e];
                }
                if (s < NK - QL)
                    q[c][s] = pack_half8(v);
                else  // read back by this lane alone
                    *(u32x4*)(ql + 1024 * (s - (NK - QL))) = __builtin_bit_cast(u32x4, pack_half8(v));
                if (KG > 0)
                    qsum[s / KS] += part;
            }
#pragma unroll
            for (int j = 0; j < NZ; ++j)
                qz[c][j] = 0.0f;
            if (KG > 0) {
                // the column's two lanes hold half of every group each
#pragma unroll
                for (int j = 0; j < NG; ++j) {
                    const float sum = qsum[j] + __shfl_xor(qsum[j], 32);
                    qz[c][j / 2] = hf == (j & 1) ? sum : qz[c][j / 2];
                }
            }
            qpos[c] = R < t.rows ? first_pos + i : kNoRow;
            m[c] = -INFINITY;
            lsum[c] = 0.0f;
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[c][j] = floatx16{};
        }
    }

    // Scores S^T (keys x query rows) of one block image; code: whether it is a
    // code block.  PF fragments are read ahead.  hook(k) runs beside fragment k.
    template <typename Hook>
    __device__ __forceinline__ void scores(const uint8_t* img, bool code, int lane, Hook hook)
    {
        if constexpr (D == 256)
            __builtin_amdgcn_s_setprio(1);  // the matrix products first: 1% at D = 256
        const int hf = lane >> 5;
        const uint8_t* fb = img + 16 * lane;  // fragment f of a part is at fb + 1024 f
        auto frag = [&](int at) { return __builtin_bit_cast(half8, *(const u32x4*)(fb + at)); };
        half8 fq[QL > 0 ? QL : 1];
        auto query = [&](int k) { return __builtin_bit_cast(half8, *(const u32x4*)(ql + 1024 * (k - (NK - QL)))); };
#pragma unroll
        for (int c = 0; c < QT; ++c)
            s[c] = floatx16{};
        if (KG > 0 && code) {
            // exact codes c: S = sum_g s_g (c_g . q_g) + z'_g (sum q_g)
            const float* ms = (const float*)(img + klo_at<D>()) + 4 * hf;
            auto scale = [&](int g, int j) { return *(const floatx4*)(ms + 32 * g + 8 * j); };
            half8 f[PF];
            floatx4 sc[4];
#pragma unroll
            for (int k = 0; k < PF; ++k)
                f[k] = frag(1024 * k);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                sc[j] = scale(0, j);
#pragma unroll
            for (int k = 0; k < NK; ++k) {
                hook(k);
#pragma unroll
                for (int c = 0; c < QT; ++c)
                    s[c] = mfma32(f[k % PF], k < NK - QL ? q[c][k] : fq[k - (NK - QL)], s[c]);
                if (k + PF >= NK - QL && k + PF < NK)
                    fq[k + PF - (NK - QL)] = query(k + PF);
                if (k + PF < NK)
                    f[k % PF] = frag(1024 * (k + PF));
                __builtin_amdgcn_sched_barrier(0);
                if (k % KS == KS - 1) {
                    // from group g's scale to the next group's (or out)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
#pragma unroll
                        for (int c = 0; c < QT; ++c)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                s[c][4 * j + i] *= sc[j][i];
                    }
                    if (k + 1 < NK) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            sc[j] = scale(k / KS + 1, j);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int j = 0; j < NZ; ++j) {
                float za = ms[32 * NG + 32 * min(2 * j + hf, NG - 1) + (lane & 31) - 4 * hf];
                za = 2 * j + hf < NG ? za : 0.0f;
#pragma unroll
                for (int c = 0; c < QT; ++c)
                    s[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(za, qz[c][j], s[c], 0, 0, 0);
            }
        } else {
            constexpr int PH = PF / 2;
            half8 fh[PH], fl[PH];
#pragma unroll
            for (int k = 0; k < PH; ++k) {
                fh[k] = frag(1024 * k);
                fl[k] = frag(klo_at<D>() + 1024 * k);
            }
#pragma unroll
            for (int k = 0; k < NK; ++k) {
                hook(k);
#pragma unroll
                for (int c = 0; c < QT; ++c) {
                    const half8 qk = k < NK - QL ? q[c][k] : fq[k - (NK - QL)];
                    s[c] = mfma32(fh[k % PH], qk, s[c]);
                    s[c] = mfma32(fl[k % PH], qk, s[c]);
                }
                if (k + PH >= NK - QL && k + PH < NK)
                    fq[k + PH - (NK - QL)] = query(k + PH);
                if (k + PH < NK) {
                    fh[k % PH] = frag(1024 * (k + PH));
                    fl[k % PH] = frag(klo_at<D>() + 1024 * (k + PH));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // Softmax of the scores and the value products of the same block; blk its
    // tail index (negative in the sink).
    __device__ __forceinline__ void update(const uint8_t* img, int blk, int lane)
    {
        const int hf = lane >> 5;
        const uint8_t* fb = img + 16 * lane;
        auto frag = [&](int at) { return __builtin_bit_cast(half8, *(const u32x4*)(fb + at)); };
        // the first value fragments, read while the softmax runs
        half8 vf[PF];
#pragma unroll
        for (int k = 0; k < PF; ++k)
            vf[k] = frag(vt_at<D>() + 1024 * k);
        if constexpr (D == 256)
            __builtin_amdgcn_s_setprio(0);
        // ---- online softmax per query column; P^T operands
        // The running maximum of a column is raised only when the block's
        // maximum exceeds it by more than 8 (log2 units): probabilities stay
        // below 2^8, and the accumulators are rescaled a few times per row,
        // not per block.  The column maximum needs the column's two lanes; it
        // is gathered only when some lane of the wave holds a score beyond its
        // running maximum + 8 (otherwise no column is raised).
        // Scores are in the units of the MFMA sums; a score times sscale is
        // the exponent (sscale > 0), and m is kept in exponent units.
        float lm[QT];
        bool up = false;
        const bool nomask = 32 * blk + 31 <= first;  // wave-uniform
#pragma unroll
        for (int c = 0; c < QT; ++c) {
            if (!nomask) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    s[c][e] = 32 * blk + 8 * (e >> 2) + 4 * hf + (e & 3) <= qpos[c] ? s[c][e] : -INFINITY;
            }
            lm[c] = s[c][0];
#pragma unroll
            for (int e = 1; e < 16; ++e)
                lm[c] = fmaxf(lm[c], s[c][e]);
            lm[c] *= sscale;
            up = up || lm[c] > m[c] + 8.0f;
        }
        if (__any(up)) {
#pragma unroll
            for (int c = 0; c < QT; ++c) {
                const float bm = fmaxf(lm[c], __shfl_xor(lm[c], 32));
                if (bm > m[c] + 8.0f) {
                    const float alpha = m[c] == -INFINITY ? 0.0f : fast_exp2(m[c] - bm);
                    m[c] = bm;
                    lsum[c] *= alpha;
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[c][t] *= alpha;
                }
            }
        }
        half8 ph[QT][2];
#pragma unroll
        for (int c = 0; c < QT; ++c) {
            // m is finite once a column has seen a key; a column that has not
            // takes 0, so that its masked -inf scores give 0, not NaN
            const float mn = m[c] == -INFINITY ? 0.0f : m[c];
            float ps = 0.0f;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float pv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    pv[e] = fast_exp2(fmaf(s[c][8 * u + e], sscale, -mn));
                    ps += pv[e];
                }
                ph[c][u] = pack_half8(pv);
            }
            lsum[c] += ps;
        }
        if constexpr (D == 256)
            __builtin_amdgcn_s_setprio(1);
        // ---- O^T += V^T P^T
#pragma unroll
        for (int k = 0; k < 2 * NT; ++k) {
#pragma unroll
            for (int c = 0; c < QT; ++c)
                acc[c][k / 2] = mfma32(vf[k % PF], ph[c][k & 1], acc[c][k / 2]);
            if (k + PF < 2 * NT)
                vf[k % PF] = frag(vt_at<D>() + 1024 * (k + PF));
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // Outputs (values were rotated back in the images: outputs are in the
    // original basis for every format): normalized to O, or with several key
    // ranges per tile this range's unnormalized partial and its (max, sum).
    __device__ __forceinline__ void finish(const AttnParams& p, const Tile& t, int split, int wave, int lane)
    {
        const int col = lane & 31, hf = lane >> 5;
#pragma unroll
        for (int c = 0; c < QT; ++c) {
            const float l = lsum[c] + __shfl_xor(lsum[c], 32);
            const int R = t.r0 + 32 * (QT * wave + c) + col;
            if (R >= t.rows)
                continue;
            float mul = 1.0f;
            float* dst;
            if (p.S_tot == 1) {
                mul = l > 0.0f ? 1.0f / l : 0.0f;
                dst = p.out + (((size_t)t.b * p.C + R / p.G) * p.H_q + (size_t)t.h * p.G + R % p.G) * D;
            } else {
                const size_t at = ((size_t)(t.unit - p.pf_u0) * p.S_tot + split) * t.rows + R;
                dst = p.part_o + at * D;
                if (hf == 0)
                    *(float2*)(p.part_ml + 2 * at) = make_float2(m[c], l);
            }
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    *(floatx4*)(dst + 32 * j + 8 * i + 4 * hf) =
                        floatx4{acc[c][j][4 * i], acc[c][j][4 * i + 1], acc[c][j][4 * i + 2], acc[c][j][4 * i + 3]} * mul;
        }
    }
};

// Workgroup w runs on XCD w mod 8: the contiguous range of work items an XCD
// takes shares a unit's blocks in its L2.
__device__ __forceinline__ int xcd_item()
{
    const int W = gridDim.x;
    return (W & 7) == 0 ? (blockIdx.x & 7) * (W >> 3) + (blockIdx.x >> 3) : blockIdx.x;
}

template <int D, int KG>
__global__ __launch_bounds__(threads<D>(), 2) void attn_kernel(AttnParams p)
{
    constexpr int NW = waves<D>(), QT = qtiles<D>();
    constexpr int BI = image_bytes<D>(), NST = stages<D>();
    constexpr int CW = BI / 1024 / NW;  // 1 KiB copies of an image per wave
    static_assert(CW * 1024 * NW == BI && CW <= D / 16, "whole copies, one beside a K fragment");
    extern __shared__ __attribute__((aligned(16))) uint8_t plds[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the longest (newest) tiles of a unit start first
    const int L = xcd_item(), uloc = __builtin_amdgcn_readfirstlane(L / p.pf_tiles);
    const Tile t = make_tile(p, p.pf_u0 + uloc, p.pf_tiles - 1 - (L - uloc * p.pf_tiles));
    Wave<D, KG, QT> w;
    w.init(p, t, plds + NST * BI, wave, lane);

    const uint32_t lbase = (uint32_t)(uintptr_t)plds;
    const uint8_t* ws_unit = p.pf_ws + (size_t)uloc * p.pf_nvb * BI;
    const uint32_t voff = 16 * lane;
    // copy k of this wave of image `it` (past the end: the last one again,
    // into a stage that is not read any more) into stage st
    auto image_at = [&](int it) {
        const int i = min(it, t.nvis - 1);
        return (uint64_t)(ws_unit + (size_t)(i < t.nsb ? i : p.pf_nsb + (i - t.nsb)) * BI) + 1024 * CW * wave;
    };
    auto copy = [&](uint64_t base, int st, int k) {
        copy16(base + 1024 * k, voff, lbase + (uint32_t)(st * BI + 1024 * (CW * wave + k)));
    };
    uint32_t m0_saved;
    asm volatile("s_mov_b32 %0, m0" : "=s"(m0_saved));
    // prologue: images 0 .. NST - 2 in flight, image 0 landed
#pragma unroll
    for (int it = 0; it < NST - 1; ++it) {
        const uint64_t base = image_at(it);
#pragma unroll
        for (int k = 0; k < CW; ++k)
            copy(base, it, k);
    }
    ring_sync(CW * (NST - 2));
    int stg = 0;  // stage of image it (it mod NST)
    for (int it = 0; it < t.nvis; ++it) {
        const int blk = it < t.nsb ? it - (p.sink >> 5) : it - t.nsb;
        const uint64_t base = image_at(it + NST - 1);
        const int pst = stg == 0 ? NST - 1 : stg - 1;  // the stage image it - 1 used
        const uint8_t* img = plds + stg * BI;
        // copies beside the first score steps, so that the wave never waits on
        // a burst of them (4% slower at the top of the block)
        w.scores(img, code_block<D>(p, it < t.nsb, blk), lane, [&](int k) {
            if (k < CW)
                copy(base, pst, k);
        });
        w.update(img, blk, lane);
        stg = stg + 1 == NST ? 0 : stg + 1;
        // image it + 1 has landed (all of this wave's copies but those of
        // the images after it), and no wave reads image it any more
        ring_sync(CW * (NST - 2));
    }
    asm volatile("s_mov_b32 m0, %0" ::"s"(m0_saved));
    __builtin_amdgcn_s_waitcnt(0);  // the trailing copies have landed before the LDS is given back
    w.finish(p, t, 0, wave, lane);
}

template <int D>
void (*pick(int kg))(AttnParams)
{
    return kg == 1   ? attn_kernel<D, (D >= 256 ? 0 : 1)>
           : kg == 2 ? attn_kernel<D, 2>
           : kg == 4 ? attn_kernel<D, (D >= 128 ? 4 : 1)>
           : kg == 8 ? attn_kernel<D, (D >= 256 ? 8 : 1)>
                     : attn_kernel<D, 0>;
}

template <int D>
hipError_t launch(const AttnParams& p0, size_t ws_bytes, hipStream_t stream)
{
    const int units = p0.B * p0.H;
    const bool rot = p0.rotate != 0;
    const size_t per_unit = (size_t)p0.pf_nvb * image_bytes<D>();
    const int group = (int)(ws_bytes / per_unit < (size_t)units ? ws_bytes / per_unit : (size_t)units);
    if (group < 1)
        return hipErrorInvalidValue;
    const int tiles = (p0.C * p0.G + kRows - 1) / kRows;
    const bool w8 = p0.k_bits == 8;  // 8-bit codes come as K and V both 8-bit
    void (*deq)(AttnParams) = w8 ? (rot ? dequant_kernel<D, true, true> : dequant_kernel<D, true, false>)
                                 : (rot ? dequant_kernel<D, false, true> : dequant_kernel<D, false, false>);
    // per-token key groups of 32 KG channels (a power of two from 32 to D)
    const int kg = p0.k_axis == KVQ_PER_TOKEN ? p0.k_group / 32 : 0;
    if (kg != 0 && kg != 1 && kg != 2 && !(kg == 4 && D >= 128) && !(kg == 8 && D >= 256))
        return hipErrorInvalidValue;
    void (*att)(AttnParams) = pick<D>(rot ? 0 : kg);
    for (int u0 = 0; u0 < units; u0 += group) {
        AttnParams p = p0;
        p.pf_u0 = u0;
        p.pf_tiles = tiles;
        p.S_tot = 1;
        const int nu = units - u0 < group ? units - u0 : group;
        launch_kernel(deq, dim3(p.pf_nvb, nu), dim3(kDqThreads), rot ? scratch_bytes<D>() : 0, stream, p);
        launch_kernel(att, dim3(tiles * nu), dim3(threads<D>()), attn_lds_bytes<D>(), stream, p);
    }
    return hipGetLastError();
}

}  // namespace pre

size_t prefill_image_bytes(int D)
{
    return (size_t)192 * D;
}

hipError_t launch_prefill(const AttnParams& p, int D, size_t ws_bytes, hipStream_t stream)
{
    switch (D) {
    case 64:
        return pre::launch<64>(p, ws_bytes, stream);
    case 128:
        return pre::launch<128>(p, ws_bytes, stream);
    case 256:
        return pre::launch<256>(p, ws_bytes, stream);
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace kvq
