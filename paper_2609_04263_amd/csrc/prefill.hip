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
// rotation; its keys are scaled by a power of two per eight tokens (see
// octet_exponent).  Two ways to the images, chosen by fused_splits:
//
//   workspace  dequant_kernel reconstructs every visible block of a unit
//              once into the caller's workspace and attn_kernel streams the
//              images through an LDS ring with global_load_lds_dwordx4.
//   fused      four waves of fused_kernel copy packed blocks into an LDS ring
//              and reconstruct them there, one block ahead of the four waves
//              that multiply: no image traffic, and the key range is split
//              over workgroups (partials in the workspace, combined by
//              merge_kernel) when the query tiles alone leave the chip idle.
//              A 128-token chunk at the end of 8001 tokens (B = 4, 32 query
//              heads on 8, D = 128, KIVI) had 64 workgroups: 398 -> 182 us;
//              32 tokens at the end of 8192 (B = 1): 350 -> 34 to 49 us.
//
// Each workgroup handles 128 or 256 query rows ((chunk token, head) pairs of a
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
// cores, was the limit (3500 cycles per block of 128 rows; now 4385 per block
// of 256, 2300 of them MFMA); 32 rows halve that, and take 128 accumulator and
// 64 query registers, which fits two waves per SIMD only because fragment
// order needs no address arithmetic.  A chunk of 2048 tokens at the end of
// 8192 (B = 8, 16 query heads on 8, D = 256): 2590 -> 2160 to 2280 us per call.
// Few tiles at D = 256 keep 16 rows per wave (Wave16).
// Sink tokens (fp16 rows) come first as blocks of their own; fp16 window
// tokens past the coded ones are read from the ring.

#include "kvq_device.h"
#include "kvq_internal.h"

namespace kvq {
namespace pre {

constexpr int kDqThreads = 256;

// Waves per workgroup of the workspace path: eight (one workgroup per CU, two
// waves per SIMD), four at D = 64, where two workgroups share a CU (each SIMD
// holds one wave of each, with independent per-block barriers).
template <int D>
constexpr int waves()
{
    return D == 64 ? 4 : 8;
}

constexpr int kRows = 256;  // query rows per workgroup

// 32-row query tiles per wave of the workspace path
template <int D>
constexpr int qtiles()
{
    return D == 64 ? 2 : 1;
}

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
template <int D, int KG>
__host__ __device__ constexpr int query_lds_fragments()
{
    return D == 256 && KG > 0 ? 2 : 0;
}

// the ring, then the query fragments
template <int D>
constexpr size_t attn_lds_bytes()
{
    return (size_t)stages<D>() * image_bytes<D>() + (size_t)waves<D>() * query_lds_fragments<D, 1>() * 1024;
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

// Whether a block (sink block when sinkblk, else tail block blk) is a code
// block: per-token key groups, no rotation, its tokens coded.
// Its image holds the key codes as exact fp16 values in place of k_hat's hi
// half, and the group scales and offsets in place of the lo half.  Groups of
// 32 at D = 256 (eight groups) keep hi + lo keys.
template <int D>
__device__ __forceinline__ bool code_block(const AttnParams& p, bool sinkblk, int blk)
{
    return p.k_axis == KVQ_PER_TOKEN && !p.rotate && !(D >= 256 && p.k_group == 32) && !sinkblk && 32 * blk < p.nq;
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
__host__ __device__ __forceinline__ SectionBytes section_bytes(const AttnParams& p)
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

// Rotation scratch: 8 rows (tokens) of D fp32 per wave, the pitch padded so
// that 16-byte reads of one channel chunk over consecutive rows hit distinct
// banks.  A wave rotates its own rows, and a wave's LDS accesses are performed
// in order, so no barrier is needed.
template <int D>
__host__ __device__ constexpr int scratch_pitch()
{
    return D + 4;
}

template <int D>
__host__ __device__ constexpr int scratch_bytes()  // of four waves
{
    return 4 * 8 * scratch_pitch<D>() * 4;
}

template <int N, int FIRST>
__device__ __forceinline__ void butterflies(float* v)
{
#pragma unroll
    for (int h = FIRST; h < N; h <<= 1)
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (!(e & h)) {
                const float s = v[e], t = v[e + h];
                v[e] = s + t;
                v[e + h] = s - t;
            }
}

// The compiler keeps the LDS accesses before and after in this order.
__device__ __forceinline__ void lds_order()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// In-place FWHT of the wave's 8 rows (butterflies of half width 1, 2, ..,
// D / 2), then * c: three half widths per pass in registers (1, 2, 4; 8, 16,
// 32; then 64 and 128).
template <int D>
__device__ __forceinline__ void fwht_rows8(float* x, int lane, float c)
{
    constexpr int PT = scratch_pitch<D>();
    lds_order();
#pragma unroll
    for (int i = lane; i < D; i += 64) {
        float* r = x + (i & 7) * PT + 8 * (i >> 3);
        const floatx4 a = *(const floatx4*)r, b = *(const floatx4*)(r + 4);
        float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        butterflies<8, 1>(v);
        *(floatx4*)r = floatx4{v[0], v[1], v[2], v[3]};
        *(floatx4*)(r + 4) = floatx4{v[4], v[5], v[6], v[7]};
    }
    lds_order();
#pragma unroll
    for (int i = lane; i < D; i += 64) {
        // lanes: eight channels of a 64-channel span, then rows, then spans
        float* r = x + ((i >> 3) & 7) * PT + 64 * (i >> 6) + (i & 7);
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = r[8 * e];
        butterflies<8, 1>(v);
#pragma unroll
        for (int e = 0; e < 8; ++e)
            r[8 * e] = D == 64 ? v[e] * c : v[e];
    }
    lds_order();
    if constexpr (D > 64) {
        constexpr int NV = D / 64;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float* r = x + i * PT + lane;
            float v[NV];
#pragma unroll
            for (int e = 0; e < NV; ++e)
                v[e] = r[64 * e];
            butterflies<NV, 1>(v);
#pragma unroll
            for (int e = 0; e < NV; ++e)
                r[64 * e] = v[e] * c;
        }
        lds_order();
    }
}

// Keys of a rotating format, eight tokens (an octet) at a time, are kept times a
// power of two that brings them below 2^12.  Binary16's range then holds any
// keys, and hi + lo is within 2^-23 of a key, or 2^-25 of the largest of its
// octet.  (A fixed 2^-4 in its place left an absolute error of 2^-21: rms 3e-4
// of keys of 1e-3, and keys from 2^20 on overflowed.)  The exponent comes from
// the octet's largest stored magnitude M < 2^(ef - 126), ef the exponent field
// of M: rotated back, a key is below sqrt(D) M <= 2^(ef - 122), and 2^(134 -
// ef) of it below 2^12.  ef is rounded up to a multiple of four, so that a
// block's four octets mostly share it and the softmax takes it as its factor;
// where they differ, the scores are brought to the largest first.
//
// The image has no room for the exponents, but bit 14 of every lo half is
// free: a lo half is at most 1 (half an ulp of a hi half below 2^12), and bit
// 14 is set from 2 on.  Bit i of octet j's ef is bit 14 of the lo half of
// token 8 j + i's channel D / 2, so a wave that has lo fragment D / 32 gathers
// all four exponents by one ballot.
//
// It costs rotating formats 2 to 3.5% of a call.  A power per block from its
// scales (no maximum over the keys) with one factor per block, or per key range
// of the fused path, cost as much.
constexpr uint32_t kExponentBit = 0x4000u;
constexpr int kExponentBias = 134;

// The value of lane l rotated by N within its 16-lane row
template <int N>
__device__ __forceinline__ uint32_t row_ror(uint32_t v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xF, 0xF, false);
}

// ef of the wave's largest |x| (mx: this lane's), from 8 to 252, so that
// 2^(ef - 134) and its inverse are normal numbers.
__device__ __forceinline__ int octet_exponent(float mx)
{
    uint32_t m = __float_as_uint(mx);  // not negative: ordered as integers
    m = max(m, row_ror<8>(m));
    m = max(m, row_ror<4>(m));
    m = max(m, row_ror<2>(m));
    m = max(m, row_ror<1>(m));
    const uint32_t a = max((uint32_t)__builtin_amdgcn_readlane(m, 0), (uint32_t)__builtin_amdgcn_readlane(m, 16));
    const uint32_t b = max((uint32_t)__builtin_amdgcn_readlane(m, 32), (uint32_t)__builtin_amdgcn_readlane(m, 48));
    return min(max((int)((max(a, b) >> 23) + 3) & ~3, 8), 252);
}

// fp32 -> fp16 hi + lo, each rounded to nearest: |v - hi - lo| <= 2^-23 |v|
// (2^-25 where lo is subnormal).  Cutting v to binary16 width for hi takes as
// many operations, but leaves a remainder of up to a whole ulp: twice the error.
__device__ __forceinline__ void split8(const float* v, half8* hi, half8* lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const _Float16 h = (_Float16)v[e];
        (*hi)[e] = h;
        (*lo)[e] = (_Float16)(v[e] - (float)h);
    }
}

// Where a rotated block's rows go back to the image: token tau's channels 8 P
// .. 8 P + 7 of the keys (mark: or'ed into the first lo half), and channel d of
// octet wv's values.
template <int D>
__device__ __forceinline__ void put_key(uint8_t* img, int tau, int P, const float* x, uint32_t mark = 0u)
{
    half8 h, l;
    split8(x, &h, &l);
    u32x4 lw = __builtin_bit_cast(u32x4, l);
    lw.x |= mark;
    *(u32x4*)(img + 512 * P + 16 * tau) = __builtin_bit_cast(u32x4, h);
    *(u32x4*)(img + klo_at<D>() + 512 * P + 16 * tau) = lw;
}

// mx: the largest magnitude this lane put into the rows.
template <int D>
__device__ __forceinline__ void rotate_keys(const AttnParams& p, uint8_t* img, float* rows, float mx, int wv, int lane)
{
    constexpr int PT = scratch_pitch<D>();
    const int ef = octet_exponent(mx);
    fwht_rows8<D>(rows, lane, p.rot_c * __uint_as_float((uint32_t)(127 + kExponentBias - ef) << 23));
#pragma unroll
    for (int i = lane; i < D; i += 64) {
        const float* src = rows + (i & 7) * PT + 8 * (i >> 3);
        const floatx4 a = *(const floatx4*)src, b = *(const floatx4*)(src + 4);
        const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        // (piece D / 16 holds channel D / 2)
        const bool mark = i >> 3 == D / 16 && ((ef >> (i & 7)) & 1);
        put_key<D>(img, 8 * wv + (i & 7), i >> 3, x, mark ? kExponentBit : 0u);
    }
    lds_order();  // the values follow through the same rows
}

template <int D>
__device__ __forceinline__ void rotate_values(const AttnParams& p, uint8_t* img, float* rows, int wv, int lane)
{
    constexpr int PT = scratch_pitch<D>();
    fwht_rows8<D>(rows, lane, p.rot_c);
#pragma unroll
    for (int d = lane; d < D; d += 64) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            x[e] = rows[e * PT + d];
        const u32x4 v = __builtin_bit_cast(u32x4, pack_half8(x));
        // octet wv is half wv % 2 of fragment chunks 2 (wv / 2) + {0, 1}
        uint8_t* dst = img + vt_at<D>() + 2048 * (d >> 5) + 1024 * (wv >> 1) + 16 * (d & 31) + 8 * (wv & 1);
        *(u32x2*)dst = u32x2{v.x, v.y};
        *(u32x2*)(dst + 512) = u32x2{v.z, v.w};
    }
    lds_order();
}

// ---- Images are built by four waves (tid 0 .. 255) without barriers, by block
// kind: a tail block of coded tokens, or one of fp16 rows (window or sink; the
// two never mix, since windows are coded 32 tokens at a time).  Tokens past the
// end are masked in the scores whatever their keys hold, and get zero values
// (0 times anything stored there must stay 0).
//
// Coded blocks.  The widths, the metadata type and the key axis are
// compile-time and their choice is made once per block: with them as run-time
// branches around every piece, a block took 6000 cycles (LDS latencies in
// series), three times its products.

// Eight codes as floats.  Conversions run at a quarter of the vector rate, so
// a byte of codes becomes the low mantissa byte of 2^23 (one permute) and 2^23
// is subtracted: exact, two full-rate operations.
template <int BITS>
struct Codes {
    uint32_t w[BITS == 8 ? 2 : 1];
};

template <int BITS>
__device__ __forceinline__ Codes<BITS> load_codes(const uint8_t* sec, int idx)
{
    Codes<BITS> c;
    if constexpr (BITS == 8) {
        const u32x2 v = ((const u32x2*)sec)[idx];
        c.w[0] = v.x;
        c.w[1] = v.y;
    } else if constexpr (BITS == 4) {
        c.w[0] = ((const uint32_t*)sec)[idx];
    } else {
        c.w[0] = ((const uint16_t*)sec)[idx];
    }
    return c;
}

__device__ __forceinline__ float byte_f32(uint32_t w, int k)
{
    return __uint_as_float(__builtin_amdgcn_perm(0x4B000000u, w, 0x070c0c00u | (uint32_t)k)) - 8388608.0f;
}

template <int BITS>
__device__ __forceinline__ void codes_f32(const Codes<BITS>& c, float* x)
{
    if constexpr (BITS == 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            x[e] = byte_f32(c.w[e >> 2], e & 3);
    } else if constexpr (BITS == 4) {
        const uint32_t a = c.w[0] & 0x0F0F0F0Fu, b = (c.w[0] >> 4) & 0x0F0F0F0Fu;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[2 * e] = byte_f32(a, e);
            x[2 * e + 1] = byte_f32(b, e);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t a = (c.w[0] >> (2 * e)) & 0x0303u;
            x[e] = byte_f32(a, 0);
            x[e + 4] = byte_f32(a, 1);
        }
    }
}

// N (4 or 8) consecutive scales or offsets from element i (a multiple of 4).
template <bool M16, int N>
__device__ __forceinline__ void meta_n(const uint8_t* sec, int i, float* v)
{
#pragma unroll
    for (int k = 0; k < N; k += 4) {
        if constexpr (M16) {
            const u32x2 h = *(const u32x2*)(sec + 2 * (i + k));
            v[k] = f16_bits_to_f32((uint16_t)h.x);
            v[k + 1] = f16_bits_to_f32((uint16_t)(h.x >> 16));
            v[k + 2] = f16_bits_to_f32((uint16_t)h.y);
            v[k + 3] = f16_bits_to_f32((uint16_t)(h.y >> 16));
        } else {
            const floatx4 a = *(const floatx4*)(sec + 4 * (i + k));
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[k + e] = a[e];
        }
    }
}

template <bool M16>
__device__ __forceinline__ float meta_1(const uint8_t* sec, int i)
{
    if constexpr (M16)
        return f16_bits_to_f32(((const uint16_t*)sec)[i]);
    else
        return ((const float*)sec)[i];
}

// Keys of a coded block, loads first: the
// compiler cannot tell the image's stores from the packed block's loads in
// LDS, so loads left beside their use would wait for each other.
// CK: a code block's exact codes, scales and offsets.  A reconstructed element
// is fma(c, s, z'), z' = z for affine codes and -2^(BITS - 1) s (exact) for
// symmetric ones, which is (c - 2^(BITS - 1)) s rounded once.
template <int D, int BITS, bool M16, bool AFF, bool PERCH, bool CK, bool ROT>
struct Keys {
    static constexpr int N = 4 * D / 256, NM = CK ? 1 : N, W = PERCH ? 8 : 1, PT = scratch_pitch<D>();
    Codes<BITS> c[N];
    float sc[NM][W], z[NM][W];

    // piece i of a thread: token tau, channels 8 P .. 8 P + 7 (a rotating wave
    // takes its own eight tokens)
    static __device__ __forceinline__ int tau(int tid) { return ROT ? 8 * (tid >> 6) + (tid & 7) : tid & 31; }
    static __device__ __forceinline__ int chunk(int tid, int i) { return (ROT ? (tid & 63) >> 3 : tid >> 5) + 8 * i; }

    __device__ __forceinline__ void load(const AttnParams& p, const Sections& s, int tid)
    {
        const uint8_t* sz = AFF || p.k_mode == KVQ_AFFINE ? s.kz : s.ks;  // symmetric: any readable address
        const int lg = PERCH ? 0 : 31 - __builtin_clz(p.k_group), t = tau(tid);
        const int r = 4 * (t >> 3) + (t & 3), half = (t >> 2) & 1;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int P = chunk(tid, i);
            c[i] = load_codes<BITS>(s.kc, (half * 64 + r + 16 * (P & 3)) * (D / 32) + (P >> 2));
            if constexpr (CK) {
                continue;
            } else if constexpr (PERCH) {
                meta_n<M16, 8>(s.ks, 8 * P, sc[i]);
                meta_n<M16, 8>(sz, 8 * P, z[i]);
            } else {
                const int mi = ((8 * P) >> lg) * 32 + t;
                sc[i][0] = meta_1<M16>(s.ks, mi);
                z[i][0] = meta_1<M16>(sz, mi);
            }
        }
    }

    __device__ __forceinline__ void finish(const AttnParams& p, const Sections& s, int valid, uint8_t* img, float* scratch,
                                           int tid)
    {
        const bool aff = AFF || p.k_mode == KVQ_AFFINE;
        constexpr float nh = -(float)(1 << (BITS - 1));
        const int lane = tid & 63, wv = tid >> 6, t = tau(tid);
        float mx = 0.0f;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int P = chunk(tid, i);
            float x[8];
            codes_f32<BITS>(c[i], x);
            if constexpr (CK) {
                *(u32x4*)(img + 512 * P + 16 * t) = __builtin_bit_cast(u32x4, pack_half8(x));
                continue;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = PERCH ? e : 0, m = CK ? 0 : i;
                x[e] = fmaf(x[e], sc[m][k], aff ? z[m][k] : nh * sc[m][k]);
            }
            if constexpr (ROT) {
                // (what dead tokens hold must not set the octet's exponent)
                if (valid < 32) {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        x[e] = t < valid ? x[e] : 0.0f;
                }
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    mx = fmaxf(mx, fabsf(x[e]));
                float* dst = scratch + t * PT + 8 * P;
                *(floatx4*)dst = floatx4{x[0], x[1], x[2], x[3]};
                *(floatx4*)(dst + 4) = floatx4{x[4], x[5], x[6], x[7]};
            } else {
                put_key<D>(img, t, P, x);
            }
        }
        if constexpr (ROT)
            rotate_keys<D>(p, img, scratch + wv * 8 * PT, mx, wv, lane);
        if constexpr (CK) {
            // the scales s (fp32, in place of the lo half), then the offsets z'
            const int n = 32 * (D >> (31 - __builtin_clz(p.k_group)));
            const uint8_t* sz = aff ? s.kz : s.ks;
            float* ms = (float*)(img + klo_at<D>());
            for (int i = tid; i < n; i += 256) {
                const float s0 = meta_1<M16>(s.ks, i), z0 = meta_1<M16>(sz, i);
                ms[i] = s0;
                ms[n + i] = aff ? z0 : nh * s0;
            }
        }
    }
};

// Values of a coded block, the first `valid` tokens live.  Wave wv takes fragment chunk wv = 2 u + h:
// codes 4 h .. 4 h + 3 of octets 2 u and 2 u + 1 (a rotating wave octet wv).
template <int D, int BITS, bool M16, bool AFF, bool ROT>
struct Values {
    static constexpr int N = D / 64, PT = scratch_pitch<D>();
    Codes<BITS> c[N][ROT ? 1 : 2];
    float sc[N][8], z[N][8];

    __device__ __forceinline__ void load(const AttnParams& p, const Sections& s, int tid)
    {
        const uint8_t* sz = AFF || p.v_mode == KVQ_AFFINE ? s.vz : s.vs;
        const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), u = wv >> 1, h = wv & 1;
        const int lg = 31 - __builtin_clz(p.v_group);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int d = lane + 64 * i, at = d % 16 * (D / 16) + d / 16, mg = (d >> lg) * 32;
            if constexpr (ROT) {
                c[i][0] = load_codes<BITS>(s.vc, at + 16 * wv * (D / 16));
                meta_n<M16, 8>(s.vs, mg + 8 * wv, sc[i]);
                meta_n<M16, 8>(sz, mg + 8 * wv, z[i]);
            } else {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    c[i][j] = load_codes<BITS>(s.vc, at + 16 * (2 * u + j) * (D / 16));
                    meta_n<M16, 4>(s.vs, mg + 16 * u + 8 * j + 4 * h, sc[i] + 4 * j);
                    meta_n<M16, 4>(sz, mg + 16 * u + 8 * j + 4 * h, z[i] + 4 * j);
                }
            }
        }
    }

    __device__ __forceinline__ void finish(const AttnParams& p, int valid, uint8_t* img, float* scratch, int tid)
    {
        const bool aff = AFF || p.v_mode == KVQ_AFFINE;
        constexpr float nh = -(float)(1 << (BITS - 1));
        const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = wv & 1;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int d = lane + 64 * i;
            float x[8];
            if constexpr (ROT) {
                codes_f32<BITS>(c[i][0], x);
            } else {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    // the codes of four tokens at the bottom (8-bit: in one word)
                    const uint32_t w0 = c[i][j].w[0], w1 = c[i][j].w[BITS == 8];
                    const uint32_t w = BITS == 8 ? w0 ^ ((w0 ^ w1) & (uint32_t)-h) : w0 >> (4 * BITS * h);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        x[4 * j + e] = BITS == 8   ? byte_f32(w, e)
                                       : BITS == 4 ? byte_f32((e & 1) ? (w >> 4) & 0x0F0Fu : w & 0x0F0Fu, e >> 1)
                                                   : byte_f32((w >> (2 * e)) & 3u, 0);
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e)
                x[e] = fmaf(x[e], sc[i][e], aff ? z[i][e] : nh * sc[i][e]);
            if (valid < 32) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    x[e] = (ROT ? 8 * wv + e : 16 * (wv >> 1) + 4 * h + 8 * (e >> 2) + (e & 3)) < valid ? x[e] : 0.0f;
            }
            if constexpr (ROT) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    scratch[(wv * 8 + e) * PT + d] = x[e];
            } else {
                *(u32x4*)(img + vt_at<D>() + 2048 * (d >> 5) + 512 * wv + 16 * (d & 31)) =
                    __builtin_bit_cast(u32x4, pack_half8(x));
            }
        }
        if constexpr (ROT)
            rotate_values<D>(p, img, scratch + wv * 8 * PT, wv, lane);
    }
};

// The image of a coded block; CK as code_block says.
template <int D, int KB, int VB, bool M16, bool AFF, bool PERCH, bool CK, bool ROT>
__device__ __forceinline__ void coded_blocks(const AttnParams& p, const Sections& s, int valid, uint8_t* img, float* scratch, int tid)
{
    Keys<D, KB, M16, AFF, PERCH, CK, ROT> k;
    Values<D, VB, M16, AFF, ROT> v;
    k.load(p, s, tid);
    v.load(p, s, tid);
    k.finish(p, s, valid, img, scratch, tid);
    v.finish(p, valid, img, scratch, tid);
}

template <int D, int KB, int VB, bool M16, bool AFF, bool CK, bool ROT>
__device__ __forceinline__ void coded_axis(const AttnParams& p, const Sections& s, int valid, uint8_t* img, float* scratch, int tid)
{
    if constexpr (CK) {
        coded_blocks<D, KB, VB, M16, AFF, false, true, false>(p, s, valid, img, scratch, tid);
    } else {
        if (p.k_axis == KVQ_PER_CHANNEL)
            coded_blocks<D, KB, VB, M16, AFF, true, false, ROT>(p, s, valid, img, scratch, tid);
        else if constexpr (ROT || D == 256)  // (other per-token keys are code blocks)
            coded_blocks<D, KB, VB, M16, AFF, false, false, ROT>(p, s, valid, img, scratch, tid);
    }
}

template <int D, bool W8, bool M16, bool AFF, bool CK, bool ROT>
__device__ __forceinline__ void coded_bits(const AttnParams& p, const Sections& s, int valid, uint8_t* img, float* scratch, int tid)
{
    if constexpr (W8) {
        coded_axis<D, 8, 8, M16, AFF, CK, ROT>(p, s, valid, img, scratch, tid);
    } else if (p.k_bits == 4) {
        if (p.v_bits == 4)
            coded_axis<D, 4, 4, M16, AFF, CK, ROT>(p, s, valid, img, scratch, tid);
        else
            coded_axis<D, 4, 2, M16, AFF, CK, ROT>(p, s, valid, img, scratch, tid);
    } else {
        if (p.v_bits == 4)
            coded_axis<D, 2, 4, M16, AFF, CK, ROT>(p, s, valid, img, scratch, tid);
        else
            coded_axis<D, 2, 2, M16, AFF, CK, ROT>(p, s, valid, img, scratch, tid);
    }
}

template <int D, bool W8, bool CK, bool ROT>
__device__ __forceinline__ void coded_image(const AttnParams& p, const Sections& s, int valid, uint8_t* img, float* scratch,
                                            int tid)
{
    if (p.meta16)
        coded_bits<D, W8, true, false, CK, ROT>(p, s, valid, img, scratch, tid);
    else if (p.k_mode == KVQ_AFFINE && p.v_mode == KVQ_AFFINE)
        coded_bits<D, W8, false, true, CK, ROT>(p, s, valid, img, scratch, tid);
    else
        coded_bits<D, W8, false, false, CK, ROT>(p, s, valid, img, scratch, tid);
}

// The image of a block of fp16 rows: token i is row (first + i) % ring of kr, vr
// [.][D], the first `valid` tokens live.  All loads first, as above.
template <int D, bool ROT>
__device__ __forceinline__ void fp16_image(const AttnParams& p, const uint16_t* kr, const uint16_t* vr, int first, int ring,
                                           int valid, uint8_t* img, float* scratch, int tid)
{
    constexpr int N = 4 * D / 256, NV = D / 64, PT = scratch_pitch<D>();
    using K = Keys<D, 2, false, false, false, true, ROT>;
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), t = K::tau(tid);
    u32x4 kw[N];
    uint16_t vw[NV][8];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        kw[i] = u32x4{0u, 0u, 0u, 0u};
        if (t < valid)
            kw[i] = *(const u32x4*)(kr + (size_t)((first + t) % ring) * D + 8 * K::chunk(tid, i));
    }
    int row[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int tok = ROT ? 8 * wv + e : 16 * (wv >> 1) + 4 * (wv & 1) + 8 * (e >> 2) + (e & 3);
        row[e] = tok < valid ? (first + tok) % ring : -1;
    }
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e)
            vw[i][e] = row[e] >= 0 ? vr[(size_t)row[e] * D + lane + 64 * i] : (uint16_t)0;
    float mx = 0.0f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int P = K::chunk(tid, i);
        if constexpr (ROT) {
            const uint32_t w[4] = {kw[i].x, kw[i].y, kw[i].z, kw[i].w};
            float* dst = scratch + t * PT + 8 * P;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                dst[e] = f16_bits_to_f32((uint16_t)(w[e >> 1] >> (16 * (e & 1))));
                mx = fmaxf(mx, fabsf(dst[e]));
            }
        } else {
            *(u32x4*)(img + 512 * P + 16 * t) = kw[i];
            *(u32x4*)(img + klo_at<D>() + 512 * P + 16 * t) = u32x4{0u, 0u, 0u, 0u};
        }
    }
    if constexpr (ROT)
        rotate_keys<D>(p, img, scratch + wv * 8 * PT, mx, wv, lane);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int d = lane + 64 * i;
        if constexpr (ROT) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                scratch[(wv * 8 + e) * PT + d] = f16_bits_to_f32(vw[i][e]);
        } else {
            u32x4 v;
            v.x = vw[i][0] | ((uint32_t)vw[i][1] << 16);
            v.y = vw[i][2] | ((uint32_t)vw[i][3] << 16);
            v.z = vw[i][4] | ((uint32_t)vw[i][5] << 16);
            v.w = vw[i][6] | ((uint32_t)vw[i][7] << 16);
            *(u32x4*)(img + vt_at<D>() + 2048 * (d >> 5) + 512 * wv + 16 * (d & 31)) = v;
        }
    }
    if constexpr (ROT)
        rotate_values<D>(p, img, scratch + wv * 8 * PT, wv, lane);
}

// fp16_image of sink block sb (sb >= 0), or of the window's tail block blk.
template <int D, bool ROT>
__device__ __forceinline__ void rows_image(const AttnParams& p, int unit, int sb, int blk, uint8_t* img, float* scratch, int tid)
{
    if (sb >= 0) {
        const size_t at = (size_t)unit * p.sink * D;
        fp16_image<D, ROT>(p, p.kq + at, p.vq + at, 32 * sb, p.sink, p.n_sink - 32 * sb, img, scratch, tid);
    } else {
        const size_t at = (size_t)unit * p.ring * D;
        fp16_image<D, ROT>(p, p.kr + at, p.vr + at, 32 * blk, p.ring, p.n - 32 * blk, img, scratch, tid);
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
    const int valid = min(32, p.nq - 32 * blk);
    if (sinkblk || valid <= 0)
        rows_image<D, ROT>(p, unit, sinkblk ? v : -1, blk, img, dq_scratch, threadIdx.x);
    else if (!ROT && code_block<D>(p, false, blk))
        coded_image<D, W8, !ROT, ROT>(p, s, valid, img, dq_scratch, threadIdx.x);
    else
        coded_image<D, W8, false, ROT>(p, s, valid, img, dq_scratch, threadIdx.x);
}

// ---------------------------------------------------------------------------
// 2. Attention over block images in LDS.

// 16 bytes per lane from global memory to LDS address lds_addr + 16 lane
// (lds_addr wave-uniform, held in M0 while the copy issues).  Inline
// assembly, so that the compiler does not make LDS reads wait for every
// outstanding copy; the kernel's own vmcnt waits order them.
// The hardware needs one wait state between a scalar write of M0 and an LDS
// load that reads it; inside an assembly string the compiler adds none.
__device__ __forceinline__ void copy16(uint64_t base, uint32_t voff, uint32_t lds_addr)
{
    const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds_addr);
    // (the builtin returns int: widen both halves as unsigned, or a low
    // word with bit 31 set would be sign-extended into the high word)
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)base);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
    const uint64_t sb = ((uint64_t)hi << 32) | (uint64_t)lo;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(m0v), "v"(voff), "s"(sb) : "memory");
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
// copies have landed, then every wave is past the same point.  Products of the
// stage that is given back must not sink below: a fragment they wait for could
// still be on its way from LDS when another wave's copy overwrites it.
__device__ __forceinline__ void ring_sync(int after)
{
    __builtin_amdgcn_sched_barrier(0);
    wait_vm(after);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Query rows of a workgroup: rows r0 .. r0 + per - 1 of a unit.  Positions are
// tail indices (token minus sink); sink tokens sit at -sink .. -1, so a chunk
// that starts in the sink has negative positions.
struct Tile {
    int unit, b, h;  // unit = b H + h
    int r0, rows;
    int nsb, nvis;   // sink blocks and all blocks that hold a visible token
};

__device__ __forceinline__ Tile make_tile(const AttnParams& p, int unit, int tile, int per)
{
    Tile t;
    t.unit = unit;
    t.b = __builtin_amdgcn_readfirstlane(unit / p.H);
    t.h = unit - t.b * p.H;
    t.rows = p.C * p.G;
    t.r0 = tile * per;
    const int newest = __builtin_amdgcn_readfirstlane(p.n - p.C + (min(t.r0 + per, t.rows) - 1) / p.G);
    const int nkb = newest >= 0 ? newest / 32 + 1 : 0;  // coded-tail blocks
    t.nsb = min((p.n_sink + 31) >> 5, (newest + p.sink) / 32 + 1);
    t.nvis = t.nsb + nkb;
    return t;
}

constexpr int kNoRow = -(1 << 30);  // position of a query row past the end: every key masked

// Queries are scaled by qscale (returned), sm_scale log2(e) rounded down to a
// power of two (exact in fp16 below 65504), and the scores take the rest, sscale
// (qscale keeps the sign of the scale, so sscale > 0; a zero or subnormal scale
// gives zero queries, zero scores, sscale 1).
__device__ __forceinline__ float query_scales(const AttnParams& p, float* sscale)
{
    const float qscale = __uint_as_float(__float_as_uint(p.sm_log2) & 0xFF800000u);
    const float rest = qscale == 0.0f ? 1.0f : p.sm_log2 / qscale;
    *sscale = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(rest)));  // a scalar register
    return qscale;
}

// One wave's state: 32 QT query rows (columns of the MFMAs: column l % 32 of
// tile q is row r0 + 32 (QT wave + q) + l % 32).  KG: key group size / 32 when
// the format's keys have per-token groups (code blocks then take exact code
// operands), 0 otherwise.  ROT: a rotating format (KG = 0), whose keys carry an
// exponent per eight tokens.
template <int D, int KG, int QT, bool ROT>
struct Wave {
    static constexpr int kRows = 32 * QT;
    static constexpr int NK = D / 16, NT = D / 32;        // K fragments, 32-channel value tiles
    static constexpr int KS = KG > 0 ? 2 * KG : NK;       // K fragments per group
    static constexpr int NG = NK / KS, NZ = (NG + 1) / 2;  // groups, offset MFMAs per tile
    static constexpr int PF = D == 256 ? 3 : 4;  // fragments read ahead (LDS latency)
    // The last QL query fragments of a wave live in LDS (the 16 KiB that the
    // ring leaves free at D = 256, where the registers do not hold them all).
    static constexpr int QL = query_lds_fragments<D, KG>();
    half8 q[QT][NK - QL];
    uint8_t* ql;
    float qz[QT][NZ];  // lane (col, h): the query's sum over group 2 j + h
    int qpos[QT];
    float sscale;      // scores times sscale are exponents (base 2)
    float bscale;      // ROT: the same for the scores of the present block
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
        const float qscale = query_scales(p, &sscale);
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
            floatx16 g[QT];
            const auto offsets = [&] {
#pragma unroll
                for (int j = 0; j < NZ; ++j) {
                    float za = ms[32 * NG + 32 * min(2 * j + hf, NG - 1) + (lane & 31) - 4 * hf];
                    za = 2 * j + hf < NG ? za : 0.0f;
#pragma unroll
                    for (int c = 0; c < QT; ++c)
                        s[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(za, qz[c][j], s[c], 0, 0, 0);
                }
            };
#pragma unroll
            for (int k = 0; k < PF; ++k)
                f[k] = frag(1024 * k);
            // One sum per group, then one FMA by its scale as stored.  (A single
            // sum moved from each group's scale to the next by their ratio
            // takes 16 registers less, but has twice the rounding error: 1.8e-7
            // against 0.8e-7 of a score at D = 256 with four groups.)  At D =
            // 256 the registers do not hold the scales ahead: half are read
            // beside the group's last product, half after it, and the offsets
            // come last, 2 to 4% slower than the ratios.
            constexpr bool kLate = D == 256;
            floatx4 sc[4];
            if (!kLate) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    sc[j] = scale(0, j);
                offsets();
            }
#pragma unroll
            for (int k = 0; k < NK; ++k) {
                hook(k);
                if (kLate && k % KS == KS - 1) {
                    sc[0] = scale(k / KS, 0);
                    sc[1] = scale(k / KS, 1);
                }
#pragma unroll
                for (int c = 0; c < QT; ++c)
                    g[c] = mfma32(f[k % PF], k < NK - QL ? q[c][k] : fq[k - (NK - QL)], k % KS == 0 ? floatx16{} : g[c]);
                if (k + PF >= NK - QL && k + PF < NK)
                    fq[k + PF - (NK - QL)] = query(k + PF);
                if (k + PF < NK)
                    f[k % PF] = frag(1024 * (k + PF));
                __builtin_amdgcn_sched_barrier(0);
                if (k % KS == KS - 1) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const floatx4 v = kLate && j >= 2 ? scale(k / KS, j) : sc[j];
#pragma unroll
                        for (int c = 0; c < QT; ++c)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                s[c][4 * j + i] = kLate && k < KS ? v[i] * g[c][4 * j + i] : fmaf(v[i], g[c][4 * j + i], s[c][4 * j + i]);
                        if (kLate && j & 1)
                            __builtin_amdgcn_sched_barrier(0);
                    }
                    if (!kLate && k + 1 < NK) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            sc[j] = scale(k / KS + 1, j);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (kLate)
                offsets();
        } else {
            constexpr int PH = PF / 2;
            half8 fh[PH], fl[PH];
            uint32_t ef = 0;  // ROT: the octets' exponents, a byte each
#pragma unroll
            for (int k = 0; k < PH; ++k) {
                fh[k] = frag(1024 * k);
                fl[k] = frag(klo_at<D>() + 1024 * k);
            }
#pragma unroll
            for (int k = 0; k < NK; ++k) {
                hook(k);
                if constexpr (ROT) {
                    if (k == NK / 2) {
                        u32x4 w = __builtin_bit_cast(u32x4, fl[k % PH]);
                        ef = (uint32_t)__ballot((w.x & kExponentBit) != 0);
                        w.x &= ~kExponentBit;
                        fl[k % PH] = __builtin_bit_cast(half8, w);
                    }
                }
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
            if constexpr (ROT) {
                int top = (int)(ef & 0xFFu);
                if (ef != (uint32_t)top * 0x01010101u) {
#pragma unroll
                    for (int j = 1; j < 4; ++j)
                        top = max(top, (int)(ef >> (8 * j) & 0xFFu));
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        // octet j is the elements 4 j .. 4 j + 3
                        const int d = 127 + (int)(ef >> (8 * j) & 0xFFu) - top;
                        const float f = __uint_as_float((uint32_t)max(d, 0) << 23);
#pragma unroll
                        for (int c = 0; c < QT; ++c)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                s[c][4 * j + i] *= f;
                    }
                }
                bscale = __uint_as_float(__float_as_uint(sscale) + ((uint32_t)(top - kExponentBias) << 23));
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
        // step k: channel tile k % NT, token half k / NT
        auto vfrag = [](int k) { return vt_at<D>() + 1024 * (2 * (k % NT) + k / NT); };
        // the first value fragments, read while the softmax runs
        half8 vf[PF];
#pragma unroll
        for (int k = 0; k < PF; ++k)
            vf[k] = frag(vfrag(k));
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
            lm[c] *= ROT ? bscale : sscale;
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
                    pv[e] = fast_exp2(fmaf(s[c][8 * u + e], ROT ? bscale : sscale, -mn));
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
                acc[c][k % NT] = mfma32(vf[k % PF], ph[c][k / NT], acc[c][k % NT]);
            if (k + PF < 2 * NT)
                vf[k % PF] = frag(vfrag(k + PF));
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // Outputs (values were rotated back in the images: outputs are in the
    // original basis for every format): normalized to O, or with several key
    // ranges per tile this range's unnormalized partial (the first range's to
    // O, the others' to part_o [unit][S - 1][rows][D]) and its (max, sum).
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
            float* dst = p.out + (((size_t)t.b * p.C + R / p.G) * p.H_q + (size_t)t.h * p.G + R % p.G) * D;
            if (p.S_tot == 1) {
                mul = l > 0.0f ? 1.0f / l : 0.0f;
            } else {
                const size_t uloc = t.unit - p.pf_u0;
                if (split > 0)
                    dst = p.part_o + ((uloc * (p.S_tot - 1) + split - 1) * t.rows + R) * D;
                if (hf == 0)
                    *(float2*)(p.part_ml + 2 * ((uloc * p.S_tot + split) * t.rows + R)) = make_float2(m[c], l);
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

// Wave with 16 query rows at D = 256, on v_mfma_f32_16x16x32_f16 (column l % 16
// of a wave is one row).  It reads every fragment for half the rows, which
// makes LDS its limit in long grids, but a tile of eight waves has 128 rows:
// where tiles of 256 leave CUs idle, or the last ones to run are the longest,
// twice the tiles are worth more (see small_tiles).
//
// Score row 4 (l / 16) + i of key tile kt is token 16 u + 4 ((l / 16) & 1) + 8 (kt
// ^ u) + i, u = l / 32: a lane's eight scores are the key slots of one 16-byte
// piece of the image's value fragments (its halves swapped where u = 1), and the
// 16 rows of a K read lie in distinct banks (with kt for kt ^ u they met in half
// of them).
template <int KG, bool ROT>
struct Wave16 {
    static constexpr int D = 256, kRows = 16;
    static constexpr int NKS = D / 32, NCT = D / 16;   // K steps, 16-channel value tiles
    static constexpr int KS = KG > 0 ? KG : NKS, NG = NKS / KS;
    static_assert(NG <= 4, "one offset product per key tile");
    half8 q[NKS];
    float qz;       // lane (col, qg): the query's sum over group qg
    int qpos;
    float sscale;   // scores times sscale are exponents (base 2)
    float bscale;   // ROT: the same for the scores of the present block
    int first;      // position of the wave's oldest query when all its rows exist
    floatx4 acc[NCT];
    floatx4 s[2];   // the scores of the block between scores() and update()
    float m, lsum;

    static __device__ __forceinline__ int token(int qg, int kt) { return 16 * (qg >> 1) + 4 * (qg & 1) + 8 * (kt ^ (qg >> 1)); }

    __device__ __forceinline__ void init(const AttnParams& p, const Tile& t, uint8_t*, int wave, int lane)
    {
        const int col = lane & 15, qg = lane >> 4;
        const float qscale = query_scales(p, &sscale);
        const int first_pos = p.n - p.C, wrow0 = t.r0 + kRows * wave, R = wrow0 + col;
        first = __builtin_amdgcn_readfirstlane(wrow0 + kRows <= t.rows ? first_pos + wrow0 / p.G : kNoRow);
        const int i = R / p.G, g = R % p.G;
        const uint16_t* src = p.q + (((size_t)t.b * p.C + i) * p.H_q + (size_t)t.h * p.G + g) * D + 8 * qg;
        float qsum[NG];
#pragma unroll
        for (int j = 0; j < NG; ++j)
            qsum[j] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            u32x4 w = {0u, 0u, 0u, 0u};
            if (R < t.rows)
                w = *(const u32x4*)(src + 32 * ks);
            const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
            float v[8], part = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[e] = __uint_as_float((e & 1) ? (ww[e >> 1] & 0xFFFF0000u) : (ww[e >> 1] << 16)) * qscale;
                part += v[e];
            }
            q[ks] = pack_half8(v);
            qsum[ks / KS] += part;
        }
        qz = 0.0f;
        if (KG > 0) {
            // the column's four lanes hold a quarter of every group each
#pragma unroll
            for (int j = 0; j < NG; ++j) {
                float sum = qsum[j] + __shfl_xor(qsum[j], 16);
                sum += __shfl_xor(sum, 32);
                qz = qg == j ? sum : qz;
            }
        }
        qpos = R < t.rows ? first_pos + i : kNoRow;
        m = -INFINITY;
        lsum = 0.0f;
#pragma unroll
        for (int j = 0; j < NCT; ++j)
            acc[j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    template <typename Hook>
    __device__ __forceinline__ void scores(const uint8_t* img, bool code, int lane, Hook hook)
    {
        const int col = lane & 15, qg = lane >> 4;
        const int row[2] = {token(col >> 2, 0) + (col & 3), token(col >> 2, 1) + (col & 3)};  // this lane's K rows
        const uint8_t* kb[2] = {img + 512 * qg + 16 * row[0], img + 512 * qg + 16 * row[1]};
        // step ks, key tile kt of a part: 32 channels of 16 tokens
        auto frag = [&](int part, int ks, int kt) {
            return __builtin_bit_cast(half8, *(const u32x4*)(kb[kt] + part + 2048 * ks));
        };
        s[0] = s[1] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        if (KG > 0 && code) {
            const float* ms = (const float*)(img + klo_at<D>());
            half8 f[2][2];
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                f[0][kt] = frag(0, 0, kt);
                const float za = ms[32 * NG + 32 * min(qg, NG - 1) + row[kt]];
                s[kt] = __builtin_amdgcn_mfma_f32_16x16x4f32(qg < NG ? za : 0.0f, qz, s[kt], 0, 0, 0);
            }
            floatx4 g[2], sc[2];
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                hook(2 * ks);
                if (ks % KS == 0) {
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt) {
                        g[kt] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
                        sc[kt] = *(const floatx4*)(ms + 32 * (ks / KS) + token(qg, kt));
                    }
                }
                if (ks + 1 < NKS) {
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt)
                        f[(ks + 1) & 1][kt] = frag(0, ks + 1, kt);
                }
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
                    g[kt] = mfma16(f[ks & 1][kt], q[ks], g[kt]);
                hook(2 * ks + 1);
                if (ks % KS == KS - 1) {
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            s[kt][i] = fmaf(sc[kt][i], g[kt][i], s[kt][i]);
                }
            }
        } else {
            half8 fh[2][2], fl[2][2];
            uint32_t ef = 0;  // ROT: the octets' exponents, a byte each
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                fh[0][kt] = frag(0, 0, kt);
                fl[0][kt] = frag(klo_at<D>(), 0, kt);
            }
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                hook(2 * ks);
                if (ks + 1 < NKS) {
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt) {
                        fh[(ks + 1) & 1][kt] = frag(0, ks + 1, kt);
                        fl[(ks + 1) & 1][kt] = frag(klo_at<D>(), ks + 1, kt);
                    }
                }
                if constexpr (ROT) {
                    if (ks == NKS / 2) {
                        // channel D / 2 (octet_exponent): lanes 0 .. 7 hold octet kt,
                        // lanes 8 .. 15 octet 3 - kt
#pragma unroll
                        for (int kt = 0; kt < 2; ++kt) {
                            u32x4 w = __builtin_bit_cast(u32x4, fl[ks & 1][kt]);
                            const uint32_t b = (uint32_t)__ballot((w.x & kExponentBit) != 0);
                            ef |= (b & 0xFFu) << (8 * kt) | (b >> 8 & 0xFFu) << (24 - 8 * kt);
                            w.x &= ~kExponentBit;
                            fl[ks & 1][kt] = __builtin_bit_cast(half8, w);
                        }
                    }
                }
#pragma unroll
                for (int kt = 0; kt < 2; ++kt) {
                    s[kt] = mfma16(fh[ks & 1][kt], q[ks], s[kt]);
                    s[kt] = mfma16(fl[ks & 1][kt], q[ks], s[kt]);
                }
                hook(2 * ks + 1);
            }
            if constexpr (ROT) {
                int top = (int)(ef & 0xFFu);
                if (ef != (uint32_t)top * 0x01010101u) {
#pragma unroll
                    for (int j = 1; j < 4; ++j)
                        top = max(top, (int)(ef >> (8 * j) & 0xFFu));
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt) {
                        const int e = (int)(ef >> (token(qg, kt) & 24) & 0xFFu);  // octet token / 8
                        s[kt] *= __uint_as_float((uint32_t)max(127 + e - top, 0) << 23);
                    }
                }
                bscale = __uint_as_float(__float_as_uint(sscale) + ((uint32_t)(top - kExponentBias) << 23));
            }
        }
    }

    __device__ __forceinline__ void update(const uint8_t* img, int blk, int lane)
    {
        const int col = lane & 15, qg = lane >> 4;
        const uint8_t* vb = img + vt_at<D>() + 512 * qg + 16 * col;
        auto vfrag = [&](int c) { return __builtin_bit_cast(half8, *(const u32x4*)(vb + 2048 * (c >> 1) + 256 * (c & 1))); };
        constexpr int PF = 3;
        half8 vf[PF];
#pragma unroll
        for (int c = 0; c < PF; ++c)
            vf[c] = vfrag(c);
        const float scale = ROT ? bscale : sscale;
        if (!(32 * blk + 31 <= first)) {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    s[kt][i] = 32 * blk + token(qg, kt) + i <= qpos ? s[kt][i] : -INFINITY;
        }
        float lm = s[0][0];
#pragma unroll
        for (int e = 1; e < 8; ++e)
            lm = fmaxf(lm, s[e >> 2][e & 3]);
        lm *= scale;
        // (the running maximum as in Wave::update)
        if (__any(lm > m + 8.0f)) {
            float bm = fmaxf(lm, __shfl_xor(lm, 16));
            bm = fmaxf(bm, __shfl_xor(bm, 32));
            if (bm > m + 8.0f) {
                const float alpha = m == -INFINITY ? 0.0f : fast_exp2(m - bm);
                m = bm;
                lsum *= alpha;
#pragma unroll
                for (int c = 0; c < NCT; ++c)
                    acc[c] *= alpha;
            }
        }
        const float mn = m == -INFINITY ? 0.0f : m;
        float pv[8], ps = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            pv[e] = fast_exp2(fmaf(s[e >> 2][e & 3], scale, -mn));
            ps += pv[e];
        }
        lsum += ps;
        const u32x4 pw = __builtin_bit_cast(u32x4, pack_half8(pv));
        const half8 ph = __builtin_bit_cast(half8, qg < 2 ? pw : u32x4{pw.z, pw.w, pw.x, pw.y});
#pragma unroll
        for (int c = 0; c < NCT; ++c) {
            acc[c] = mfma16(vf[c % PF], ph, acc[c]);
            if (c + PF < NCT)
                vf[c % PF] = vfrag(c + PF);
        }
    }

    __device__ __forceinline__ void finish(const AttnParams& p, const Tile& t, int, int wave, int lane)
    {
        const int col = lane & 15, qg = lane >> 4, R = t.r0 + kRows * wave + col;
        float l = lsum + __shfl_xor(lsum, 16);
        l += __shfl_xor(l, 32);
        if (R >= t.rows)
            return;
        const float mul = l > 0.0f ? 1.0f / l : 0.0f;
        float* dst = p.out + (((size_t)t.b * p.C + R / p.G) * p.H_q + (size_t)t.h * p.G + R % p.G) * D;
#pragma unroll
        for (int c = 0; c < NCT; ++c)
            *(floatx4*)(dst + 16 * c + 4 * qg) = acc[c] * mul;
    }
};

// Workgroup w runs on XCD w mod 8: the contiguous range of work items an XCD
// takes shares a unit's blocks in its L2.
__device__ __forceinline__ int xcd_item()
{
    const int W = gridDim.x;
    return (W & 7) == 0 ? (blockIdx.x & 7) * (W >> 3) + (blockIdx.x >> 3) : blockIdx.x;
}

// W: a wave's state and rows; W::kRows waves<D>() query rows per tile.
template <int D, typename W>
__global__ __launch_bounds__(64 * waves<D>(), 2) void attn_kernel(AttnParams p)
{
    constexpr int NW = waves<D>();
    constexpr int BI = image_bytes<D>(), NST = stages<D>();
    constexpr int CW = BI / 1024 / NW;  // 1 KiB copies of an image per wave
    static_assert(CW * 1024 * NW == BI && CW <= D / 16, "whole copies, one beside a K fragment");
    extern __shared__ __attribute__((aligned(16))) uint8_t plds[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the longest (newest) tiles of a unit start first
    const int L = xcd_item(), uloc = __builtin_amdgcn_readfirstlane(L / p.pf_tiles);
    const Tile t = make_tile(p, p.pf_u0 + uloc, p.pf_tiles - 1 - (L - uloc * p.pf_tiles), W::kRows * NW);
    W w;
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

// ---------------------------------------------------------------------------
// 3. The fused path: packed blocks through an LDS ring, reconstructed there
// one block ahead of the one being multiplied.  Eight waves: waves 0 .. 3 (one
// per SIMD) multiply, 32 query rows each, waves 4 .. 7 copy and reconstruct, so
// that each SIMD always has vector work beside its matrix products and the
// reconstruction needs none of the accumulators' registers (done by the
// multiplying waves themselves it spilled 80 to 116 registers at D = 256).
// Work item (unit, key range, query tile of 128 rows); key range `split` takes
// blocks [nvis split / S, nvis (split + 1) / S) of its tile.
constexpr int kFusedRows = 128, kFusedThreads = 512;

// raw blocks in flight or being reconstructed
template <int D, bool W8, bool ROT>
__host__ __device__ constexpr int raw_slots()
{
    return D == 256 && (W8 || ROT) ? 2 : 3;
}

// LDS bytes of one packed block: codes, scales and offsets of K, then of V
// (each a multiple of 16 bytes)
__host__ __device__ __forceinline__ int raw_bytes(const SectionBytes& n)
{
    return n.kc + 2 * n.km + n.vc + 2 * n.vm;
}

template <int D, int KG, bool W8, bool ROT>
struct FusedLds {  // two images, query fragments, rotation scratch, raw ring
    static constexpr int kQuery = 2 * image_bytes<D>();
    static constexpr int kScratch = kQuery + 4 * query_lds_fragments<D, KG>() * 1024;
    static constexpr int kRaw = kScratch + (ROT ? scratch_bytes<D>() : 0);
};

template <int D, int KG, bool W8, bool ROT>
__global__ __launch_bounds__(kFusedThreads, 2) void fused_kernel(AttnParams p)
{
    using LD = FusedLds<D, KG, W8, ROT>;
    constexpr int BI = image_bytes<D>(), NR = raw_slots<D, W8, ROT>();
    extern __shared__ __attribute__((aligned(16))) uint8_t plds[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int L = xcd_item(), S = p.S_tot;
    const int us = __builtin_amdgcn_readfirstlane(L / p.pf_tiles), uloc = __builtin_amdgcn_readfirstlane(us / S);
    const int split = us - uloc * S;
    const Tile t = make_tile(p, p.pf_u0 + uloc, p.pf_tiles - 1 - (L - us * p.pf_tiles), kFusedRows);
    const int it0 = __builtin_amdgcn_readfirstlane((int)((long long)t.nvis * split / S));
    const int it1 = __builtin_amdgcn_readfirstlane((int)((long long)t.nvis * (split + 1) / S));
    const auto tail_block = [&](int it) { return it < t.nsb ? it - (p.sink >> 5) : it - t.nsb; };
    const auto code_at = [&](int it) { return code_block<D>(p, it < t.nsb, tail_block(it)); };
    // Barriers, the same number for every wave: the first packed block has
    // landed; the first image is built; then one per block.
    if (wave < 4) {
        auto sync = [&]() {
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        };
        Wave<D, KG, 1, ROT> w;
        w.init(p, t, plds + LD::kQuery, wave, lane);
        sync();
        sync();
        for (int it = it0; it < it1; ++it) {
            const uint8_t* img = plds + ((it - it0) & 1) * BI;
            w.scores(img, code_at(it), lane, [](int) {});
            w.update(img, tail_block(it), lane);
            sync();
        }
        w.finish(p, t, split, wave, lane);
        return;
    }

    // ---- waves 4 .. 7: packed blocks and images
    const int bw = wave - 4;
    const SectionBytes n = section_bytes<D, W8>(p);
    const int rs = raw_bytes(n), ncb = (p.nq + 31) >> 5;  // ncb: blocks of coded tokens
    const Sections g = cache_sections(p, n, (size_t)t.unit * (p.T >> 5));
    const uint32_t lbase = (uint32_t)(uintptr_t)plds + LD::kRaw;
    // wave 0 copies the K codes, 1 the K scales and offsets, 2 and 3 those of
    // V, 1 KiB at a time
    const bool val = bw >= 2, codes = (bw & 1) == 0;
    const int clen = val ? n.vc : n.kc, mlen = val ? n.vm : n.km, at0 = (val ? n.kc + 2 * n.km : 0) + (codes ? 0 : clen);
    const uint8_t* src0 = codes ? (val ? g.vc : g.kc) : (val ? g.vs : g.ks);
    const uint8_t* src1 = codes ? nullptr : (val ? g.vz : g.kz);
    const int len = codes ? clen : mlen;
    const int cw = ncb > 0 ? ((len + 1023) >> 10) * (src1 ? 2 : 1) : 0;  // this wave's copies of a block
    // copies of block `it` (clamped to the coded blocks; a block of fp16 rows is
    // read from the cache when its image is built)
    auto copy_raw = [&](int it, int slot) __attribute__((always_inline)) {
        if (ncb == 0)
            return;
        const int blk = min(max(it - t.nsb, 0), ncb - 1);
        for (int o = 0; o < len; o += 1024)
            if (o + 16 * lane < len) {
                const size_t off = (size_t)blk * len + o;
                copy16((uint64_t)(src0 + off), 16 * lane, lbase + (uint32_t)(slot * rs + at0 + o));
                if (src1)
                    copy16((uint64_t)(src1 + off), 16 * lane, lbase + (uint32_t)(slot * rs + at0 + mlen + o));
            }
    };
    auto build = [&](int it, int slot, int im) __attribute__((always_inline)) {
        const int blk = tail_block(it);
        const bool sinkblk = it < t.nsb;
        uint8_t* img = plds + im * BI;
        float* scratch = (float*)(plds + LD::kScratch);
        const int tid = threadIdx.x - 256;
        if (!sinkblk && blk < ncb) {
            const uint8_t* r = plds + LD::kRaw + slot * rs;
            Sections s;
            s.kc = r;
            s.ks = r + n.kc;
            s.kz = s.ks + n.km;
            s.vc = s.kz + n.km;
            s.vs = s.vc + n.vc;
            s.vz = s.vs + n.vm;
            coded_image<D, W8, (KG > 0), ROT>(p, s, min(32, p.nq - 32 * blk), img, scratch, tid);
        } else {
            rows_image<D, ROT>(p, t.unit, sinkblk ? it : -1, blk, img, scratch, tid);
        }
    };
    // this wave's LDS writes are done, its copies but the newest `after` have
    // landed, and all waves are past the same point
    auto sync = [&](int after) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        ring_sync(after);
    };
    uint32_t m0_saved;
    asm volatile("s_mov_b32 %0, m0" : "=s"(m0_saved));
    if (it0 < it1)
        for (int j = 0; j < NR; ++j)
            copy_raw(it0 + j, j);
    sync(cw * (NR - 1));
    if (it0 < it1)
        build(it0, 0, 0);
    sync(cw * (NR - 2));
    int slot = 0;  // raw slot of block `it`
    for (int it = it0; it < it1; ++it) {
        copy_raw(it + NR, slot);  // block it's image is built: its slot is free
        slot = slot + 1 == NR ? 0 : slot + 1;
        if (it + 1 < it1)
            build(it + 1, slot, (it + 1 - it0) & 1);
        sync(cw * (NR - 2));
    }
    asm volatile("s_mov_b32 m0, %0" ::"s"(m0_saved));
    __builtin_amdgcn_s_waitcnt(0);  // the trailing copies have landed before the LDS is given back
}

// O = sum_s 2^(m_s - M) o_s / sum_s 2^(m_s - M) l_s over the key ranges of a
// query row, four channels per thread.
constexpr int kMergeThreads = 256;

template <int D>
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(AttnParams p)
{
    const int rows = p.C * p.G, S = p.S_tot;
    const int R = blockIdx.x * (kMergeThreads / (D / 4)) + threadIdx.x / (D / 4), d = 4 * (threadIdx.x % (D / 4));
    if (R >= rows)
        return;
    const int uloc = blockIdx.y, unit = p.pf_u0 + uloc;
    const float* ml = p.part_ml + 2 * ((size_t)uloc * S * rows + R);
    const float* po = p.part_o + ((size_t)uloc * (S - 1) * rows + R) * D + d;
    const int i = R / p.G, g = R % p.G;
    // the first range's partial is where the output goes
    float* dst = p.out + (((size_t)(unit / p.H) * p.C + i) * p.H_q + (size_t)(unit % p.H) * p.G + g) * D + d;
    float M = -INFINITY;
    for (int s = 0; s < S; ++s)
        M = fmaxf(M, ml[2 * (size_t)s * rows]);
    auto weight = [&](float m) { return m == -INFINITY ? 0.0f : fast_exp2(m - M); };
    float w0 = weight(ml[0]), l = ml[1] * w0;
    floatx4 acc = *(const floatx4*)dst * w0;
#pragma unroll 4
    for (int s = 1; s < S; ++s) {
        const float2 v = *(const float2*)(ml + 2 * (size_t)s * rows);
        const float w = weight(v.x);
        acc += *(const floatx4*)(po + (size_t)(s - 1) * rows * D) * w;
        l += v.y * w;
    }
    *(floatx4*)dst = acc * (l > 0.0f ? 1.0f / l : 0.0f);
}

typedef void (*Kernel)(AttnParams);

template <int D, int KG, bool ROT = false>
constexpr Kernel attn_of = attn_kernel<D, Wave<D, KG, qtiles<D>(), ROT>>;

template <int D>
Kernel pick(int kg, bool rot)
{
    return rot       ? attn_of<D, 0, true>
           : kg == 1 ? attn_of<D, (D >= 256 ? 0 : 1)>
           : kg == 2 ? attn_of<D, 2>
           : kg == 4 ? attn_of<D, (D >= 128 ? 4 : 1)>
           : kg == 8 ? attn_of<D, (D >= 256 ? 8 : 1)>
                     : attn_of<D, 0>;
}

template <int D>
Kernel pick16(int kg, bool rot)
{
    static_assert(D == 256);
    return rot       ? attn_kernel<D, Wave16<0, true>>
           : kg == 2 ? attn_kernel<D, Wave16<2, false>>
           : kg == 4 ? attn_kernel<D, Wave16<4, false>>
           : kg == 8 ? attn_kernel<D, Wave16<8, false>>
                     : attn_kernel<D, Wave16<0, false>>;
}

// Key ranges per query tile on the fused path, or 0 for the workspace path.
// The choice and the count depend on the call alone, not on the workspace
// given, so that a smaller workspace changes no output bit.  The estimates are
// of the whole call, from times per 32-token block measured at contexts of
// 1000 to 8192 tokens and chunks of 32 to 2048: building an image (chip-wide),
// a block's products for one round of workgroups (256 rows), and a block of
// the fused path (128 rows; reconstruction is its limit, and a rotating
// format's costs two to three times as much).  Measured at B = 1, C = 32 of
// 8192 tokens: 30 to 70 us fused against 220 to 470; at B = 8, C = 200 of 3000
// and D = 128: 250 against 152.
// At D = 64 the LDS holds two workgroups per CU: together they take 1.4 times
// as long per block as one alone, so more ranges than 256 workgroups need
// still pay while each has eight blocks or more (32 query heads on 4, 4-bit:
// B = 2, C = 300 of 8000 tokens 246 -> 118 us, B = 8, C = 64 of 3000 56 -> 45;
// with ranges down to four blocks B = 8, C = 40 of 700 went 22.0 -> 23.8).
template <int D>
int fused_splits(const AttnParams& p)
{
    if (D == 256 && p.rotate && p.k_bits == 8)
        return 0;  // two images, the scratch and two packed blocks exceed the LDS
    const long long units = (long long)p.B * p.H, rows = (long long)p.C * p.G, nb = p.pf_nvb;
    const double dq = D == 64 ? 0.004 : D == 128 ? 0.007 : 0.0106, a = D == 64 ? 1.0 : D == 128 ? 1.15 : 1.9;  // us
    const double f = p.rotate ? (D == 64 ? 1.7 : D == 128 ? 3.1 : 5.7) : (D == 64 ? 1.0 : D == 128 ? 1.3 : 2.2);
    const double f2 = p.rotate ? 2.3 : 1.4;  // two workgroups per CU, D = 64
    const auto rounds = [](long long wgs, int at_once) { return (double)((wgs + at_once - 1) / at_once); };
    const double image = units * nb * dq + nb * a * rounds(units * ((rows + kRows - 1) / kRows), D == 64 ? 512 : 256);
    // Key ranges: to fill the CUs, at least four blocks each, and their
    // partials (the first range's outputs wait in O itself) within the units'
    // shares of the workspace
    const long long wgs = units * ((rows + kFusedRows - 1) / kFusedRows);
    const auto ranges = [&](int at_once, int least) {
        long long S = at_once / wgs < nb / least ? at_once / wgs : nb / least;
        while (S > 1 && (S - 1) * rows * D * 4 + S * rows * 8 > nb * image_bytes<D>())
            --S;
        return S < 1 ? 1 : S;
    };
    const auto cost = [&](long long S) {
        const double block = D == 64 && wgs * S > 256 ? f2 * rounds(wgs * S, 512) : f * rounds(wgs * S, 256);
        return (S > 1 ? 10.0 : 0.0) + (double)((nb + S - 1) / S) * block;
    };
    long long S = ranges(256, 4);
    if (D == 64) {
        const long long two = ranges(512, 8);
        S = cost(two) < cost(S) ? two : S;
    }
    return cost(S) < image ? (int)S : 0;
}

// Whether the workspace path at D = 256 takes tiles of 128 query rows (Wave16)
// instead of 256.  A block takes the smaller tile 0.7 times as long (measured with
// both filling the CUs once), so it wins where tiles of 256 rows do not cover the
// CUs, or finish unevenly.  estimate: blocks the last CU computes; tiles start
// unit by unit, a unit's longest first, so that the last unit's longest may start
// when the first short tiles end.  Measured, 256 / 128 rows (groups of 64, 8 heads
// of two query heads): 2048 tokens at B = 1 137 / 100 us, B = 2 145 / 121, B = 3
// 188 / 203; 2048 of 8192 at B = 1 450 / 321, B = 3 937 / 930; hi + lo keys, 2048
// tokens at B = 1 148 / 103, B = 2 158 / 130; rotated, B = 1 145 / 104.
template <int D>
bool small_tiles(const AttnParams& p)
{
    static_assert(D == 256);
    const long long units = (long long)p.B * p.H, rows = (long long)p.C * p.G;
    const double nb = p.pf_nvb;
    const auto estimate = [&](int per) {
        const double n = (double)(units * ((rows + per - 1) / per));
        if (n <= 256)
            return nb;
        const double tok = (double)per / p.G, shortest = nb - (p.C > tok ? p.C - tok : 0.0) / 32;
        const double even = n * (nb + shortest) / 2 / 256, rounds = (double)(((long long)n + 255) / 256) * nb;
        const double uneven = shortest + (even > nb ? even : nb);
        return uneven < rounds ? uneven : rounds;
    };
    return 0.7 * estimate(kRows / 2) < estimate(kRows);
}

template <int D, int KG, bool W8, bool ROT>
void launch_fused(const AttnParams& p, int groups, hipStream_t stream)
{
    const size_t lds = FusedLds<D, KG, W8, ROT>::kRaw + (size_t)raw_slots<D, W8, ROT>() * raw_bytes(section_bytes<D, W8>(p));
    launch_kernel(fused_kernel<D, KG, W8, ROT>, dim3(groups), dim3(kFusedThreads), lds, stream, p);
}

template <int D, bool W8>
void launch_fused(const AttnParams& p, int kg, int groups, hipStream_t stream)
{
    if (p.rotate) {
        if constexpr (!(D == 256 && W8))
            launch_fused<D, 0, W8, true>(p, groups, stream);
    } else if (kg == 1 && D < 256) {
        launch_fused<D, D < 256 ? 1 : 0, W8, false>(p, groups, stream);
    } else if (kg == 2) {
        launch_fused<D, 2, W8, false>(p, groups, stream);
    } else if (kg == 4) {
        launch_fused<D, D >= 128 ? 4 : 2, W8, false>(p, groups, stream);
    } else if (kg == 8) {
        launch_fused<D, D >= 256 ? 8 : 2, W8, false>(p, groups, stream);
    } else {
        launch_fused<D, 0, W8, false>(p, groups, stream);
    }
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
    const int rows = p0.C * p0.G;
    const bool w8 = p0.k_bits == 8;  // 8-bit codes come as K and V both 8-bit
    // per-token key groups of 32 KG channels (a power of two from 32 to D)
    const int kg = p0.k_axis == KVQ_PER_TOKEN ? p0.k_group / 32 : 0;
    if (kg != 0 && kg != 1 && kg != 2 && !(kg == 4 && D >= 128) && !(kg == 8 && D >= 256))
        return hipErrorInvalidValue;
    const int splits = fused_splits<D>(p0);
    if (splits > 0) {
        constexpr int MR = kMergeThreads / (D / 4);  // rows per merge workgroup
        for (int u0 = 0; u0 < units; u0 += group) {
            AttnParams p = p0;
            p.pf_u0 = u0;
            p.pf_tiles = (rows + kFusedRows - 1) / kFusedRows;
            p.S_tot = splits;
            const int nu = units - u0 < group ? units - u0 : group;
            p.part_o = (float*)p.pf_ws;
            p.part_ml = p.part_o + (size_t)nu * (splits - 1) * rows * D;
            const int groups = p.pf_tiles * splits * nu;
            if (w8)
                launch_fused<D, true>(p, kg, groups, stream);
            else
                launch_fused<D, false>(p, kg, groups, stream);
            if (splits > 1)
                launch_kernel(merge_kernel<D>, dim3((rows + MR - 1) / MR, nu), dim3(kMergeThreads), 0, stream, p);
        }
        return hipGetLastError();
    }
    void (*deq)(AttnParams) = w8 ? (rot ? dequant_kernel<D, true, true> : dequant_kernel<D, true, false>)
                                 : (rot ? dequant_kernel<D, false, true> : dequant_kernel<D, false, false>);
    Kernel att = pick<D>(kg, rot);
    int per = kRows;
    if constexpr (D == 256) {
        if (small_tiles<D>(p0)) {
            att = pick16<D>(kg, rot);
            per = kRows / 2;
        }
    }
    const int tiles = (rows + per - 1) / per;
    for (int u0 = 0; u0 < units; u0 += group) {
        AttnParams p = p0;
        p.pf_u0 = u0;
        p.pf_tiles = tiles;
        p.S_tot = 1;
        const int nu = units - u0 < group ? units - u0 : group;
        launch_kernel(deq, dim3(p.pf_nvb, nu), dim3(kDqThreads), rot ? scratch_bytes<D>() : 0, stream, p);
        launch_kernel(att, dim3(tiles * nu), dim3(64 * waves<D>()), attn_lds_bytes<D>(), stream, p);
    }
    return hipGetLastError();
}

}  // namespace pre

// Built once per head size (KVQ_PREFILL_D): the kernels of one size take as
// long to compile as the rest of the library.
hipError_t launch_prefill_64(const AttnParams& p, size_t ws_bytes, hipStream_t stream);
hipError_t launch_prefill_128(const AttnParams& p, size_t ws_bytes, hipStream_t stream);
hipError_t launch_prefill_256(const AttnParams& p, size_t ws_bytes, hipStream_t stream);
int prefill_ranges_64(const AttnParams& p);
int prefill_ranges_128(const AttnParams& p);
int prefill_ranges_256(const AttnParams& p);
int prefill_tile_rows_256(const AttnParams& p);

#if KVQ_PREFILL_D == 64
hipError_t launch_prefill_64(const AttnParams& p, size_t ws_bytes, hipStream_t stream)
{
    return pre::launch<64>(p, ws_bytes, stream);
}

int prefill_ranges_64(const AttnParams& p)
{
    return pre::fused_splits<64>(p);
}

int prefill_ranges(const AttnParams& p, int D)
{
    return D == 64 ? prefill_ranges_64(p) : D == 128 ? prefill_ranges_128(p) : prefill_ranges_256(p);
}

int prefill_tile_rows(const AttnParams& p, int D)
{
    return D == 256 ? prefill_tile_rows_256(p) : pre::kRows;
}

size_t prefill_image_bytes(int D)
{
    return (size_t)192 * D;
}

hipError_t launch_prefill(const AttnParams& p, int D, size_t ws_bytes, hipStream_t stream)
{
    switch (D) {
    case 64:
        return launch_prefill_64(p, ws_bytes, stream);
    case 128:
        return launch_prefill_128(p, ws_bytes, stream);
    case 256:
        return launch_prefill_256(p, ws_bytes, stream);
    default:
        return hipErrorInvalidValue;
    }
}
#elif KVQ_PREFILL_D == 128
hipError_t launch_prefill_128(const AttnParams& p, size_t ws_bytes, hipStream_t stream)
{
    return pre::launch<128>(p, ws_bytes, stream);
}

int prefill_ranges_128(const AttnParams& p)
{
    return pre::fused_splits<128>(p);
}
#else
hipError_t launch_prefill_256(const AttnParams& p, size_t ws_bytes, hipStream_t stream)
{
    return pre::launch<256>(p, ws_bytes, stream);
}

int prefill_ranges_256(const AttnParams& p)
{
    return pre::fused_splits<256>(p);
}

int prefill_tile_rows_256(const AttnParams& p)
{
    return pre::small_tiles<256>(p) ? pre::kRows / 2 : pre::kRows;
}
#endif

}  // namespace kvq
