// Quantize-and-pack append into the physically packed incremental cache
// (Sec. 3.1 of the paper: new key/value states are coded with Eq. (3) or the
// symmetric control, bit-packed and appended; KIVI keeps an fp16 window).
//
// Bit-exactness: codes and metadata must equal the CPU reference bit for
// bit, so this file is compiled with -ffp-contract=off and the coder takes
// exactly the reference's IEEE binary32 steps: subtract, correctly rounded
// divide, round half to even, clamp (the rounded quotient comes from a
// reciprocal product wherever that provably gives the same code; see
// rint_quotient).  Min/max are exact.
//
// One workgroup (256 threads) codes one aligned block of 32 tokens of one
// (sequence, KV head): a thread holds eight channels of one or a few rows
// (rotated by the fixed Hadamard butterflies when the format rotates, rounded
// to fp16 when a window exists), group statistics are reduced per (token,
// group) or per channel, and every output piece (eight codes) is assembled by
// one thread, keys first, then values.  V codes are packed along tokens: a
// piece shared with tokens outside the block range keeps earlier tokens' bits
// and clears later ones, so the image is independent of call boundaries.
//
// Pieces are stored in the order the decode kernel consumes them (per
// 32-token block, a 64-lane MFMA layout; see include/kvq.h): token tau of a
// block is row 4 (tau / 8) + tau % 4 of half (tau / 4) % 2, and the lane of
// key piece P is row + 16 (P % 4); value piece (octet o, channel d) belongs
// to lane d % 16 + 16 o.

#include "coder.h"
#include "kvq_device.h"
#include "kvq_internal.h"

namespace kvq {
namespace {

constexpr int kThreads = 256;
constexpr int kBlockTok = 32;

// Index of key piece P (channels 8P..8P+7) of position tau in block `blk`
// (blk counted over the whole section: unit * NB + block).
template <int D>
__device__ __forceinline__ size_t key_piece(size_t blk, int tau, int P)
{
    const int row = 4 * (tau >> 3) + (tau & 3), half = (tau >> 2) & 1;
    return ((blk * 2 + half) * 64 + row + 16 * (P & 3)) * (D / 32) + (P >> 2);
}

// Index of value piece (octet o of the block, channel d).
template <int D>
__device__ __forceinline__ size_t value_piece(size_t blk, int o, int d)
{
    return (blk * 64 + (d & 15) + 16 * o) * (D / 16) + (d >> 4);
}

// The normalized transform of one row held by D / 8 consecutive lanes, eight
// channels each (piece `piece` of the row): half widths 1, 2, 4 inside a lane,
// 8 .. D / 2 across lanes, then one multiply by c.  Every butterfly adds or
// subtracts the same two values as the serial transform, so results are
// identical.
template <int D>
__device__ __forceinline__ void rotate8(float* r, int piece, float c)
{
#pragma unroll
    for (int hw = 1; hw < 8; hw <<= 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (e & hw)
                continue;
            const float a = r[e], b = r[e + hw];
            r[e] = a + b;
            r[e + hw] = a - b;
        }
    }
#pragma unroll
    for (int hl = 1; hl < D / 8; hl <<= 1) {
        const bool upper = (piece & hl) != 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float other = __shfl_xor(r[e], hl);
            r[e] = upper ? other - r[e] : r[e] + other;
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
        r[e] *= c;
}

// Staging of the block's rows of K (which = 0) or V (which = 1) as the coder
// sees them.  Row i is token tb + i; rows outside [q0, q1) are zero.  Thread
// j moves eight channels of one row per step (one 16-byte load); the D / 8
// threads of a row are consecutive lanes of one wave.
template <int D>
struct RowStage {
    static constexpr int kSteps = kBlockTok * (D / 8) / kThreads;
    static_assert(kSteps >= 1 && kBlockTok * (D / 8) % kThreads == 0, "uniform staging steps");
    u32x4 w[kSteps];

    __device__ static int row(int k) { return ((int)threadIdx.x + kThreads * k) / (D / 8); }
    __device__ static int chan(int k) { return 8 * (((int)threadIdx.x + kThreads * k) % (D / 8)); }

    // Issue the loads (bf16 input for tokens of this call, fp16 window slots
    // for tokens appended earlier).
    __device__ void load(const AppendParams& p, int which, int b, int h, int tb)
    {
        const uint16_t* in = which ? p.vin : p.kin;
        const uint16_t* ring = which ? p.vr : p.kr;
#pragma unroll
        for (int k = 0; k < kSteps; ++k) {
            const int t = tb + row(k), d8 = chan(k);
            w[k] = u32x4{0u, 0u, 0u, 0u};
            if (t >= p.q0 && t < p.q1)
                w[k] = t >= p.n0 ? *(const u32x4*)(in + (((size_t)b * p.n_new + (t - p.n0)) * p.H + h) * D + d8)
                                 : *(const u32x4*)(ring + (((size_t)b * p.H + h) * p.ring + t % p.ring) * D + d8);
        }
    }

    // The eight values of step k as the coder sees them: widened to fp32; for
    // tokens of this call rotated, and rounded to fp16 when a window exists.
    __device__ __forceinline__ void widen(const AppendParams& p, int tb, int k, float* v) const
    {
        const int t = tb + row(k);
        const bool fresh = !(t >= p.q0 && t < p.q1) || t >= p.n0;  // bf16 (zero rows: zero words)
        const uint32_t ww[4] = {w[k].x, w[k].y, w[k].z, w[k].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (fresh) {
                v[2 * q] = __uint_as_float(ww[q] << 16);
                v[2 * q + 1] = __uint_as_float(ww[q] & 0xFFFF0000u);
            } else {
                v[2 * q] = f16_bits_to_f32((uint16_t)ww[q]);
                v[2 * q + 1] = f16_bits_to_f32((uint16_t)(ww[q] >> 16));
            }
        }
        const bool input = t >= p.q0 && t < p.q1 && t >= p.n0;
        if (p.rotate) {
            float r[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                r[e] = v[e];
            rotate8<D>(r, chan(k) >> 3, p.rot_c);
            if (input) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    v[e] = r[e];
            }
        }
        if (p.ring && input) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v[e] = f16_bits_to_f32(f32_to_f16_bits(v[e]));
        }
    }
};

// 16-byte copy of `bytes` (a multiple of 16) from LDS to global memory.
__device__ __forceinline__ void copy_out(const uint8_t* src, uint8_t* dst, int bytes)
{
    for (int off = 16 * (int)threadIdx.x; off < bytes; off += 16 * kThreads)
        *(u32x4*)(dst + off) = *(const u32x4*)(src + off);
}

// A block shared with earlier or later calls (per-token groups: a block of
// per-channel keys is one whole group), written piece by piece: value pieces
// keep the bits of tokens appended earlier.  vcode: 32 D bytes of LDS for the
// value codes [token][D].
template <int D>
__device__ __forceinline__ void edge_block(const AppendParams& p, int unit, int tb, uint8_t* vcode)
{
    const int b = unit / p.H, h = unit % p.H;
    const int lo = max(p.q0, tb), hi = min(p.q1, tb + kBlockTok);

    // ------------------------------------------------------------ keys
    const size_t blk = (size_t)unit * (size_t)(p.T / kBlockTok) + (size_t)(tb / kBlockTok);
    RowStage<D> kst, vst;
    kst.load(p, 0, b, h, tb);
    vst.load(p, 1, b, h, tb);  // in flight while the keys are coded
    const int kb = p.k_bits;
    {
        const int lanes = p.k_group / 8, ng = D / p.k_group;
        const size_t mbase = blk * (size_t)(ng * kBlockTok);
#pragma unroll
        for (int k = 0; k < RowStage<D>::kSteps; ++k) {
            const int i = RowStage<D>::row(k), P = RowStage<D>::chan(k) / 8, t = tb + i;
            float x[8];
            kst.widen(p, tb, k, x);
            float s, z;
            piece_group_stats(x, lanes, p.k_mode, kb, &s, &z);
            round_meta(p.meta16, &s, &z);
            if (t < lo || t >= hi)
                continue;
            if (P % lanes == 0) {
                const size_t mi = mbase + (size_t)(P / lanes) * kBlockTok + i;
                store_meta(p.ks, mi, s, p.meta16);
                if (p.k_mode == KVQ_AFFINE)
                    store_meta(p.kz, mi, z, p.meta16);
            }
            const float r = __builtin_amdgcn_rcpf(s);
            uint64_t word = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                word |= (uint64_t)code_one(x[e], s, r, z, p.k_mode, kb) << (kb * e);
            store_piece(p.kc, key_piece<D>(blk, i, P), kb, word);
        }
    }

    // ---------------------------------------------------------- values
    const int vb = p.v_bits;
    const int vlanes = p.v_group / 8;
    const size_t mbase = blk * (size_t)((D / p.v_group) * kBlockTok);
#pragma unroll
    for (int k = 0; k < RowStage<D>::kSteps; ++k) {
        const int i = RowStage<D>::row(k), P = RowStage<D>::chan(k) / 8, t = tb + i;
        float x[8];
        vst.widen(p, tb, k, x);
        float s, z;
        piece_group_stats(x, vlanes, p.v_mode, vb, &s, &z);
        round_meta(p.meta16, &s, &z);
        if (t >= lo && t < hi && P % vlanes == 0) {
            const size_t mi = mbase + (size_t)(P / vlanes) * kBlockTok + i;
            store_meta(p.vs, mi, s, p.meta16);
            if (p.v_mode == KVQ_AFFINE)
                store_meta(p.vz, mi, z, p.meta16);
        }
        const float r = __builtin_amdgcn_rcpf(s);
        uint32_t c[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            c[e] = code_one(x[e], s, r, z, p.v_mode, vb);
        *(uint2*)(vcode + i * D + 8 * P) =
            make_uint2(c[0] | (c[1] << 8) | (c[2] << 16) | (c[3] << 24), c[4] | (c[5] << 8) | (c[6] << 16) | (c[7] << 24));
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < (kBlockTok / 8) * D; idx += kThreads) {
        int o = idx / D, d = idx % D;
        int tfirst = tb + 8 * o;
        if (tfirst + 8 <= lo || tfirst >= hi)
            continue;
        uint64_t word = 0;
        if (tfirst < lo) {  // keep the bits of tokens appended earlier
            int keep_n = lo - tfirst;
            word = load_piece(p.vc, value_piece<D>(blk, o, d), vb) & low_codes(vb, keep_n);
        }
        for (int e = 0; e < 8; ++e) {
            int t = tfirst + e;
            if (t < lo || t >= hi)
                continue;
            word |= (uint64_t)vcode[(t - tb) * D + d] << (vb * e);
        }
        store_piece(p.vc, value_piece<D>(blk, o, d), vb, word);
    }
}

// ---- blocks

// The eight codes of a piece.  The quotient is the product with the hardware
// reciprocal wherever that provably rounds to the same code (rint_quotient);
// the eight distances to the rounded values are folded into one test, and a
// piece with a near tie takes the exact divisions.  Codes are packed by fp32
// sums (below 2^24, exact), one conversion per 16 bits: conversions, shifts
// and the per-element branch took half of the instructions before.
template <int BITS>
__device__ __forceinline__ uint64_t piece_codes(const float* x, const float* s, const float* r, const float* z, int mode)
{
#pragma clang fp contract(off)
    const float top = (float)((1 << BITS) - 1), qmax = (float)((1 << (BITS - 1)) - 1), half = (float)(1 << (BITS - 1));
    const bool aff = mode == KVQ_AFFINE;
    float c[8], worst = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float d = aff ? x[e] - z[e] : x[e], q = d * r[e];
        c[e] = __builtin_rintf(q);
        worst = fmaxf(worst, fabsf(q - c[e]));
    }
    if (worst >= 0.5f - 0x1p-10f) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            c[e] = __builtin_rintf((aff ? x[e] - z[e] : x[e]) / s[e]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
        c[e] = aff ? __builtin_amdgcn_fmed3f(c[e], 0.0f, top) : __builtin_amdgcn_fmed3f(c[e], -qmax, qmax) + half;
    constexpr int N = 16 / BITS;  // codes per 16 bits
    uint64_t word = 0;
#pragma unroll
    for (int k = 0; k < 8 / N; ++k) {
        float v = 0.0f;
#pragma unroll
        for (int e = N - 1; e >= 0; --e)
            v = __builtin_fmaf(v, (float)(1 << BITS), c[N * k + e]);
        if constexpr (BITS == 8)
            word |= (uint64_t)(uint32_t)v << (16 * k);
        else
            word = (uint32_t)word | ((uint32_t)v << (16 * k));
    }
    return word;
}

// The value of lane l ^ 8 (a rotation by half a 16-lane row).
__device__ __forceinline__ float row_ror8(float v)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x128, 0xF, 0xF, false));
}

// One workgroup per 32-token block of one (sequence, KV head); a block this
// call does not write whole takes edge_block (in a launch of its own it cost
// 5 to 10 us a call).  Per-token groups: each thread takes the eight channels of one piece, the
// group's statistics are reduced across the group's lanes.  Per-channel keys:
// a thread's eight channels of its rows are reduced over the rows in
// registers, by shuffles and over the four waves.  Key pieces go to LDS as
// they are; value words (eight channels of one token) are transposed there,
// one thread per (octet, eight channels).  Each section holds a block's bytes
// as one range, written with contiguous 16-byte stores.
// Vector work bounds it.  A KIVI chunk of 2048 tokens (B = 32, 8 heads of 128,
// 348 MB) took 164 us with rows staged in LDS, one thread per channel for the
// statistics, codes as bytes and 64-bit shifts; 115 now, window rows included.
template <int D, bool PERCH, int KB, int VB>
__global__ __launch_bounds__(kThreads) void append_block_kernel(AppendParams p)
{
    constexpr int PPT = D / 8, kOut = 4 * D * (KB > VB ? KB : VB);
    // a section's pieces, and the value codes by token (edge_block: all of it)
    constexpr int kPool = kOut + 4 * D * VB > 32 * D ? kOut + 4 * D * VB : 32 * D;
    __shared__ __attribute__((aligned(16))) uint8_t pool[kPool];
    uint8_t* ob = pool;
    uint32_t* vw = (uint32_t*)(pool + kOut);
    __shared__ __attribute__((aligned(16))) float mb[2][kBlockTok * 8];  // its scales, offsets (<= 1 KB each)
    __shared__ __attribute__((aligned(16))) float red[PERCH ? 2 : 1][PERCH ? 4 : 1][PERCH ? D : 4];
    __shared__ __attribute__((aligned(16))) float cs[PERCH ? 3 : 1][PERCH ? D : 4];  // channel scales, reciprocals, offsets
    constexpr int kSteps = RowStage<D>::kSteps;

    const int unit = blockIdx.y;
    const int b = unit / p.H, h = unit % p.H;
    const int tb = (p.q0 / kBlockTok + (int)blockIdx.x) * kBlockTok;
    if constexpr (!PERCH) {
        if (tb < p.q0 || tb + kBlockTok > p.q1) {
            edge_block<D>(p, unit, tb, pool);
            return;
        }
    }
    const int msz = p.meta16 ? 2 : 4;
    const size_t blk = (size_t)unit * (size_t)(p.T / kBlockTok) + (size_t)(tb / kBlockTok);
    RowStage<D> kst, vst;
    kst.load(p, 0, b, h, tb);
    vst.load(p, 1, b, h, tb);  // in flight while the keys are coded

    // ------------------------------------------------------------ keys
    int kmeta;  // metadata elements per block
    if constexpr (!PERCH) {
        const int lanes = p.k_group / 8;
        kmeta = D / p.k_group * kBlockTok;
#pragma unroll
        for (int k = 0; k < kSteps; ++k) {
            const int i = RowStage<D>::row(k), P = RowStage<D>::chan(k) / 8;
            float x[8], s, z;
            kst.widen(p, tb, k, x);
            piece_group_stats(x, lanes, p.k_mode, KB, &s, &z);
            round_meta(p.meta16, &s, &z);
            if (P % lanes == 0) {
                store_meta(mb[0], (P / lanes) * kBlockTok + i, s, p.meta16);
                if (p.k_mode == KVQ_AFFINE)
                    store_meta(mb[1], (P / lanes) * kBlockTok + i, z, p.meta16);
            }
            const float r = __builtin_amdgcn_rcpf(s);
            const float s8[8] = {s, s, s, s, s, s, s, s}, r8[8] = {r, r, r, r, r, r, r, r}, z8[8] = {z, z, z, z, z, z, z, z};
            store_piece(ob, key_piece<D>(0, i, P), KB, piece_codes<KB>(x, s8, r8, z8, p.k_mode));
        }
    } else {
        kmeta = D;
        float x[kSteps][8], mn[8], mx[8];
#pragma unroll
        for (int k = 0; k < kSteps; ++k)
            kst.widen(p, tb, k, x[k]);
        const bool aff = p.k_mode == KVQ_AFFINE;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            mn[e] = x[0][e];
            mx[e] = aff ? x[0][e] : fabsf(x[0][e]);
#pragma unroll
            for (int k = 1; k < kSteps; ++k) {
                mn[e] = fminf(mn[e], x[k][e]);
                mx[e] = fmaxf(mx[e], aff ? x[k][e] : fabsf(x[k][e]));
            }
            // (shuffles are LDS operations, which the vector-bound large chunks
            // do not notice: row swaps instead took 125 against 115 us)
            if constexpr (PPT <= 8) {
                mn[e] = fminf(mn[e], row_ror8(mn[e]));
                mx[e] = fmaxf(mx[e], row_ror8(mx[e]));
            }
#pragma unroll
            for (int off = PPT < 16 ? 16 : PPT; off < 64; off <<= 1) {
                mn[e] = fminf(mn[e], __shfl_xor(mn[e], off));
                mx[e] = fmaxf(mx[e], __shfl_xor(mx[e], off));
            }
        }
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c8 = RowStage<D>::chan(0);
        if (lane < PPT) {
            *(float4*)&red[0][wave][c8] = make_float4(mn[0], mn[1], mn[2], mn[3]);
            *(float4*)&red[0][wave][c8 + 4] = make_float4(mn[4], mn[5], mn[6], mn[7]);
            *(float4*)&red[1][wave][c8] = make_float4(mx[0], mx[1], mx[2], mx[3]);
            *(float4*)&red[1][wave][c8 + 4] = make_float4(mx[4], mx[5], mx[6], mx[7]);
        }
        __syncthreads();
        for (int d = threadIdx.x; d < D; d += kThreads) {
            const float lo[1] = {fminf(fminf(red[0][0][d], red[0][1][d]), fminf(red[0][2][d], red[0][3][d]))};
            const float hi = fmaxf(fmaxf(red[1][0][d], red[1][1][d]), fmaxf(red[1][2][d], red[1][3][d]));
            // group_stats of the group's extremes: the same minimum, maximum
            // and magnitude, so the same scale and offset
            const float ends[2] = {aff ? lo[0] : hi, hi};
            float s, z;
            group_stats(ends, 1, 2, p.k_mode, KB, &s, &z);
            round_meta(p.meta16, &s, &z);
            cs[0][d] = s;
            cs[1][d] = __builtin_amdgcn_rcpf(s);
            cs[2][d] = z;
            store_meta(mb[0], d, s, p.meta16);
            if (aff)
                store_meta(mb[1], d, z, p.meta16);
        }
        __syncthreads();
        float s8[8], r8[8], z8[8];
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
            *(float4*)(s8 + e) = *(const float4*)&cs[0][c8 + e];
            *(float4*)(r8 + e) = *(const float4*)&cs[1][c8 + e];
            *(float4*)(z8 + e) = *(const float4*)&cs[2][c8 + e];
        }
#pragma unroll
        for (int k = 0; k < kSteps; ++k)
            store_piece(ob, key_piece<D>(0, RowStage<D>::row(k), c8 / 8), KB, piece_codes<KB>(x[k], s8, r8, z8, p.k_mode));
    }
    __syncthreads();
    copy_out(ob, (uint8_t*)p.kc + blk * (size_t)(4 * D * KB), 4 * D * KB);
    copy_out((const uint8_t*)mb[0], (uint8_t*)p.ks + blk * (size_t)(kmeta * msz), kmeta * msz);
    if (p.k_mode == KVQ_AFFINE)
        copy_out((const uint8_t*)mb[1], (uint8_t*)p.kz + blk * (size_t)(kmeta * msz), kmeta * msz);
    __syncthreads();  // the key copies have read ob and mb

    // ---------------------------------------------------------- values
    const int vlanes = p.v_group / 8, vmeta = (D / p.v_group) * kBlockTok;
#pragma unroll
    for (int k = 0; k < kSteps; ++k) {
        const int i = RowStage<D>::row(k), P = RowStage<D>::chan(k) / 8;
        float x[8], s, z;
        vst.widen(p, tb, k, x);
        piece_group_stats(x, vlanes, p.v_mode, VB, &s, &z);
        round_meta(p.meta16, &s, &z);
        if (P % vlanes == 0) {
            store_meta(mb[0], (P / vlanes) * kBlockTok + i, s, p.meta16);
            if (p.v_mode == KVQ_AFFINE)
                store_meta(mb[1], (P / vlanes) * kBlockTok + i, z, p.meta16);
        }
        const float r = __builtin_amdgcn_rcpf(s);
        const float s8[8] = {s, s, s, s, s, s, s, s}, r8[8] = {r, r, r, r, r, r, r, r}, z8[8] = {z, z, z, z, z, z, z, z};
        store_piece(vw, i * PPT + P, VB, piece_codes<VB>(x, s8, r8, z8, p.v_mode));
    }
    __syncthreads();
    // (octet o, channels 8 P .. 8 P + 7): the eight tokens' words transposed
    for (int idx = threadIdx.x; idx < 4 * PPT; idx += kThreads) {
        const int o = idx / PPT, P = idx % PPT;
        uint64_t w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            w[j] = load_piece(vw, (8 * o + j) * PPT + P, VB);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if constexpr (VB == 8) {
                uint64_t v = 0;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    v |= (w[j] >> (8 * e) & 0xFFu) << (8 * j);
                store_piece(ob, value_piece<D>(0, o, 8 * P + e), VB, v);
            } else {
                uint32_t v = 0;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    v |= ((uint32_t)w[j] >> (VB * e) & ((1u << VB) - 1u)) << (VB * j);
                store_piece(ob, value_piece<D>(0, o, 8 * P + e), VB, v);
            }
        }
    }
    __syncthreads();
    copy_out(ob, (uint8_t*)p.vc + blk * (size_t)(4 * D * VB), 4 * D * VB);
    copy_out((const uint8_t*)mb[0], (uint8_t*)p.vs + blk * (size_t)(vmeta * msz), vmeta * msz);
    if (p.v_mode == KVQ_AFFINE)
        copy_out((const uint8_t*)mb[1], (uint8_t*)p.vz + blk * (size_t)(vmeta * msz), vmeta * msz);
}

// One decoded token per (sequence, KV head) without a window: a workgroup of
// D threads, thread d owning channel d of the token's K and V.  Every load
// (the token's K and V, and the value piece it shares with earlier tokens)
// is issued first; the rotation runs as the same butterflies as rotate8;
// group statistics are all-reduced across the group's threads (min, max and
// max-magnitude are exact in any order, so they equal the block kernel's),
// then each thread codes its channel, key pieces are OR-reduced over eight
// lanes and each value piece is merged with the bits of earlier tokens.
template <int D>
__device__ __forceinline__ float group_reduce(float v, int g, bool is_max, float* red, int slot)
{
    const int lanes = g < 64 ? g : 64;
    for (int off = 1; off < lanes; off <<= 1) {
        const float o = __shfl_xor(v, off);
        v = is_max ? fmaxf(v, o) : fminf(v, o);
    }
    if (g > 64) {
        // one value per wave, combined over the g / 64 waves of the group
        const int wave = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0)
            red[slot * 4 + wave] = v;
        __syncthreads();
        const int w0 = (wave / (g / 64)) * (g / 64);
        v = red[slot * 4 + w0];
        for (int w = 1; w < g / 64; ++w)
            v = is_max ? fmaxf(v, red[slot * 4 + w0 + w]) : fminf(v, red[slot * 4 + w0 + w]);
    }
    return v;
}

template <int D>
__global__ __launch_bounds__(D) void append_token_kernel(AppendParams p)
{
    __shared__ float xs[2][D];
    __shared__ float red[8 * 4];
    const int unit = blockIdx.x, b = unit / p.H, h = unit % p.H, d = threadIdx.x;
    const int t = p.n0, tau = t & 31, j = t & 7;
    const size_t blk = (size_t)unit * (p.T / kBlockTok) + (size_t)(t / kBlockTok);
    const size_t vpi = value_piece<D>(blk, tau >> 3, d);
    const size_t in = ((size_t)b * p.H + h) * D + d;  // n_new == 1
    float x[2] = {bf16_to_f32(p.kin[in]), bf16_to_f32(p.vin[in])};
    const uint64_t old = load_piece(p.vc, vpi, p.v_bits);
    if (p.rotate) {
        xs[0][d] = x[0];
        xs[1][d] = x[1];
        __syncthreads();
        for (int hw = 1; hw < D; hw <<= 1) {
            float nv[2];
#pragma unroll
            for (int w = 0; w < 2; ++w)
                nv[w] = (d & hw) ? xs[w][d - hw] - xs[w][d] : xs[w][d] + xs[w][d + hw];
            __syncthreads();
            xs[0][d] = nv[0];
            xs[1][d] = nv[1];
            __syncthreads();
        }
        x[0] = xs[0][d] * p.rot_c;
        x[1] = xs[1][d] * p.rot_c;
    }
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const int mode = w ? p.v_mode : p.k_mode, bits = w ? p.v_bits : p.k_bits;
        const int g = w ? p.v_group : p.k_group, gi = d / g, ng = D / g;
        float s, z;
        if (mode == KVQ_AFFINE) {
            const float mn = group_reduce<D>(x[w], g, false, red, 2 * w);
            const float mx = group_reduce<D>(x[w], g, true, red, 2 * w + 1);
            const float top = (float)((1 << bits) - 1);
            s = (mx - mn) / top;
            if (!(s >= 1e-8f))
                s = 1e-8f;
            z = mn + 0.0f;  // canonical +0 for a signed-zero minimum
        } else {
            const float ma = group_reduce<D>(fabsf(x[w]), g, true, red, 2 * w);
            const float qmax = (float)((1 << (bits - 1)) - 1);
            s = ma / qmax;
            if (!(s >= 1e-8f))
                s = 1e-8f;
            z = 0.0f;
        }
        round_meta(p.meta16, &s, &z);
        const uint32_t c = code_one(x[w], s, __builtin_amdgcn_rcpf(s), z, mode, bits);
        if (d % g == 0) {
            const size_t mi = (blk * ng + gi) * kBlockTok + tau;
            store_meta(w ? p.vs : p.ks, mi, s, p.meta16);
            if (mode == KVQ_AFFINE)
                store_meta(w ? p.vz : p.kz, mi, z, p.meta16);
        }
        if (w == 0) {
            // key piece d / 8: codes of channels 8P .. 8P + 7 at bits k_bits e,
            // OR-reduced as two 32-bit halves
            const uint64_t mine = (uint64_t)c << (bits * (d & 7));
            uint32_t lo32 = (uint32_t)mine, hi32 = (uint32_t)(mine >> 32);
#pragma unroll
            for (int off = 1; off < 8; off <<= 1) {
                lo32 |= __shfl_xor(lo32, off);
                hi32 |= __shfl_xor(hi32, off);
            }
            if ((d & 7) == 0)
                store_piece(p.kc, key_piece<D>(blk, tau, d >> 3), bits, ((uint64_t)hi32 << 32) | lo32);
        } else {
            const uint64_t keep = low_codes(bits, j);
            store_piece(p.vc, vpi, bits, (old & keep) | ((uint64_t)c << (bits * j)));
        }
    }
}

// fp16 window: slot t mod (R + F) <- fp16 of token t (rotated first when
// the format rotates), for t in [ring_lo, n0 + n_new).  Runs after the coder
// of the same call, which may still read the slots being replaced.  The
// sink rows are written by the same kernel with ring = sink (slot t).
// A thread moves eight channels of one row of K and of V with 16-byte loads and
// stores, a workgroup kRingRows<D> rows (one row per workgroup with 2-byte
// loads: 128 rows of 256 units 33 us, now 8).
template <int D>
constexpr int kRingRows = kThreads / (D / 8);

template <int D>
__global__ __launch_bounds__(kThreads) void append_ring_kernel(AppendParams p, int hi)
{
    const int unit = blockIdx.y;
    const int b = unit / p.H, h = unit % p.H;
    const int c8 = 8 * ((int)threadIdx.x % (D / 8));
    const int t = p.ring_lo + kRingRows<D> * (int)blockIdx.x + (int)threadIdx.x / (D / 8);
    const size_t at = (((size_t)b * p.n_new + (t - p.n0)) * p.H + h) * D + c8;
    u32x4 w[2] = {u32x4{0u, 0u, 0u, 0u}, u32x4{0u, 0u, 0u, 0u}};
    if (t < hi) {
        w[0] = *(const u32x4*)(p.kin + at);
        w[1] = *(const u32x4*)(p.vin + at);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint32_t ww[4] = {w[q].x, w[q].y, w[q].z, w[q].w};
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = __uint_as_float((e & 1) ? ww[e >> 1] & 0xFFFF0000u : ww[e >> 1] << 16);
        if (p.rotate)  // (every lane of a row takes part)
            rotate8<D>(v, c8 >> 3, p.rot_c);
        if (t < hi) {
            uint32_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                o[e] = f32_to_f16_bits(v[2 * e]) | ((uint32_t)f32_to_f16_bits(v[2 * e + 1]) << 16);
            *(u32x4*)((q ? p.vr : p.kr) + ((size_t)unit * p.ring + t % p.ring) * D + c8) = u32x4{o[0], o[1], o[2], o[3]};
        }
    }
}

template <int D, bool PERCH>
void launch_blocks(const AppendParams& p, int blocks, int units, hipStream_t stream)
{
    const dim3 g(blocks, units), t(kThreads);
    if (p.k_bits == 8)  // 8-bit codes come as K and V both 8-bit
        launch_kernel((append_block_kernel<D, PERCH, 8, 8>), g, t, 0, stream, p);
    else if (p.k_bits == 4 && p.v_bits == 4)
        launch_kernel((append_block_kernel<D, PERCH, 4, 4>), g, t, 0, stream, p);
    else if (p.k_bits == 4)
        launch_kernel((append_block_kernel<D, PERCH, 4, 2>), g, t, 0, stream, p);
    else if (p.v_bits == 4)
        launch_kernel((append_block_kernel<D, PERCH, 2, 4>), g, t, 0, stream, p);
    else
        launch_kernel((append_block_kernel<D, PERCH, 2, 2>), g, t, 0, stream, p);
}

template <int D>
hipError_t launch_append_d(const AppendParams& p, hipStream_t stream)
{
    const int units = p.B * p.H;
    if (p.n_new == 1 && p.ring == 0 && p.k_axis == KVQ_PER_TOKEN) {
        launch_kernel(append_token_kernel<D>, dim3(units), dim3(D), 0, stream, p);
        return hipGetLastError();
    }
    if (p.q1 > p.q0) {
        const int blocks = (p.q1 + kBlockTok - 1) / kBlockTok - p.q0 / kBlockTok;
        if (p.k_axis == KVQ_PER_CHANNEL)
            launch_blocks<D, true>(p, blocks, units, stream);
        else
            launch_blocks<D, false>(p, blocks, units, stream);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    int n1 = p.n0 + p.n_new;
    if (p.ring && n1 > p.ring_lo) {
        launch_kernel(append_ring_kernel<D>, dim3((n1 - p.ring_lo + kRingRows<D> - 1) / kRingRows<D>, units), dim3(kThreads), 0,
                      stream, p, n1);
        return hipGetLastError();
    }
    return hipSuccess;
}

template <int D>
hipError_t launch_rows_d(const AppendParams& p, int hi, hipStream_t stream)
{
    if (hi > p.ring_lo)
        launch_kernel(append_ring_kernel<D>, dim3((hi - p.ring_lo + kRingRows<D> - 1) / kRingRows<D>, p.B * p.H), dim3(kThreads), 0,
                      stream, p, hi);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_append_rows(const AppendParams& p, int D, int hi, hipStream_t stream)
{
    switch (D) {
    case 64:
        return launch_rows_d<64>(p, hi, stream);
    case 128:
        return launch_rows_d<128>(p, hi, stream);
    case 256:
        return launch_rows_d<256>(p, hi, stream);
    default:
        return hipErrorInvalidValue;
    }
}

hipError_t launch_append(const AppendParams& p, int D, hipStream_t stream)
{
    switch (D) {
    case 64:
        return launch_append_d<64>(p, stream);
    case 128:
        return launch_append_d<128>(p, stream);
    case 256:
        return launch_append_d<256>(p, stream);
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace kvq
