// FP8 (E4M3) attention kernel and its pre-passes.
#pragma once
#include "common.hpp"

namespace {

// ---------------------------------------------------------------------------------------------
// FP8 (E4M3) path: the 8-bit tensor regime of the paper's performance discussion ("C8V32": matrix
// products in 8 bit, softmax in fp32).  v_mfma_f32_32x32x64_f8f6f4 does a 32 x 32 x 64 product in
// 64 cycles, twice the bf16 rate, so a 64-key tile is 4 + 4 MFMAs per wave instead of 16 + 16 and the
// softmax arithmetic, unchanged, weighs twice as much.  Measured pairing of the operands: byte j of
// lane (row, half) of A meets byte j of lane (col, same half) of B, so any assignment of the 64
// k-indices to (half, byte) works as long as both operands use the same one:
//   Q.K^T  k-step kh (0, 1): byte j of half hh = feature 64 kh + 32 hh + j, for K rows and Q rows alike
//   P.V    byte j of half hh = key 32 (j / 16) + 8 ((j % 16) / 4) + 4 hh + j % 4 of the tile: the order in
//          which the score accumulators of a lane, packed four to a dword, already sit; V is stored
//          transposed and permuted to that order by the packing pre-pass, so one 32-byte read per
//          lane is the whole A operand and no transposing read is needed.
// exp(S - m) goes to E4M3 scaled by 2^(8 - H): the conversion instruction does not saturate (beyond
// 448 it writes NaN), so the value is capped by the clamp modifier of the exponential itself:
// q = min(exp2(s c - m - H), 1), stored as q 2^8, and l sums the same q.  H = 0 for the exact-max
// baseline (exp <= 1 by construction); the frozen-max mode takes H = 4: exact while the frozen max
// is at most 4 log2-units (2.8 nats) below the true one, capped (never NaN) beyond.
typedef __attribute__((ext_vector_type(8))) int i32x8;
typedef __attribute__((ext_vector_type(2))) short s16x2;

struct Tile8 {
    static constexpr int KBYTES = BN * 128;   // K tile: 64 rows of 128 bytes
    static constexpr int VBYTES = 128 * BN;   // V^T tile: 128 rows (features) of 64 bytes (keys, permuted)
    // 16-byte chunk c of row r is stored at chunk position c ^ key(r); chosen so that 16 consecutive
    // rows reading the same logical chunk cover all 64 banks
    __device__ static int k_off(int r, int c) { return r * 128 + ((c ^ ((r >> 1) & 7)) << 4); }
    __device__ static int v_off(int r, int c) { return r * 64 + ((c ^ ((r >> 2) & 3)) << 4); }
};

// E4M3 x E4M3; scale_a = four copies of an E8M0 exponent byte that multiplies the A operand's 32-element
// blocks by 2^(byte - 127) inside the instruction (0x7f7f7f7f = 2^0); the B operand is not scaled
__device__ __forceinline__ f32x16 mfma_f8(const i32x8& a, const i32x8& b, const f32x16& c, int scale_a = 0x7f7f7f7f) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, scale_a, 0, 0x7f7f7f7f);
}

// a wave-uniform pointer as two scalar registers (the compiler cannot always see that it is uniform)
__device__ __forceinline__ uint64_t uniform_ptr(const void* ptr) {
    const uint64_t b64 = (uint64_t)(uintptr_t)ptr;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b64);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b64 >> 32));
    return ((uint64_t)hi << 32) | (uint64_t)lo;
}

// one LDS-direct load: lane l's 16 (BYTES = 16) or 4 bytes at base + off go to LDS address lds_addr + BYTES * l.
// Scalar base plus a 32-bit lane offset: one address register per lane instead of a 64-bit pointer.
template <int BYTES>
__device__ __forceinline__ void lds_dma(uint64_t base, uint32_t off, uint32_t lds_addr) {
    uint32_t m0_save;
    if (BYTES == 16)
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
                     : "=&s"(m0_save)
                     : "s"(lds_addr), "v"(off), "s"(base)
                     : "memory");
    else
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %2, %3\n\ts_mov_b32 m0, %0"
                     : "=&s"(m0_save)
                     : "s"(lds_addr), "v"(off), "s"(base)
                     : "memory");
}

// 64 rows of 128 bytes from a row-major [*, 128] array, rows clamped to row_limit - 1 -> LDS, 8 one-KiB pieces shared by 4 waves.
// base is the same for all lanes of the wave.
__device__ __forceinline__ void load_tile8(const uint8_t* base, int first_row, int row_limit, uint8_t* dst, int wave, int lane) {
    const uint64_t sb = uniform_ptr(base);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int q = u * 4 + wave;
        const int r = 8 * q + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
        const uint32_t lds_addr = __builtin_amdgcn_readfirstlane(
            (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)(dst + q * 1024));
        lds_dma<16>(sb, (uint32_t)min(first_row + r, row_limit - 1) * 128u + (uint32_t)(c * 16), lds_addr);
    }
}

__device__ __forceinline__ uint32_t lds_address(const uint8_t* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t*)p;
}

__device__ __forceinline__ i32x8 lds_frag8(const uint8_t* a0, const uint8_t* a1) {
    const u32x4 lo = *reinterpret_cast<const u32x4*>(a0), hi = *reinterpret_cast<const u32x4*>(a1);
    return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
}

// S^T tile from an E4M3 K tile: st[t][i] as in qk_tile: products of the codes' values times the power of two in scale_a
__device__ __forceinline__ void qk_tile8(const uint8_t* kt, const i32x8* qf, f32x16* st, int ql, int hh, int scale_a) {
    i32x8 f[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {  // e = 2 t + kh
        const int row = 32 * (e >> 1) + ql, c0 = 4 * (e & 1) + 2 * hh;
        f[e] = lds_frag8(kt + Tile8::k_off(row, c0), kt + Tile8::k_off(row, c0 + 1));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) st[e >> 1] = mfma_f8(f[e], qf[e & 1], (e & 1) ? st[e >> 1] : f32x16{0}, scale_a);
}

// four values in [0, 1] -> one dword of 8-bit codes: E4M3 of q * 2^8, or (P_BF8) E5M2 of q * 2^15, which trades one
// mantissa bit for 14 more binades below 1: for a frozen max that may sit far above the scores
template <bool P_BF8>
__device__ __forceinline__ uint32_t pack_p8(const float* q) {
    // each conversion writes one half of w and keeps the other: start from whatever the register holds (an empty
    // asm "defines" it) instead of spending a move per dword on a zero that the second conversion overwrites
    uint32_t w0;
    asm volatile("" : "=v"(w0));
    s16x2 w = __builtin_bit_cast(s16x2, w0);
    if (P_BF8) {
        w = __builtin_amdgcn_cvt_scalef32_pk_bf8_f32(w, q[0], q[1], 0x1p-15f, false);
        w = __builtin_amdgcn_cvt_scalef32_pk_bf8_f32(w, q[2], q[3], 0x1p-15f, true);
    } else {
        w = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w, q[0], q[1], 0.00390625f, false);  // / 2^-8
        w = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w, q[2], q[3], 0.00390625f, true);
    }
    return __builtin_bit_cast(uint32_t, w);
}

// softmax step with E4M3 output: as softmax_tile, but q = min(exp2(s c - m - H), 1) (clamp modifier of the
// exponential), lsum += q, and four q's go to one dword as q * 2^8 (pk[0..7] = the B operand of P.V)
template <bool SPECIAL, bool MASKED, bool P_BF8 = false>
__device__ __forceinline__ void softmax_tile8(f32x16* st, uint32_t* pk, f32x16* ot, float& m2, float& lsum, float c,
                                              float headroom, int key0, int limit, int hh) {
    if (MASKED) {
        const int rel = limit - key0 - 4 * hh;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) st[t][r] = (32 * t + 8 * (r >> 2) + (r & 3) <= rel) ? st[t][r] : -INFINITY;
    }
    float msub = m2;
    if (SPECIAL) {
        const float mx = tile_rowmax<false>(st, 0, 0, hh);
        const float m_new = fmaxf(m2, xhalf_max(mx) * c);
        msub = (m_new == -INFINITY) ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m2 - msub);
        lsum *= alpha;
#pragma unroll
        for (int db = 0; db < 4; ++db) ot[db] *= alpha;
        m2 = m_new;
    }
    const float sub = msub + headroom;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
            float q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                q[e] = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(__builtin_fmaf(st[t][r + e], c, -sub)), 0.f, 1.f);
                lsum += q[e];
            }
            pk[4 * t + (r >> 2)] = pack_p8<P_BF8>(q);
        }
}

// The same for a frozen tile when the scores arrive as s c - m - H already (scale folded into the MFMA, the
// rest into its accumulator start): exp, sum, convert.  Nothing per score is left of the scaling and the
// subtraction, which the exact-max path cannot avoid because its m depends on the very tile.
template <bool MASKED, bool P_BF8 = false>
__device__ __forceinline__ void softmax_tile8_folded(f32x16* st, uint32_t* pk, float& lsum, int key0, int limit, int hh) {
    if (MASKED) {
        const int rel = limit - key0 - 4 * hh;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) st[t][r] = (32 * t + 8 * (r >> 2) + (r & 3) <= rel) ? st[t][r] : -INFINITY;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
            float q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                q[e] = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(st[t][r + e]), 0.f, 1.f);
                lsum += q[e];
            }
            pk[4 * t + (r >> 2)] = pack_p8<P_BF8>(q);
        }
}

// ---- Alg. 1 without exponentials (NOEXP).  The code of a small float read as an integer is a piecewise-linear
// logarithm: an E5M2 code c = 4 E + m stands for 2^(E - 15) (1 + m / 4), the chord approximation of
// 2^(c / 4 - 15), never more than 6.15 % above it.  So when a score arrives as x = s - m - H in log2 units, the
// code of exp2(x) 2^15 is, up to that chord error and the rounding to a quarter of a binade, just
// round(4 x + 120): a multiply-add, half a conversion, half a clamp and a quarter of a byte permute (see codes_tile8).  The offset is lowered by
// 4 log2(1.0303) = 0.1723 to centre the chord error: weight / exact weight lies in [0.89, 1.12] (the format's
// own rounding would give +-12.5 %).  E5M2 rather than E4M3 because the window has to hold, below the frozen max,
// the headroom, the overshoot of the seed and the spread of the row, and E4M3's subnormal codes, which the
// rounded-exponential path leans on for its last three binades, are not logarithmic.  The row sum comes from
// the same rounded weights through one more MFMA (a block of ones times P), so O = sum(w v) / sum(w) is a properly
// normalised average under weights that are each within 12 % of the exact ones; LSE inherits that error.
constexpr float kCodeOffset = 119.8277f;  // 4 * (15 + 15) - 0.1723
constexpr float kCodesPerBinade = 4.f;

// A code's worth is 256 / 65535 (kCodeUnit): v_cvt_pknorm_u16_f32 takes two values in [0, 1] to the nearest whole 65535ths, i.e. to the
// nearest 256ths of a code, z, and the code is z's upper byte.  That is one rounding and not two: with half a code less half of a
// 256th on top (kCodeHalf) z reaches 256 k exactly where the code before rounding reaches k - 1/2.  One v_perm_b32 collects four codes:
// 72 instructions a tile, where a clamp and v_cvt_pk_u8_f32 for every score took 96 (4 x 32 heads, 3000 tokens, 8-bit 175 / 169 us, 4-bit
// 155 / 150; with an add and a unit of 2^-8, which leaves a shift of up to half of a 256th, 8-bit 174 for 177, 4-bit 160 for 159).
constexpr float kCodeUnit = 256.f / 65535.f;
constexpr float kCodeHalf = 0.5f - 0x1p-9f;
constexpr uint32_t kMaxCode2 = 0x7bff7bffu;  // 0x7B = 57344, the largest finite E5M2 value, in the upper bytes of both halves
typedef __attribute__((ext_vector_type(2))) unsigned short u16x2_t;
template <bool MASKED>
__device__ __forceinline__ void codes_tile8(f32x16* st, uint32_t* pk, int key0, int limit, int hh, float add) {
    const int rel = limit - key0 - 4 * hh;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
            uint32_t w[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                float c[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int i = r + 2 * e + u;
                    c[u] = __builtin_fmaf(st[t][i], kCodesPerBinade * kCodeUnit, add);
                    if (MASKED) c[u] = 32 * t + 8 * (i >> 2) + (i & 3) <= rel ? c[u] : 0.f;
                }
                const auto q = __builtin_amdgcn_cvt_pknorm_u16(c[0], c[1]);
                w[e] = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, q), __builtin_bit_cast(u16x2_t, kMaxCode2)));
            }
            pk[4 * t + (r >> 2)] = __builtin_amdgcn_perm(w[1], w[0], 0x07050301u);
        }
}

// One query's row of O = O^T * inv in 16-byte stores, as in store_output; every lane of the wave has to get here, `live` says
// whether its row is there.
__device__ __forceinline__ void store_row8(uint16_t* Og, bool live, const f32x16* ot, float inv, int hh) {
    u32x4 w[4][2];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int e = 8 * u;  // first accumulator register of run 2u; run 2u + 1 starts four registers on
            const f32x16& o = ot[db];
            const uint32_t a0 = pack_bf16(o[e] * inv, o[e + 1] * inv), a1 = pack_bf16(o[e + 2] * inv, o[e + 3] * inv);
            const uint32_t b0 = pack_bf16(o[e + 4] * inv, o[e + 5] * inv), b1 = pack_bf16(o[e + 6] * inv, o[e + 7] * inv);
            // lower half lanes keep run 2u and receive the partner's run 2u (elements 16u .. 16u+7);
            // upper half lanes receive the partner's run 2u + 1 and keep their own (elements 16u+8 .. 16u+15)
            const auto r0 = __builtin_amdgcn_permlane32_swap(a0, b0, false, false);
            const auto r1 = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
            w[db][u] = u32x4{r0[0], r1[0], r0[1], r1[1]};
        }
    if (live) {
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int u = 0; u < 2; ++u) *reinterpret_cast<u32x4*>(Og + 32 * db + 16 * u + 8 * hh) = w[db][u];
    }
}

struct Fp8Params {
    const uint8_t* Q;      // [B, Hq, N, 128] E4M3
    const uint8_t* K;      // [B, Hkv, N, 128]
    const uint8_t* Vt;     // [B, Hkv, Tc, 128, 64]: per key tile, features x permuted keys
    const uint8_t* Krepr;  // [B, Hkv, Tc, 128]
    uint16_t* O;           // [B, Hq, N, 128] bf16
    float* LSE;
    int B, Hq, Hkv, N, Tr, Tc;
    int causal, n_sink, n_local, use_minit;
    float c;          // softmax scale * descale_q * descale_k * log2(e): multiplies the raw code products
    int scale_a;      // FOLD: that factor is a power of two and sits here as four E8M0 bytes (then c = 1)
    float descale_v;  // multiplies O
    float headroom;   // H above
};

// The tile products that Alg. 1's max is taken from in front of the main loop (all its blocks are frozen ones then, see
// attn_frozen.hpp): tiles [0, n_sum) of the block summaries that cover the nv visible key blocks, then the sink and the local
// blocks of K.  An 8-bit Q.K^T is cheap beside the exact-max softmax of a tile (max chain, rescale of l and O), which this
// form does not have: see attn_fp8_kernel.
struct MaxTiles {
    int n_sum, n1, lo2, total;
    __device__ __forceinline__ int block(int t) const { return t - n_sum < n1 ? t - n_sum : lo2 + (t - n_sum - n1); }  // of K, for t >= n_sum
};
__device__ __forceinline__ MaxTiles max_tiles(int use_minit, int n_sink, int n_local, int a_lo, int a_hi, int nv) {
    MaxTiles m;
    m.n_sum = use_minit ? (nv + BN - 1) / BN : 0;
    m.n1 = min(n_sink, nv);
    m.lo2 = max(max(0, a_lo - (n_local - 1)), m.n1);
    m.total = m.n_sum + m.n1 + (n_local > 0 ? max(0, min(a_hi, nv - 1) + 1 - m.lo2) : 0);
    return m;
}

// One workgroup = 4 waves x 32 query rows = one 128-row query block of one head; three-deep K / V^T ring (48 KiB, the max phase in its
// second and third stage), filled two tiles ahead, three workgroups per CU.  MODE_FA or MODE_VFA.
// What bounds it: on long sequences the matrix unit at the clock the power budget leaves (16384 tokens, 2 x 32 heads: 760 cycles a wave
// and tile at 1.7 GHz, 512 of them MFMA; the vector unit needs 490 for 32 exponentials, 32 adds and 16 conversions, the latter as slow
// as an exponential); on short ones the start of an item (a tile's latencies, 3 to 4 us of them the max phase) too.  Attention
// alone in us, before / after the deeper ring, the buffer loads and fragment addresses that stay in registers (no other vector
// instruction left in a tile): folded, 32 heads, 8192 tokens 266 / 252, 4 x 3000 178 / 169, 777 14.9 / 13.8, 2 x 16384 1987 / 1879.
// FOLD (Alg. 1 only, when the factor between code products and log2-domain scores is a power of two): the
// K operand's block scale applies it inside every Q.K^T MFMA, and on frozen tiles the accumulators start at
// -(m + H), so the scores come out of the matrix unit ready for exp2.
template <int MODE, bool FOLD, bool NOEXP = false>
__global__ __launch_bounds__(256, FOLD ? 3 : 2) void attn_fp8_kernel(const Fp8Params p) {
    static_assert(!FOLD || MODE == MODE_VFA, "folding needs a max that is known before the tile");
    static_assert(!NOEXP || FOLD, "codes straight from the matrix unit need the scale and the max folded into it");
    const int sa = FOLD ? p.scale_a : 0x7f7f7f7f;
    constexpr int D = 128, BM = 128, DB = 4;
    constexpr int S = 3, STAGE = Tile8::KBYTES + Tile8::VBYTES;  // stages of a K and a V^T tile
    __shared__ __attribute__((aligned(16))) uint8_t smem[S * STAGE];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ql = lane & 31, hh = lane >> 5;
    const int g = p.Hq / p.Hkv;
    int b, h, i;
    {
        const int id = blockIdx.x, G = p.B * p.Hkv;
        if ((G & 7) == 0) {
            const int x = id & 7, y = id >> 3;
            const int per = p.Tr * g;
            const int kvl = y / per, rem = y - kvl * per;
            i = p.Tr - 1 - rem / g;
            const int kv = kvl * 8 + x;
            b = kv / p.Hkv;
            h = (kv - b * p.Hkv) * g + rem % g;
        } else {
            const int bh = id % (p.B * p.Hq);
            i = p.Tr - 1 - id / (p.B * p.Hq);
            b = bh / p.Hq;
            h = bh - b * p.Hq;
        }
    }
    const int hkv = h / g, N = p.N;
    const int row0 = i * BM, last_row = min(N, row0 + BM) - 1;
    const int a_lo = row0 / BN, a_hi = last_row / BN;
    const int j_hi = p.causal ? a_hi : p.Tc - 1;
    const uint8_t* Kg = p.K + ((size_t)(b * p.Hkv + hkv) * N) * D;
    const uint8_t* Vg = p.Vt + ((size_t)(b * p.Hkv + hkv) * p.Tc) * Tile8::VBYTES;
    const int qrow = row0 + 32 * wave + ql, qrow_c = min(qrow, N - 1);
    const int limit = p.causal ? qrow_c : N - 1;
    i32x8 qf[2];
    {
        const uint8_t* qp = p.Q + ((size_t)(b * p.Hq + h) * N + qrow_c) * D + 32 * hh;
#pragma unroll
        for (int kh = 0; kh < 2; ++kh) {
            const u32x4 lo = *reinterpret_cast<const u32x4*>(qp + 64 * kh), hi = *reinterpret_cast<const u32x4*>(qp + 64 * kh + 16);
            qf[kh] = i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
        }
    }
    const int nv = j_hi + 1;
    const uint32_t off_k = (uint32_t)((16 * wave + (lane >> 3)) * 128 + (((lane & 7) ^ (lane >> 4)) << 4)), off_k1 = off_k ^ 64;
    const uint32_t off_v = (uint32_t)((32 * wave + (lane >> 2)) * 64 + (((lane & 3) ^ ((lane >> 4) & 3)) << 4));
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem)) + 2048 * wave;
    auto load_kv = [&](int j, uint32_t stage) __attribute__((always_inline)) {  // (stage: its byte offset; past the last tile nothing is read)
        request2((uint64_t)(uintptr_t)Kg + (uint32_t)j * 8192ull, (uint32_t)(j < nv ? min(N - j * BN, BN) : 0) * 128u, off_k, off_k1, lds0 + stage);
        request2((uint64_t)(uintptr_t)Vg + (uint32_t)j * 8192ull, j < nv ? 8192u : 0u, off_v, off_v, lds0 + stage + Tile8::KBYTES);
    };
    float m2 = -INFINITY;
    if (MODE == MODE_VFA) {
        // four tiles at a time, staged in the ring behind its first stage, which takes the main loop's first tiles
        const uint8_t* Rg = p.Krepr + ((size_t)(b * p.Hkv + hkv) * p.Tc) * D;
        const MaxTiles mt = max_tiles(p.use_minit, p.n_sink, p.n_local, a_lo, a_hi, nv);
        auto stage = [&](int u) __attribute__((always_inline)) { return smem + STAGE + u * Tile8::KBYTES; };
        float mx = -INFINITY;
        for (int t0 = 0; t0 < mt.total; t0 += 4) {
            if (t0) __syncthreads();
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u;  // (summaries: rows clamped to the visible blocks; a repeated row changes no max)
                if (t < mt.total) load_tile8(t < mt.n_sum ? Rg : Kg, (t < mt.n_sum ? t : mt.block(t)) * BN, t < mt.n_sum ? nv : N, stage(u), wave, lane);
            }
            if (t0 == 0) {
                load_kv(0, 0);
                __builtin_amdgcn_s_waitcnt(0x0F74);  // vmcnt(4): the staged tiles have landed, not yet those of the main loop
            } else {
                __builtin_amdgcn_s_waitcnt(0x0F70);
            }
            __syncthreads();
#pragma unroll 1
            for (int t = t0; t < min(t0 + 4, mt.total); ++t) {
                f32x16 st[2];
                qk_tile8(stage(t - t0), qf, st, ql, hh, sa);
                const int j = mt.block(t);
                if (t < mt.n_sum || (j * BN + BN <= N && !(p.causal && j * BN + BN - 1 > row0))) mx = fmaxf(mx, tile_rowmax<false>(st, 0, 0, hh));
                else mx = fmaxf(mx, tile_rowmax<true>(st, j * BN, limit, hh));
            }
        }
        m2 = finite_max(xhalf_max(mx) * p.c);
    } else {
        load_kv(0, 0);
    }
    wait_vm0_and_sync();
    f32x16 ot[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) ot[db] = f32x16{0};
    float lsum = 0.f;
    f32x16 start;  // FOLD: -(m + H) of this lane's query in all 16 registers, set once the max is frozen
    float code0 = 0.f;  // NOEXP: code offset - 4 (m + H), added on the vector side (16 registers matter more than 32 adds)
    f32x16 lt = {0};  // NOEXP: 32 copies of this lane's row sum of the rounded weights (times 2^15)
    if (FOLD) {
        const float v = -(m2 + p.headroom);
        if (NOEXP) code0 = kCodeUnit * (kCodeOffset + kCodeHalf + kCodesPerBinade * v);
#pragma unroll
        for (int r = 0; r < 16; ++r) start[r] = v;
    }
    load_kv(1, STAGE);
    // fragment addresses in a stage: all others follow by constant offsets, which go into the instructions (the loop is unrolled by
    // the stages)
    uint32_t ka[4], va[2];
#pragma unroll
    for (int e = 0; e < 4; ++e) ka[e] = lds_address(smem) + Tile8::k_off(ql, 4 * (e >> 1) + 2 * hh + (e & 1));
#pragma unroll
    for (int e = 0; e < 2; ++e) va[e] = lds_address(smem) + Tile8::KBYTES + Tile8::v_off(ql, 2 * hh + e);
    typedef const __attribute__((address_space(3))) u32x4* lds_ptr;
    auto frag = [&](uint32_t a0, uint32_t a1, uint32_t off) __attribute__((always_inline)) {
        const u32x4 lo = *(lds_ptr)(a0 + off), hi = *(lds_ptr)(a1 + off);
        return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
    };
    // One tile; MASKED is compile-time so that each of the two loops below has one softmax body (the baseline's takes the exact
    // max, Alg. 1's is a frozen one).
    auto visit = [&](int j, uint32_t stage, uint32_t next2, auto masked_c) __attribute__((always_inline)) {
        constexpr bool SPECIAL = is_fa(MODE), MASKED = decltype(masked_c)::value;
        f32x16 st[2];
        uint32_t pk[8];
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const i32x8 g0 = frag(ka[0], ka[1], stage + t * 4096), g1 = frag(ka[2], ka[3], stage + t * 4096);
            st[t] = mfma_f8(g0, qf[0], FOLD && !NOEXP ? start : f32x16{0}, sa);
            st[t] = mfma_f8(g1, qf[1], st[t], sa);
        }
        __builtin_amdgcn_s_setprio(0);
        load_kv(j + 2, next2);
        const bool needs_mask = (p.causal && j * BN + BN - 1 > row0) || (j + 1) * BN > N;
        if (NOEXP) codes_tile8<MASKED>(st, pk, j * BN, needs_mask ? limit : 0x3fffffff, hh, code0);
        else if (FOLD) softmax_tile8_folded<MASKED>(st, pk, lsum, j * BN, needs_mask ? limit : 0x3fffffff, hh);
        else softmax_tile8<SPECIAL, MASKED>(st, pk, ot, m2, lsum, p.c, p.headroom, j * BN, needs_mask ? limit : 0x3fffffff, hh);
        const i32x8 pf = {(int)pk[0], (int)pk[1], (int)pk[2], (int)pk[3], (int)pk[4], (int)pk[5], (int)pk[6], (int)pk[7]};
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const i32x8 g = frag(va[0], va[1], stage + db * 2048);
            ot[db] = NOEXP ? __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(g, pf, ot[db], 0, 1, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f) : mfma_f8(g, pf, ot[db]);
        }
        if (NOEXP) {
            // row sums of the rounded weights: a block of ones times P (E5M2).  The ones are E2M1 (1.0 = code 2): a
            // 4-bit operand takes four registers instead of eight, and with all elements equal the different order of
            // the k index in 4-bit and 8-bit operands does not matter
            const i32x8 ones = {0x22222222, 0x22222222, 0x22222222, 0x22222222, 0, 0, 0, 0};
            lt = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ones, pf, lt, 4, 1, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f);
        }
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_s_waitcnt(0x0F74);  // vmcnt(4): tile j + 1 has landed
        __syncthreads();
    };
    using std::false_type;
    using std::true_type;
    int j_masked = p.causal ? a_lo : p.Tc;  // first tile that needs masking
    if (N % BN) j_masked = min(j_masked, p.Tc - 1);
    int j = 0;
    for (; j + S <= min(j_masked, nv); j += S) {
        visit(j, 0, 2 * STAGE, false_type{});
        visit(j + 1, STAGE, 0, false_type{});
        visit(j + 2, 2 * STAGE, STAGE, false_type{});
    }
#pragma unroll 1
    for (uint32_t stage = 0; j < nv; ++j) {
        const uint32_t next = stage == 2 * STAGE ? 0 : stage + STAGE;
        visit(j, stage, next == 2 * STAGE ? 0 : next + STAGE, true_type{});
        stage = next;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // (requests past the last tile write zeros to LDS: not behind this workgroup's end)
    // O = descale_v * 2^-8 * O^T / l (the codes of P carry 2^8); LSE = (m2 + H + log2 l) ln 2  (l sums exp2(s c - m2 - H))
    // (NOEXP: every register of lt holds the whole row sum, with the same 2^15 as the numerator)
    const float l = NOEXP ? lt[0] * 0x1p-15f : xhalf_sum(lsum);
    const float inv = l > 0.f ? p.descale_v * (NOEXP ? 0x1p-15f : 0x1p-8f) / l : 0.f;
    const size_t row = (size_t)(b * p.Hq + h) * N + qrow;
    store_row8(p.O + row * D, qrow < N, ot, inv, hh);
    if (qrow < N && p.LSE && hh == 0)
        p.LSE[row] = l > 0.f ? (m2 + p.headroom + __builtin_amdgcn_logf(l)) * kLn2 : -INFINITY;
}

// The run `i` of eight elements (zeros past the end).  STREAM: a non-temporal load.
template <bool STREAM>
__device__ __forceinline__ u32x4 quant_load(const uint16_t* __restrict__ X, long long i, long long n8) {
    if (i >= n8) return u32x4{0, 0, 0, 0};
    const u32x4* const a = reinterpret_cast<const u32x4*>(X + i * 8);
    return STREAM ? __builtin_nontemporal_load(a) : *a;
}
// bf16 -> E4M3 codes of x * inv_scale (saturated at +-448), same layout.  A workgroup takes QUANT_CHUNKS * 256 runs of eight
// elements, all loads in flight at once (see vfa_fp8_quantize for how many).
template <int QUANT_CHUNKS, bool STREAM>
__global__ __launch_bounds__(256) void fp8_quantize_kernel(const uint16_t* __restrict__ X, uint8_t* __restrict__ Y,
                                                           long long n8, float inv_scale) {
    const long long i0 = (long long)blockIdx.x * (256 * QUANT_CHUNKS) + threadIdx.x;
    u32x4 x[QUANT_CHUNKS];
#pragma unroll
    for (int u = 0; u < QUANT_CHUNKS; ++u)
        x[u] = quant_load<STREAM>(X, i0 + 256 * u, n8);
#pragma unroll
    for (int u = 0; u < QUANT_CHUNKS; ++u) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[2 * e] = fminf(fmaxf(__uint_as_float(x[u][e] << 16) * inv_scale, -448.f), 448.f);
            v[2 * e + 1] = fminf(fmaxf(__uint_as_float(x[u][e] & 0xffff0000u) * inv_scale, -448.f), 448.f);
        }
        int w0 = __builtin_amdgcn_cvt_pk_fp8_f32(v[0], v[1], 0, false);
        w0 = __builtin_amdgcn_cvt_pk_fp8_f32(v[2], v[3], w0, true);
        int w1 = __builtin_amdgcn_cvt_pk_fp8_f32(v[4], v[5], 0, false);
        w1 = __builtin_amdgcn_cvt_pk_fp8_f32(v[6], v[7], w1, true);
        if (i0 + 256 * u < n8) *reinterpret_cast<u32x2*>(Y + (i0 + 256 * u) * 8) = u32x2{(uint32_t)w0, (uint32_t)w1};
    }
}

// V [BH, N, 128] bf16 -> per 64-key tile a [128 features][64 keys] E4M3 block with the keys in the order the
// P.V operand wants them (byte 32 hh + j of a row = key 32 (j / 16) + 8 ((j % 16) / 4) + 4 hh + j % 4);
// keys beyond N are written as 0.  One workgroup per (tile, head).  Four neighbouring bytes of a row are four neighbouring
// keys, so a thread takes four keys x eight features with 16-byte loads, converts straight into the eight dwords, and only
// those go through LDS, to leave in 16-byte pieces of whole rows.  HBM bound (4 x 8 heads of 3000 keys, 36 MiB: 13.9 us when
// each byte was stored and gathered by itself, 8.1 now).
__global__ __launch_bounds__(256) void fp8_pack_v_kernel(const uint16_t* __restrict__ V, uint8_t* __restrict__ Vt, int N,
                                                         int Tc, float inv_scale) {
    // dword q (keys) of feature f at f * 16 + (q ^ 4 ((f / 8) % 4)): 16-byte pieces stay whole, features 8 apart use other banks
    __shared__ __attribute__((aligned(16))) uint32_t rows[128 * 16];
    const int j = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x;
    const int fc = tid & 15, kg = tid >> 4;  // features 8 fc .. + 7, keys 4 kg .. + 3
    const uint16_t* src = V + ((size_t)bh * N + (size_t)j * BN + 4 * kg) * 128 + 8 * fc;
    u32x4 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        x[u] = j * BN + 4 * kg + u < N ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + u * 128)) : u32x4{0, 0, 0, 0};
    const int q = 8 * (kg & 1) + 4 * (kg >> 3) + ((kg & 7) >> 1);  // byte 32 (kg % 2) + 16 (kg / 8) + 4 ((kg % 8) / 2) of the row
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t w = x[u][e >> 1];
            v[u] = fminf(fmaxf(__uint_as_float((e & 1) ? w & 0xffff0000u : w << 16) * inv_scale, -448.f), 448.f);
        }
        int c = __builtin_amdgcn_cvt_pk_fp8_f32(v[0], v[1], 0, false);
        c = __builtin_amdgcn_cvt_pk_fp8_f32(v[2], v[3], c, true);
        rows[(8 * fc + e) * 16 + (q ^ (4 * (fc & 3)))] = (uint32_t)c;
    }
    __syncthreads();
    uint8_t* dst = Vt + ((size_t)bh * Tc + j) * Tile8::VBYTES;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int idx = 256 * u + tid, f = idx >> 2, c = idx & 3;  // 16-byte piece c of feature f
        *reinterpret_cast<u32x4*>(dst + idx * 16) = *reinterpret_cast<const u32x4*>(&rows[f * 16 + 4 * (c ^ ((f >> 3) & 3))]);
    }
}

// sabsmax over E4M3 codes (sign-magnitude: the 7 low bits order the magnitudes; tie -> the positive code, the
// smaller one; the rule is commutative and associative, so any reduction order gives the same bytes).
// 256 threads: thread (rg, ch) takes the 16-byte chunk ch of rows rg and rg + 32 (rows past the end of a ragged
// block repeat its last row, which changes nothing), then 128 threads fold the 32 partial rows of one feature each.
__device__ __forceinline__ uint32_t fp8_sabs_pick(uint32_t a, uint32_t b) {
    const uint32_t ma = a & 0x7f, mb = b & 0x7f;
    return mb > ma ? b : (ma > mb ? a : min(a, b));
}
__global__ __launch_bounds__(256) void fp8_kblock_summary_kernel(const uint8_t* __restrict__ K, uint8_t* __restrict__ R, int N,
                                                                 int Tc) {
    __shared__ u32x4 part[32][8];
    const int j = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x;
    const int rg = tid >> 3, ch = tid & 7;
    const int rows = min(BN, N - j * BN);
    const uint8_t* base = K + ((size_t)bh * N + (size_t)j * BN) * 128 + ch * 16;
    const u32x4 a = *reinterpret_cast<const u32x4*>(base + (size_t)min(rg, rows - 1) * 128);
    const u32x4 b = *reinterpret_cast<const u32x4*>(base + (size_t)min(rg + 32, rows - 1) * 128);
    u32x4 best;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t w = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) w |= fp8_sabs_pick((a[e] >> (8 * q)) & 0xffu, (b[e] >> (8 * q)) & 0xffu) << (8 * q);
        best[e] = w;
    }
    part[rg][ch] = best;
    __syncthreads();
    if (tid < 128) {
        const uint8_t* col = reinterpret_cast<const uint8_t*>(&part[0][0]) + tid;
        uint32_t v = col[0];
        for (int r = 1; r < 32; ++r) v = fp8_sabs_pick(v, col[r * 128]);
        R[((size_t)bh * Tc + j) * 128 + tid] = (uint8_t)v;
    }
}

}  // namespace
