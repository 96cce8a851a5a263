// Attention with MXFP4 scores (E2M1 elements, E8M0 block scales) and its pre-passes.
#pragma once
#include "common.hpp"
#include "fp8.hpp"

namespace {

// ---------------------------------------------------------------------------------------------
// MXFP4 scores: the 4-bit tensor regime (Q.K^T on E2M1 elements with one E8M0 scale per 32 features, the
// published MX block format; P.V stays on E4M3 as above, since exp(S - m) in [0, 1] needs more than the one
// mantissa bit of E2M1).  v_mfma_scale_f32_32x32x64_f8f6f4 with both operands E2M1 runs a 64-deep step in
// 32 cycles, twice the E4M3 rate, and takes the block scales as operands: lane (row, half hh) supplies the
// scale byte of its own 32 elements, k = 32 hh .. 32 hh + 31 of the step, which are features
// 64 kh + 32 hh .. + 31: exactly one MX block.  The scale byte is replicated into all four bytes of its
// register, so the byte select of the instruction does not matter.
// Key-block summaries of MXFP4 keys are not MXFP4 vectors (their entries come from keys with different
// scales): they are kept as MX blocks of E5M2 elements (two mantissa bits cover the one of E2M1, and the 29
// binades below the block maximum cover the spread of the keys' scales), and the m-initialisation multiplies
// them with the E2M1 queries in the same instruction (A = E5M2, B = E2M1).  Measured for that mixed form: the
// k index of an element is 32 hh + j for nibble j of a 4-bit operand, but 16 hh + j (j < 16) or
// 32 + 16 hh + (j - 16) for byte j of an 8-bit operand, and the scale of lane half b covers k = 32 b .. 32 b + 31
// in both (for 8-bit data: bytes 16 b .. 16 b + 15 of BOTH halves).  Two operands of equal width pair up whatever
// the order, which is all the paths above need; here the summary's 16-byte chunks are picked to match.
struct Tile4 {
    static constexpr int KBYTES = BN * 64;  // K tile: 64 rows of 64 bytes (128 nibbles)
    // 16-byte chunk c (0..3) of row r sits at chunk position c ^ ((r >> 2) & 3): 16 consecutive rows reading one
    // logical chunk cover all 64 banks
    __device__ static int k_off(int r, int c) { return r * 64 + ((c ^ ((r >> 2) & 3)) << 4); }
};

// X bf16 -> MXFP4: thread = 8 consecutive elements, 4 threads = one block of 32.  y = x * pre_scale (fp32);
// scale byte = exponent field of max|y| - 2, at least 0; element = y / 2^(byte - 127) rounded to the nearest
// of 0, 0.5, 1, 1.5, 2, 3, 4, 6, ties to the even mantissa, saturated at 6.  The rounding is integer arithmetic on the bits of
// |y| 2^(127 - byte): from 1 up the code is the top of the float rounded to one mantissa bit (nearest even: half an ulp less
// one, plus the bit that stays last), below 1 it is 2 |y| rounded to a whole number (nearest even), and at 1 the two agree.
// (Seven comparisons per element took 36 us for 94 MiB, bound by the vector unit; 31 now.)
template <int QUANT_CHUNKS, bool STREAM>
__global__ __launch_bounds__(256) void mx4_quantize_kernel(const uint16_t* __restrict__ X, uint8_t* __restrict__ Y,
                                                           uint8_t* __restrict__ S, long long n8, float pre_scale) {
    // (a workgroup's loads as in fp8_quantize_kernel.  n8 is a multiple of 4, so the four threads of a block are live together)
    const long long i0 = (long long)blockIdx.x * (256 * QUANT_CHUNKS) + threadIdx.x;
    u32x4 x[QUANT_CHUNKS];
#pragma unroll
    for (int u = 0; u < QUANT_CHUNKS; ++u)
        x[u] = quant_load<STREAM>(X, i0 + 256 * u, n8);
#pragma unroll
    for (int u = 0; u < QUANT_CHUNKS; ++u) {
        const long long i = i0 + 256 * u;
        float v[8];
        float amax = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[2 * e] = __uint_as_float(x[u][e] << 16) * pre_scale;
            v[2 * e + 1] = __uint_as_float(x[u][e] & 0xffff0000u) * pre_scale;
            amax = fmaxf(amax, fmaxf(fabsf(v[2 * e]), fabsf(v[2 * e + 1])));
        }
        amax = fmaxf(amax, __shfl_xor(amax, 1));
        amax = fmaxf(amax, __shfl_xor(amax, 2));
        const int ef = (int)((__float_as_uint(amax) >> 23) & 0xffu);
        const int sb = max(ef - 2, 0);
        const float mult = __uint_as_float((uint32_t)(254 - sb) << 23);  // 2^(127 - sb)
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float y = __builtin_amdgcn_fmed3f(fabsf(v[e]) * mult, 0.f, 6.f);  // (a NaN becomes 0)
            const uint32_t b = __float_as_uint(y);
            const uint32_t hi = ((b + 0x1fffffu + ((b >> 22) & 1u)) >> 22) - 252u;  // 1.0 = 0x3f800000 -> 254 -> code 2
            const uint32_t lo = (uint32_t)__builtin_rintf(y + y);
            uint32_t c = y < 1.f ? lo : hi;
            c |= (__float_as_uint(v[e]) >> 28) & 8u;
            w |= c << (4 * e);
        }
        if (i < n8) {
            *reinterpret_cast<uint32_t*>(Y + i * 4) = w;
            if ((threadIdx.x & 3) == 0) S[i >> 2] = (uint8_t)sb;
        }
    }
}

// sabsmax of a block of MXFP4 keys, per feature over the dequantised values (tie -> the positive one), stored
// as MX blocks of E5M2: scale byte = exponent field of the block maximum - 15; codes [B*Hkv, Tc, 128],
// scales [B*Hkv, Tc, 4].  Magnitudes are compared as whole numbers: an element of magnitude code m (1 .. 7) under scale byte s
// has rank 2 s + {0, 2, 3, 4, 5, 6, 7}[m - 1] + 2 (two ranks to a binade, so equal values have equal ranks whatever their scales),
// a zero has rank 0, and the key (rank << 1 | positive) picks the larger magnitude and of equal ones the positive.
// 256 threads: thread (row group, c) takes dword c (eight features) of four rows (rows past the end of a ragged block repeat its
// last row); lanes, then the four waves, combine.
__global__ __launch_bounds__(256) void mx4_kblock_summary_kernel(const uint8_t* __restrict__ K4, const uint8_t* __restrict__ KS,
                                                                 uint8_t* __restrict__ R, uint8_t* __restrict__ RS, int N,
                                                                 int Tc) {
    __shared__ uint32_t part[4][128];
    const int j = blockIdx.x, bh = blockIdx.y, tid = threadIdx.x;
    const int rows = min(BN, N - j * BN);
    const int c = tid & 15, rg = tid >> 4;
    uint32_t best[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) best[q] = 1u;  // +0
    uint32_t w[4], sc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const size_t r = (size_t)bh * N + (size_t)j * BN + min(4 * rg + u, rows - 1);
        w[u] = *reinterpret_cast<const uint32_t*>(K4 + r * 64 + 4 * c);
        sc[u] = KS[r * 4 + (c >> 2)];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t code = (w[u] >> (4 * q)) & 0xfu, m = code & 7u;
            const uint32_t rank = m == 0u ? 0u : 2u * sc[u] + 2u + (m == 1u ? 0u : m);
            best[q] = max(best[q], (rank << 1) | (code < 8u ? 1u : 0u));
        }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        best[q] = max(best[q], (uint32_t)__shfl_xor((int)best[q], 16));
        best[q] = max(best[q], (uint32_t)__shfl_xor((int)best[q], 32));
    }
    if ((tid & 63) < 16)
#pragma unroll
        for (int q = 0; q < 8; ++q) part[tid >> 6][8 * c + q] = best[q];
    __syncthreads();
    if (tid < 128) {
        const int t = tid;
        const uint32_t key = max(max(part[0][t], part[1][t]), max(part[2][t], part[3][t]));
        const int rank = (int)(key >> 1) - 2;  // 2 E + man: the magnitude is (1 + man / 2) 2^(E - 1 - 127)
        float v = key < 2u ? 0.f : __builtin_ldexpf((rank & 1) ? 1.5f : 1.f, (rank >> 1) - 128);
        v = (key & 1u) ? v : -v;
        v = v == 0.f ? 0.f : v;  // (a column of zeros of either sign: +0)
        float amax = fabsf(v);
#pragma unroll
        for (int o = 16; o >= 1; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o));  // the 32 features of one MX block
        const int ef = (int)((__float_as_uint(amax) >> 23) & 0xffu);
        const int sb = max(ef - 15, 0);
        const float y = __builtin_ldexpf(v, 127 - sb);  // at most 1.5 * 2^15: inside E5M2's finite range
        R[((size_t)bh * Tc + j) * 128 + t] = (uint8_t)(__builtin_amdgcn_cvt_pk_bf8_f32(y, 0.f, 0, false) & 0xff);
        if ((t & 31) == 0) RS[((size_t)bh * Tc + j) * 4 + (t >> 5)] = (uint8_t)sb;
    }
}

__device__ __forceinline__ f32x16 mfma_f4(const u32x4& a, const u32x4& b, const f32x16& c, int scale_a, int scale_b) {
    const i32x8 av = {(int)a[0], (int)a[1], (int)a[2], (int)a[3], 0, 0, 0, 0};
    const i32x8 bv = {(int)b[0], (int)b[1], (int)b[2], (int)b[3], 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 4, 4, 0, scale_a, 0, scale_b);
}
__device__ __forceinline__ f32x16 mfma_bf8_f4(const i32x8& a, const u32x4& b, const f32x16& c, int scale_a, int scale_b) {
    const i32x8 bv = {(int)b[0], (int)b[1], (int)b[2], (int)b[3], 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, bv, c, 1, 4, 0, scale_a, 0, scale_b);
}

// byte n (0..3, per lane) of x in all four bytes
__device__ __forceinline__ int spread_byte(uint32_t x, uint32_t n) {
    return (int)__builtin_amdgcn_perm(x, x, n * 0x01010101u);
}

// 64 dwords (the four scale bytes of rows first_row .. first_row + 63 of a row-major [*, 4] array, rows clamped
// to row_limit - 1) -> LDS, by one wave; base is the same for all lanes
__device__ __forceinline__ void load_scales64(const uint8_t* base, int first_row, int row_limit, uint32_t* dst, int lane) {
    const uint32_t lds_addr =
        __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)dst);
    lds_dma<4>(uniform_ptr(base), (uint32_t)min(first_row + lane, row_limit - 1) * 4u, lds_addr);
}

// MXFP4 K tile (64 rows of 64 bytes from a row-major [*, 64] array, rows clamped) -> LDS: four one-KiB pieces,
// one per wave; base is the same for all lanes
__device__ __forceinline__ void load_tile4(const uint8_t* base, int first_row, int row_limit, uint8_t* dst, int wave,
                                           int lane) {
    const int r = 16 * wave + (lane >> 2);
    const int c = (lane & 3) ^ ((r >> 2) & 3);
    const uint32_t lds_addr = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)(dst + wave * 1024));
    lds_dma<16>(uniform_ptr(base), (uint32_t)min(first_row + r, row_limit - 1) * 64u + (uint32_t)(c * 16), lds_addr);
}

// S^T tile from an MXFP4 K tile and its scales: st[t][i] as in qk_tile, in units of the dequantised products
// (the block scales are applied inside the instruction)
__device__ __forceinline__ void qk_tile4(const uint8_t* kt, const uint32_t* ksc, const u32x4* qf, const int* qs, f32x16* st,
                                         int ql, int hh) {
    u32x4 f[4];
    uint32_t sc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) sc[t] = ksc[32 * t + ql];
#pragma unroll
    for (int e = 0; e < 4; ++e)  // e = 2 t + kh
        f[e] = *reinterpret_cast<const u32x4*>(kt + Tile4::k_off(32 * (e >> 1) + ql, 2 * (e & 1) + hh));
#pragma unroll
    for (int e = 0; e < 4; ++e)
        st[e >> 1] = mfma_f4(f[e], qf[e & 1], (e & 1) ? st[e >> 1] : f32x16{0}, spread_byte(sc[e >> 1], 2 * (e & 1) + hh), qs[e & 1]);
}

struct Mx4Params {
    const uint8_t* Q;       // [B, Hq, N, 64] E2M1 pairs
    const uint8_t* Qs;      // [B, Hq, N, 4] E8M0
    const uint8_t* K;       // [B, Hkv, N, 64]
    const uint8_t* Ks;      // [B, Hkv, N, 4]
    const uint8_t* Vt;      // [B, Hkv, Tc, 128, 64] E4M3, as in the FP8 path
    const uint8_t* Krepr;   // [B, Hkv, Tc, 128] E5M2
    const uint8_t* KreprS;  // [B, Hkv, Tc, 4] E8M0
    uint16_t* O;
    float* LSE;
    int B, Hq, Hkv, N, Tr, Tc;
    int causal, n_sink, n_local, use_minit;
    float c;          // softmax scale * log2(e) (1 when FOLD)
    float descale_v;
    float headroom;
};

// As attn_fp8_kernel with the score product on MXFP4 operands.  FOLD (Alg. 1 only, softmax scale * log2(e) = 1,
// i.e. the caller folded that factor into Q before quantising): frozen tiles start their accumulators at
// -(m + H) and go to exp2 untouched.
// NOEXP (with FOLD): the weights' E5M2 codes are taken from the scores as in attn_fp8_kernel's form without
// exponentials.
// The loop is that of attn_fp8_kernel.  Attention alone in us, before / after it (and, without exponentials, codes by
// v_cvt_pknorm_u16_f32): 4 x 32 heads, 3000 tokens, without exponentials 155 / 143, folded 164 / 156; 8192 tokens 231 / 214, 242 / 232.
template <int MODE, bool FOLD, bool NOEXP = false>
__global__ __launch_bounds__(256, 3) void attn_mx4_kernel(const Mx4Params p) {
    static_assert(!FOLD || MODE == MODE_VFA, "folding needs a max that is known before the tile");
    static_assert(!NOEXP || FOLD, "codes straight from the matrix unit need the scores in log2 units");
    constexpr int D = 128, BM = 128, DB = 4;
    // Alg. 1 keeps exp(S - m) in E5M2: the summaries of MXFP4 keys collect the upward rounding errors of 64 keys per
    // feature, so the seeded max can sit ten binades above the scores, more than E4M3 has to spare
    constexpr bool P_BF8 = MODE == MODE_VFA;
    // three stages of a K tile of 4 KiB and a V^T tile of 8 KiB; Alg. 1: one tile of 8 KiB more for the max phase (with the second and
    // third stage four slots, each large enough for a tile of summaries)
    constexpr int S = 3, STAGE = Tile4::KBYTES + Tile8::VBYTES;
    __shared__ __attribute__((aligned(16))) uint8_t smem[S * STAGE + (MODE == MODE_VFA ? Tile8::KBYTES : 0)];
    __shared__ uint32_t kscale[4][S][BN];  // (a copy for each wave: every wave then waits for the same number of requests)
    __shared__ uint32_t mscale[MODE == MODE_VFA ? 4 : 1][BN];
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
    const uint8_t* Kg = p.K + ((size_t)(b * p.Hkv + hkv) * N) * 64;
    const uint8_t* Ksg = p.Ks + ((size_t)(b * p.Hkv + hkv) * N) * 4;
    const uint8_t* Vg = p.Vt + ((size_t)(b * p.Hkv + hkv) * p.Tc) * Tile8::VBYTES;
    const int qrow = row0 + 32 * wave + ql, qrow_c = min(qrow, N - 1);
    const int limit = p.causal ? qrow_c : N - 1;
    u32x4 qf[2];
    int qs[2];
    {
        const size_t qr = (size_t)(b * p.Hq + h) * N + qrow_c;
        const uint32_t sw = *reinterpret_cast<const uint32_t*>(p.Qs + qr * 4);
#pragma unroll
        for (int kh = 0; kh < 2; ++kh) {
            qf[kh] = *reinterpret_cast<const u32x4*>(p.Q + qr * 64 + 32 * kh + 16 * hh);
            qs[kh] = spread_byte(sw, 2 * kh + hh);
        }
    }
    const int nv = j_hi + 1;
    const uint32_t off_k = (uint32_t)((16 * wave + (lane >> 2)) * 64 + (((lane & 3) ^ ((lane >> 4) & 3)) << 4));
    const uint32_t off_v = (uint32_t)((32 * wave + (lane >> 2)) * 64 + (((lane & 3) ^ ((lane >> 4) & 3)) << 4));
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem)), lds_k = lds0 + 1024 * wave, lds_v = lds0 + Tile4::KBYTES + 2048 * wave;
    const uint32_t lds_s = __builtin_amdgcn_readfirstlane(lds_address(reinterpret_cast<const uint8_t*>(kscale[wave])));
    auto load_kv = [&](int j, uint32_t stage, uint32_t st) __attribute__((always_inline)) {  // (stage = its byte offset, st = its number; past the last tile nothing is read)
        const uint32_t rows = (uint32_t)(j < nv ? min(N - j * BN, BN) : 0);
        request1((uint64_t)(uintptr_t)Kg + (uint32_t)j * 4096ull, rows * 64u, off_k, lds_k + stage);
        request2((uint64_t)(uintptr_t)Vg + (uint32_t)j * 8192ull, j < nv ? 8192u : 0u, off_v, off_v, lds_v + stage);
        request_dwords((uint64_t)(uintptr_t)Ksg + (uint32_t)j * 256ull, rows * 4u, lane * 4u, lds_s + st * 256u);
    };
    float m2 = -INFINITY;
    if (MODE == MODE_VFA) {
        // as in attn_fp8_kernel
        const uint8_t* Rg = p.Krepr + ((size_t)(b * p.Hkv + hkv) * p.Tc) * D;
        const uint8_t* RSg = p.KreprS + ((size_t)(b * p.Hkv + hkv) * p.Tc) * 4;
        const MaxTiles mt = max_tiles(p.use_minit, p.n_sink, p.n_local, a_lo, a_hi, nv);
        auto stage = [&](int u) __attribute__((always_inline)) { return smem + STAGE + u * Tile8::KBYTES; };
        float mx = -INFINITY;
        for (int t0 = 0; t0 < mt.total; t0 += 4) {
            if (t0) __syncthreads();
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u;
                if (t < mt.n_sum) {
                    load_tile8(Rg, t * BN, nv, stage(u), wave, lane);
                    if (wave == 0) load_scales64(RSg, t * BN, nv, mscale[u], lane);
                } else if (t < mt.total) {
                    load_tile4(Kg, mt.block(t) * BN, N, stage(u), wave, lane);
                    if (wave == 0) load_scales64(Ksg, mt.block(t) * BN, N, mscale[u], lane);
                }
            }
            if (t0 == 0) {
                load_kv(0, 0, 0);
                __builtin_amdgcn_s_waitcnt(0x0F74);  // the staged tiles have landed, not yet those of the main loop
            } else {
                __builtin_amdgcn_s_waitcnt(0x0F70);
            }
            __syncthreads();
#pragma unroll 1
            for (int t = t0; t < min(t0 + 4, mt.total); ++t) {
                const uint8_t* const tile = stage(t - t0);
                const uint32_t* const sc = mscale[t - t0];
                f32x16 st[2];
                if (t < mt.n_sum) {
#pragma unroll
                    for (int h2 = 0; h2 < 2; ++h2) {
                        const int row = 32 * h2 + ql;
#pragma unroll
                        for (int kh = 0; kh < 2; ++kh) {
                            // 8-bit operand: bytes 0..15 of half hh are k = 16 hh + j, bytes 16..31 are k = 32 + 16 hh + j
                            const int c0 = 4 * kh + hh;
                            const i32x8 f = lds_frag8(tile + Tile8::k_off(row, c0), tile + Tile8::k_off(row, c0 + 2));
                            st[h2] = mfma_bf8_f4(f, qf[kh], kh ? st[h2] : f32x16{0}, spread_byte(sc[row], 2 * kh + hh), qs[kh]);
                        }
                    }
                } else {
                    qk_tile4(tile, sc, qf, qs, st, ql, hh);
                }
                const int j = mt.block(t);
                if (t < mt.n_sum || (j * BN + BN <= N && !(p.causal && j * BN + BN - 1 > row0))) mx = fmaxf(mx, tile_rowmax<false>(st, 0, 0, hh));
                else mx = fmaxf(mx, tile_rowmax<true>(st, j * BN, limit, hh));
            }
        }
        m2 = finite_max(xhalf_max(mx) * p.c);
    } else {
        load_kv(0, 0, 0);
    }
    wait_vm0_and_sync();
    load_kv(1, STAGE, 1);
    f32x16 ot[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) ot[db] = f32x16{0};
    float lsum = 0.f;
    f32x16 start;  // FOLD: -(m + H) of this lane's query in all 16 registers, set once the max is frozen
    f32x16 lt = {0};   // NOEXP: 32 copies of this lane's row sum of the rounded weights (times 2^15)
    float code0 = 0.f;  // NOEXP: code offset - 4 (m + H)
    if (FOLD) {
        const float v = -(m2 + p.headroom);
        if (NOEXP) code0 = kCodeUnit * (kCodeOffset + kCodeHalf + kCodesPerBinade * v);
#pragma unroll
        for (int r = 0; r < 16; ++r) start[r] = v;
    }
    // fragment addresses in a stage: see attn_fp8_kernel
    uint32_t ka[2], va[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        ka[e] = lds_address(smem) + Tile4::k_off(ql, 2 * e + hh);
        va[e] = lds_address(smem) + Tile4::KBYTES + Tile8::v_off(ql, 2 * hh + e);
    }
    const uint32_t sa = lds_s + 4 * ql;
    typedef const __attribute__((address_space(3))) u32x4* lds_ptr;
    typedef const __attribute__((address_space(3))) uint32_t* lds_dword;
    auto visit = [&](int j, uint32_t stage, uint32_t st_no, uint32_t next2, uint32_t next2_no, auto masked_c) __attribute__((always_inline)) {
        constexpr bool SPECIAL = is_fa(MODE), MASKED = decltype(masked_c)::value;
        f32x16 st[2];
        uint32_t pk[8];
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t sc = *(lds_dword)(sa + st_no * 256 + t * 128);
            const u32x4 g0 = *(lds_ptr)(ka[0] + stage + t * 2048), g1 = *(lds_ptr)(ka[1] + stage + t * 2048);
            st[t] = mfma_f4(g0, qf[0], FOLD && !NOEXP ? start : f32x16{0}, spread_byte(sc, hh), qs[0]);
            st[t] = mfma_f4(g1, qf[1], st[t], spread_byte(sc, 2 + hh), qs[1]);
        }
        __builtin_amdgcn_s_setprio(0);
        load_kv(j + 2, next2, next2_no);
        const bool needs_mask = (p.causal && j * BN + BN - 1 > row0) || (j + 1) * BN > N;
        if (NOEXP) codes_tile8<MASKED>(st, pk, j * BN, needs_mask ? limit : 0x3fffffff, hh, code0);
        else if (FOLD) softmax_tile8_folded<MASKED, P_BF8>(st, pk, lsum, j * BN, needs_mask ? limit : 0x3fffffff, hh);
        else softmax_tile8<SPECIAL, MASKED, P_BF8>(st, pk, ot, m2, lsum, p.c, p.headroom, j * BN, needs_mask ? limit : 0x3fffffff, hh);
        const i32x8 pf = {(int)pk[0], (int)pk[1], (int)pk[2], (int)pk[3], (int)pk[4], (int)pk[5], (int)pk[6], (int)pk[7]};
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const u32x4 lo = *(lds_ptr)(va[0] + stage + db * 2048), hi = *(lds_ptr)(va[1] + stage + db * 2048);
            const i32x8 g = {(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
            ot[db] = P_BF8 ? __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(g, pf, ot[db], 0, 1, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f) : mfma_f8(g, pf, ot[db]);
        }
        if (NOEXP) {  // row sums of the rounded weights: a block of E2M1 ones times P (E5M2)
            const i32x8 ones = {0x22222222, 0x22222222, 0x22222222, 0x22222222, 0, 0, 0, 0};
            lt = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ones, pf, lt, 4, 1, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f);
        }
        __builtin_amdgcn_s_setprio(0);
        // tile j + 1 has landed
        __builtin_amdgcn_s_waitcnt(0x0F74);
        __syncthreads();
    };
    using std::false_type;
    using std::true_type;
    int j_masked = p.causal ? a_lo : p.Tc;  // first tile that needs masking
    if (N % BN) j_masked = min(j_masked, p.Tc - 1);
    int j = 0;
    for (; j + S <= min(j_masked, nv); j += S) {
        visit(j, 0, 0, 2 * STAGE, 2, false_type{});
        visit(j + 1, STAGE, 1, 0, 0, false_type{});
        visit(j + 2, 2 * STAGE, 2, STAGE, 1, false_type{});
    }
#pragma unroll 1
    for (uint32_t no = 0; j < nv; ++j) {
        const uint32_t next = no == 2 ? 0 : no + 1, next2 = next == 2 ? 0 : next + 1;
        visit(j, no * STAGE, no, next2 * STAGE, next2, true_type{});
        no = next;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // (requests past the last tile write zeros to LDS: not behind this workgroup's end)
    // (NOEXP: every register of lt holds the whole row sum, with the same 2^15 as the numerator)
    const float l = NOEXP ? lt[0] * 0x1p-15f : xhalf_sum(lsum);
    const float inv = l > 0.f ? p.descale_v * (P_BF8 ? 0x1p-15f : 0x1p-8f) / l : 0.f;
    const size_t row = (size_t)(b * p.Hq + h) * N + qrow;
    store_row8(p.O + row * D, qrow < N, ot, inv, hh);
    if (qrow < N && p.LSE && hh == 0)
        p.LSE[row] = l > 0.f ? (m2 + p.headroom + __builtin_amdgcn_logf(l)) * kLn2 : -INFINITY;
}

}  // namespace
