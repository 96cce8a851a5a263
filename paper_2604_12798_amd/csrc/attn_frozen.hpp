// Alg. 1 with the max fixed before the first softmax: bf16, one 128-row query block per workgroup, the keys split over KS
// groups of four waves.  d = 64 but for short sequences (attn_short.hpp); d = 128 where the ping-pong kernel
// (attn_pingpong.hpp), which works in items of 256 rows, would leave compute units idle, and the rest rows of its calls without a mask.
#pragma once
#include "common.hpp"

namespace {

// ---------------------------------------------------------------------------------------------
// Alg. 1's max is final once the sink and local blocks have been seen, and nothing but their scores goes into it.  So their
// row maxima are taken first, together with q . summary (the same tile product), and every block, sink and local ones
// included, is then a frozen one: no row max, no rescale, no order, and the groups that share the keys add their sums in the
// end without weights.  The price is one more Q.K^T for the sink and local blocks (three of them by default).
//
// Step k of a wave: Q.K^T of its tile k + 1 and P.V of its tile k - 1 with the softmax of tile k dealt out between the MFMAs.
// Two score buffers and two sets of packed P; the fast loop is unrolled by two so that they swap without moves.
// What bounds it: at d = 64 the vector unit (measured in a loop of nothing else: a slice of two scores takes it 35 cycles and an
// MFMA 10 of its issue, so 740 cycles per wave and tile against 512 of MFMA; the kernel takes about 900 with three waves on a SIMD, which
// fit with a ring of four fragments, each loaded again behind the MFMA that used it, and two tiles of K and V: 4 x 16
// heads, N = 4096 165 us with two waves and rings of four tiles, 160 with two, 157 with three), at d = 128 the matrix unit (1024 cycles per wave and tile; 1500 with two waves on a
// SIMD).  Outside the steps a workgroup spends 14 - 17 K cycles: 2 K to its first request, 6 K until the first tiles are there,
// 3.5 K on the max, 3 K on the groups' exchange and the output.
// Kernel times in us, before and after: 32 heads over 8, causal, d = 128: N = 256 15.7 / 12.0, 777 25.0 / 18.9, 1024 29.0 / 21.5
// (the ping-pong kernel's items leave more than half of the compute units idle); 16 heads, not causal, N = 5000 234 / 216;
// d = 64 against the generic kernel: 32 heads over 8, causal, N = 777 16.5 / 12.4, 2048 37 / 30; 4 x 16 heads, N = 4096 179 / 157.
// Each group has rings of S K tiles and S V tiles, filled by LDS-direct loads up to S - 1 steps ahead; one barrier per step.
// With two groups the waves of the first request the K tiles of both and those of the second the V tiles (adjacent tiles, one
// address to work out per step).
template <int D, int KS>
struct Frozen {
    static constexpr bool TIGHT = D == 64 && KS == 1;          // three workgroups to a compute unit: only the first K tile is requested in front of the max
    static constexpr int S = D == 64 && !TIGHT ? 4 : 2;
    static constexpr int RING = 2 * S * Tile<D>::BYTES;        // one group's
    static constexpr int EXTRA = TIGHT ? 1 : 4 - 2 * KS;       // staging slots beside those that a group's prologue leaves free (two of V; TIGHT: one of K, two of V)
    static constexpr int LDS_BYTES = KS * RING + EXTRA * Tile<D>::BYTES + (KS == 2 ? 1024 : 0);  // (and the exchange of the max)
};

// ROWS64: the call is causal and in blocks of 64 rows, and a block of 128 stands for two of them.
template <int D, int KS, bool ROWS64>
__global__ __launch_bounds__(256 * KS, (Frozen<D, KS>::TIGHT ? 3 : 2)) void attn_fwd_frozen_kernel(const Params p) {
    using T = Tile<D>;
    using F = Frozen<D, KS>;
    constexpr int BM = 128, KK = D / 16, DB = D / 32, S = F::S;
    constexpr int NG = D / 32;           // groups of four MFMAs of one product
    constexpr int LI = T::BYTES / 4096;  // load instructions per wave and tile
    extern __shared__ __attribute__((aligned(16))) uint8_t frozen_smem[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = KS == 1 ? 0 : wave >> 2, w4 = wave & 3;
    const int ql = lane & 31;
    const int hh = lane >> 5;
    uint8_t* const Ks = frozen_smem + grp * F::RING;
    uint8_t* const Vs = Ks + S * T::BYTES;

    // items: late (long) query blocks first; the KV heads congruent mod 8 on one XCD, as in the other kernels
    const int g = p.Hq / p.Hkv;
    int b, h, i;
    {
        const int id = blockIdx.x, G = p.B * p.Hkv;
        if ((G & 7) == 0) {
            const int x = id & 7, y = id >> 3, per = p.Tr * g;
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
    b = __builtin_amdgcn_readfirstlane(b);  // (the divisions run on the vector unit: back to scalar registers)
    h = __builtin_amdgcn_readfirstlane(h);
    i = __builtin_amdgcn_readfirstlane(i);
    const int hkv = __builtin_amdgcn_readfirstlane(h / g);
    const int N = p.N;
    const int row0 = p.row_base + i * BM;
    const int last_row = min(N, row0 + BM) - 1;
    const int a_lo = row0 / BN, a_hi = last_row / BN;
    const int j_hi = p.causal ? a_hi : p.Tc - 1;
    const int nv = j_hi + 1;

    const uint16_t* Qg = p.Q + ((size_t)(b * p.Hq + h) * N) * D;
    const uint16_t* Kg = p.K + ((size_t)(b * p.Hkv + hkv) * N) * D;
    const uint16_t* Vg = p.V + ((size_t)(b * p.Hkv + hkv) * N) * D;
    const uint16_t* Rg = p.Krepr + ((size_t)(b * p.Hkv + hkv) * p.Tc) * D;

    const int qrow = row0 + 32 * w4 + ql;
    const int qrow_c = min(qrow, N - 1);
    const int limit = p.causal ? qrow_c : N - 1;
    // Last key block that may reach this wave's rows: with ROWS64 the diagonal one of its own 64.  The summary
    // of the next one may lie far above every score that the rows see (all their exponentials would be 0), and a weight of 0 times
    // a NaN among its values is not 0.
    const int own_hi = ROWS64 ? min(j_hi, a_lo + (w4 >> 1)) : j_hi;
    bf16x8 qf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
        qf[kk] = *reinterpret_cast<const bf16x8*>(Qg + (size_t)qrow_c * D + 16 * kk + 8 * hh);

    // ---- tile requests: a wave moves LI adjacent pieces of a tile (a piece = 1 KiB of whole rows).  Buffer loads with the tile
    // as the buffer: rows past the end of the sequence are out of its range (LDS gets zeros), and a request past the last tile
    // has an empty buffer, so every step issues the same instructions without a branch.  The instruction offset moves both the
    // global and the LDS side, so M0 (the LDS base of such a load) is set once per tile.
    constexpr int RPI = 1024 / T::ROWB;
    const int cp = lane % T::CH;
    uint32_t offK[LI], off[LI];
    const bool role_v = KS == 2 && grp == 1;
#pragma unroll
    for (int u = 0; u < LI; ++u) {
        const int r0 = RPI * LI * w4 + lane / T::CH, r = r0 + RPI * u;  // (row of the first piece; of this one)
        offK[u] = (uint32_t)(r0 * T::ROWB + ((cp ^ T::k_mix(r)) << 4));
        off[u] = role_v ? (uint32_t)(r0 * T::ROWB + ((cp ^ T::v_mix(r)) << 4)) : offK[u];
    }
    const uint32_t offV = (uint32_t)((RPI * LI * w4 + lane / T::CH) * T::ROWB +
                                     ((cp ^ T::v_mix(RPI * LI * w4 + lane / T::CH)) << 4));  // (KS = 1: the same for all pieces)
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)(frozen_smem + w4 * LI * 1024));
    // `rows` rows (0 to BN, a negative number counts as 0) at address a to LDS byte `at`
    auto request = [&](uint64_t a, int rows, const uint32_t o0, const uint32_t o1, const uint32_t o2, const uint32_t o3, uint32_t at)
                       __attribute__((always_inline)) {
        const uint32_t bytes = min(max(rows, 0), BN) * T::ROWB;
        if (LI == 4) request4(a, bytes, o0, o1, o2, o3, lds0 + at);
        else request2(a, bytes, o0, o1, lds0 + at);
    };
    auto tile_addr = [&](const uint16_t* base, int j) __attribute__((always_inline)) {
        return (uint64_t)(uintptr_t)base + (uint64_t)(uint32_t)j * (BN * T::ROWB);
    };
    // what step k requests: K of step k + S - 1's Q.K^T (tiles KS (k + S) ..) and V of step k + S - 1's P.V (tiles KS (k + S - 2) ..)
    const uint16_t* const role_base = role_v ? Vg : Kg;
    const int role_dk = role_v ? S - 2 : S;
    auto request_step = [&](int k) __attribute__((always_inline)) {
        if (KS == 2) {
            const int kk = k + role_dk, j = 2 * kk;
            const int rows = j < nv ? N - j * BN : 0;
            const uint64_t a = tile_addr(role_base, j);
            const uint32_t at = ((role_v ? S : 0) + kk % S) * T::BYTES;
            request(a, rows, off[0], off[1], off[LI - 2], off[LI - 1], at);
            request(a + BN * T::ROWB, rows - BN, off[0], off[1], off[LI - 2], off[LI - 1], at + F::RING);
        } else {
            const int jk = k + S, jv = k + S - 2;
            request(tile_addr(Kg, jk), jk < nv ? N - jk * BN : 0, off[0], off[1], off[LI - 2], off[LI - 1], (jk % S) * T::BYTES);
            request(tile_addr(Vg, jv), jv < nv ? N - jv * BN : 0, offV, offV, offV, offV, (S + jv % S) * T::BYTES);
        }
    };

    // ---- the max: tiles of 64 summaries that cover the visible blocks, then the sink and the local tiles of K, four at a time,
    // dealt out to the groups; the first tiles of the main loop are requested behind the first four
    const int n_sum = p.use_minit ? (nv + BN - 1) / BN : 0;
    const int n1 = min(p.n_sink, nv);
    const int lo2 = p.n_local > 0 ? max(max(0, a_lo - (p.n_local - 1)), n1) : nv, n2 = max(0, min(a_hi, j_hi) + 1 - lo2);
    const int n_max = n_sum + n1 + (p.n_local > 0 ? n2 : 0);
    auto stage = [&](int u) __attribute__((always_inline)) {  // LDS offset of staging slot u
        if (F::TIGHT) return (uint32_t)((1 + u) * T::BYTES);
        return (uint32_t)(u < 2 * KS ? (u % KS) * F::RING + (2 * S - 1 - u / KS) * T::BYTES : KS * F::RING + (u - 2 * KS) * T::BYTES);
    };
    f32x16 sa[2], sb[2];
    float mx = -INFINITY;
    for (int t0 = 0; t0 < n_max; t0 += 4) {
        if (t0) __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = t0 + u;
            if (u % KS == grp && t < n_max) {
                if (t < n_sum) {  // (rows clamped to the visible blocks: a repeated row changes no max)
                    load_tile<D, 4>(Rg, t * BN, nv, frozen_smem + stage(u), false, w4, lane);
                } else {
                    const int j = t - n_sum < n1 ? t - n_sum : lo2 + (t - n_sum - n1);
                    request(tile_addr(Kg, j), N - j * BN, offK[0], offK[1], offK[LI - 2], offK[LI - 1], stage(u));
                }
            }
        }
        if (t0 == 0) {  // the main loop's first tiles; the max phase does not wait for them
            if (KS == 2) {
                if (role_v) {
#pragma unroll
                    for (int k = -(S - 2); k < 0; ++k) request_step(k);
                    constexpr int out = 2 * (S - 2) * LI;
                    __builtin_amdgcn_s_waitcnt((out < 16 ? 0x0F70 : 0x4F70) | (out & 15));
                } else {
#pragma unroll
                    for (int k = -S; k < 0; ++k) request_step(k);
                    constexpr int out = 2 * S * LI;
                    __builtin_amdgcn_s_waitcnt(0x0F70 | (out & 15) | ((out >> 4) << 14));
                }
            } else {
#pragma unroll
                for (int k = 0; k < (F::TIGHT ? 1 : S); ++k) request(tile_addr(Kg, k), k < nv ? N - k * BN : 0, off[0], off[1], off[LI - 2], off[LI - 1], k * T::BYTES);
#pragma unroll
                for (int k = 0; k < S - 2; ++k) request(tile_addr(Vg, k), k < nv ? N - k * BN : 0, offV, offV, offV, offV, (S + k) * T::BYTES);
                constexpr int out = (F::TIGHT ? 1 : 2 * S - 2) * LI;
                __builtin_amdgcn_s_waitcnt(0x0F70 | (out & 15) | ((out >> 4) << 14));
            }
        } else {
            __builtin_amdgcn_s_waitcnt(0x0F70);
        }
        __syncthreads();
#pragma unroll 1
        for (int u = grp; u < 4; u += KS) {
            const int t = t0 + u;
            if (t >= n_max) break;
            qk_tile_pipe<D>(frozen_smem + stage(u), qf, sa, ql, hh);
            const int j = t - n_sum < n1 ? t - n_sum : lo2 + (t - n_sum - n1);
            if (t < n_sum ? (!ROWS64 || own_hi == j_hi) : (j * BN + BN <= N && !(p.causal && j * BN + BN - 1 > row0))) mx = fmaxf(mx, tile_rowmax<false>(sa, 0, 0, hh));
            else if (ROWS64) mx = fmaxf(mx, tile_rowmax<true>(sa, (t < n_sum ? t : j) * BN, t < n_sum ? own_hi : limit, hh));
            else mx = fmaxf(mx, tile_rowmax<true>(sa, j * BN, limit, hh));
        }
    }
    mx = xhalf_max(mx);
    float* const xm = reinterpret_cast<float*>(frozen_smem + KS * F::RING + F::EXTRA * T::BYTES);
    if (KS == 2 && hh == 0) xm[grp * BM + 32 * w4 + ql] = mx;
    wait_vm0_and_sync();
    if (KS == 2) mx = fmaxf(mx, xm[(grp ^ 1) * BM + 32 * w4 + ql]);
    const float m2 = finite_max(mx * p.c);
    // step 0 finds "V of tile -1" all zeros (an empty buffer; what the slot held, times zero weights, could be NaN)
    request(0, 0, off[0], off[1], off[LI - 2], off[LI - 1], grp * F::RING + (2 * S - 1) * T::BYTES);
    if (F::TIGHT) {
#pragma unroll
        for (int k = 1; k < S; ++k) request(tile_addr(Kg, k), k < nv ? N - k * BN : 0, off[0], off[1], off[LI - 2], off[LI - 1], k * T::BYTES);
    }
    qk_tile_pipe<D>(Ks, qf, sa, ql, hh);
    wait_vm0_and_sync();  // (also: step 0 requests into K slot 0)

    f32x16 ot[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) ot[db] = f32x16{0};
    float lsum = 0.f;
    uint32_t pa[16], pb[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) pa[e] = pb[e] = 0;

    const int kbase = T::k_base(ql, hh), vbase = T::v_base(lane, hh);
    auto mf_v = [&](const bf16x8* f, const uint32_t* pk, int gq, int e) __attribute__((always_inline)) {
        const int c = (4 * gq + e) / DB, db = (4 * gq + e) % DB;
        const u32x4 pw = {pk[4 * c], pk[4 * c + 1], pk[4 * c + 2], pk[4 * c + 3]};
        ot[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[e], __builtin_bit_cast(bf16x8, pw), ot[db], 0, 0, 0);
    };
    auto mf_k = [&](const bf16x8* f, f32x16* st, int gq, int e) __attribute__((always_inline)) {
        st[e & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[e], qf[2 * gq + (e >> 1)], gq == 0 && e < 2 ? f32x16{0} : st[e & 1], 0, 0, 0);
    };
    auto mask = [&](int k, f32x16* st) __attribute__((always_inline)) {
        const int j = KS * k + grp;
        const int rel = (j < nv ? limit : -1) - j * BN - 4 * hh;  // (a tile past the last one, where the groups' shares differ)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) st[t][r] = (32 * t + 8 * (r >> 2) + (r & 3) <= rel) ? st[t][r] : -INFINITY;
    };
    // two scores: seven instructions
    auto slice = [&](int q, const f32x16* st, uint32_t* pk) __attribute__((always_inline)) {
        const int t = q >> 3, r = 2 * (q & 7);
        const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[t][r], p.c, -m2));
        const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[t][r + 1], p.c, -m2));
        lsum += e0;
        lsum += e1;
        pk[q] = pack_bf16(e0, e1);
    };
    // step k: scores of tile k in s0, P of tile k - 1 in p1; leaves scores of tile k + 1 in s1 and P of tile k in p0.
    // LAST: the last tile, no next one to multiply.
    auto step = [&](int k, f32x16* s0, f32x16* s1, uint32_t* p0, const uint32_t* p1, auto masked_c, auto last_c) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_c)::value, LAST = decltype(last_c)::value;
        const uint8_t* kt = Ks + ((k + 1) % S) * T::BYTES;
        const uint8_t* vt = Vs + ((k + S - 1) % S) * T::BYTES;
        constexpr int G0 = LAST ? NG : 0;           // groups of MFMAs: [0, NG) are Q.K^T, [NG, 2 NG) P.V
        constexpr int NM = 4 * (2 * NG - G0);
        constexpr int LEAD = 2;  // slices in front of the first MFMA, while its fragments are on their way
        if (LAST && S == 2) request_step(k);  // (its own V, which a deeper ring has asked for by now)
        if (MASKED) mask(k, s0);
        bf16x8 f[4];
        auto ld1 = [&](int x) __attribute__((always_inline)) {  // fragment x of the step: those of Q.K^T, then those of P.V
            const int gq = x >> 2, e = x & 3;
            if (gq < NG) return *reinterpret_cast<const bf16x8*>(kt + (kbase ^ ((2 * gq + (e >> 1)) << 5)) + (e & 1) * 32 * T::ROWB);
            const int c = (4 * (gq - NG) + e) / DB, db = (4 * (gq - NG) + e) % DB;
            const uint8_t* a = vt + (vbase ^ (db << 6)) + 16 * c * T::ROWB;
            const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a));
            const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a + 8 * T::ROWB));
            const u32x2 a0 = __builtin_bit_cast(u32x2, v0), a1 = __builtin_bit_cast(u32x2, v1);
            const u32x4 aw = {a0[0], a0[1], a1[0], a1[1]};
            return __builtin_bit_cast(bf16x8, aw);
        };
#pragma unroll
        for (int x = 4 * G0; x < 4 * G0 + 4; ++x) f[x & 3] = ld1(x);
        __builtin_amdgcn_sched_barrier(0);
        int q = 0;
#pragma unroll
        for (; q < LEAD; ++q) slice(q, s0, p0);
#pragma unroll
        for (int gq = G0; gq < 2 * NG; ++gq) {
            if (!LAST && gq == 1) request_step(k);  // (here and not in front, so that the MFMAs start right behind the barrier)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (gq < NG) mf_k(f, s1, gq, e);
                else mf_v(f, p1, gq - NG, e);
                if (4 * gq + e + 4 < 8 * NG) f[e] = ld1(4 * gq + e + 4);
#pragma unroll
                for (; q < 16 && (q - LEAD) * NM < (4 * (gq - G0) + e + 1) * (16 - LEAD); ++q) slice(q, s0, p0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // K(k + 2) and V(k), requested S - 2 steps ago, have to have landed
        constexpr int out = LAST ? 0 : 2 * (S - 2) * LI;
        __builtin_amdgcn_s_waitcnt(0x0F70 | (out & 15) | ((out >> 4) << 14));
        __builtin_amdgcn_s_barrier();
    };
    using std::false_type;
    using std::true_type;
    const int n_steps = (nv + KS - 1) / KS;
    int j_masked = min(p.causal ? a_lo : p.Tc, nv);  // first tile that needs masking
    if (N % BN) j_masked = min(j_masked, p.Tc - 1);
    const int k_fast = j_masked / KS;                // steps below it are unmasked for every group
    int k = 0;
    for (; k + 2 <= min(k_fast, n_steps - 1); k += 2) {
        step(k, sa, sb, pb, pa, false_type{}, false_type{});
        step(k + 1, sb, sa, pa, pb, false_type{}, false_type{});
    }
#pragma unroll 1
    for (; k < n_steps - 1; ++k) {  // (an odd one out, and where more than the last step needs masks)
        step(k, sa, sb, pb, pa, true_type{}, false_type{});
#pragma unroll
        for (int t = 0; t < 2; ++t) sa[t] = sb[t];
#pragma unroll
        for (int e = 0; e < 16; ++e) pa[e] = pb[e];
    }
    step(k, sa, sb, pb, pa, true_type{}, true_type{});
    if (!ROWS64 || KS * k + grp <= own_hi) pv_tile_pipe<D>(Vs + (k % S) * T::BYTES, pb, ot, lane, hh);  // (the next 64's block is the last tile)

    if (KS == 1) {
        store_output<D, 0, DB>(p, ot, m2, lsum, b, h, qrow, hh);
    } else {
        // the groups trade halves of O^T through LDS and add; each stores its half of the columns
        wait_vm0_and_sync();  // (requests past the last tile may still be writing zeros to the rings)
        constexpr int H = DB / 2;
        float* const ex = reinterpret_cast<float*>(frozen_smem) + (size_t)w4 * (H * 16 + 1) * 64 + lane;
        constexpr int GS = 4 * (H * 16 + 1) * 64;
        auto put = [&](auto own_c) __attribute__((always_inline)) {
            constexpr int G = decltype(own_c)::value;  // this group keeps d blocks [G H, G H + H)
            float* const to = ex + (G ^ 1) * GS;       // the other group's mailbox
#pragma unroll
            for (int db = 0; db < H; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) to[(db * 16 + r) * 64] = ot[(G ^ 1) * H + db][r];
            to[H * 16 * 64] = lsum;
            __syncthreads();
            const float* const from = ex + G * GS;
#pragma unroll
            for (int db = 0; db < H; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) ot[G * H + db][r] += from[(db * 16 + r) * 64];
            lsum += from[H * 16 * 64];
            store_output<D, G * H, H>(p, ot, m2, lsum, b, h, qrow, hh);
        };
        if (grp == 0) put(std::integral_constant<int, 0>{});
        else put(std::integral_constant<int, 1>{});
    }
}

}  // namespace
