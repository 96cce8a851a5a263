// Alg. 2 (skipping) at d = 128, blocks of 128 rows: bf16, one query block per workgroup of four waves, two workgroups per compute unit.
#pragma once
#include "common.hpp"

namespace {

// ---------------------------------------------------------------------------------------------
// Alg. 2's max is final once the sink and local blocks have been seen, and what they decide depends on nothing but their row maxima and
// the max so far.  So their scores are taken first, together with q . summary; every wave then walks them in Alg. 2's order for all 128
// rows by itself (the row maxima meet in LDS; no vote between waves), which fixes the max and those blocks' fates.  All other blocks are
// independent of each other, and the main loop takes all blocks in ascending order: no rescaling, one barrier a step.
//
// Step k of a wave: P.V of tile k - 1, if that one was kept; Q.K^T of tile k + 1 with the softmax of tile k dealt out between the MFMAs, if
// that tile is kept; and its vote on tile k + 1, which the other waves read behind the step's barrier.  A dropped tile costs its Q.K^T and
// its row max, and its V is not requested.
//
// Bound by the matrix pipe where tiles are kept (32 MFMAs a tile and wave; 63 % busy at N = 65536, 60 % dropped), by the serial end of a step
// where they are dropped (row max, vote, barrier, requests: with eight waves behind one barrier 1500 of a step's 3400 cycles).  So a workgroup is four waves, and the two of a compute unit
// drift apart and fill each other's ends; eight waves behind one barrier, the keys split in two, took 378 us where this takes 338
// (32/8 heads, N = 8000, 71 % dropped) and gained on it only below one item per compute unit.  Priority while a wave issues MFMAs: 2 %
// (921 to 902 us, the same heads, non-causal); requests in front of P.V instead of behind it: 1 % slower.
// us on the other kernels / here, 32/8 heads, causal: N = 2048 59 / 51 (59 % dropped) and 67 / 58 (3 %), 4096 134 / 116 and 177 / 152, 8000
// 411 / 347 and 555 / 502; 8 heads: 16384 438 / 354 and 569 / 516, 65536 5135 / 4387 (88 %) and 7819 / 7470 (25 %).
struct Sparse {
    static constexpr int S = 2;                  // K tiles and V tiles in LDS
    static constexpr int RING = 2 * S * Tile<128>::BYTES;
    static constexpr int MAX_LEAD = 9;           // sink and local blocks: up to four and four, and one more that a block of 128 rows covers
    static constexpr int LDS_BYTES = RING + (1 + MAX_LEAD) * 512 + 64;
};

__global__ __launch_bounds__(256, 2) void attn_sparse_kernel(const Params p) {
    constexpr int D = 128, BM = 128, KK = D / 16, DB = D / 32, S = Sparse::S;
    using T = Tile<D>;
    extern __shared__ __attribute__((aligned(16))) uint8_t sparse_smem[];
    float* const minit = reinterpret_cast<float*>(sparse_smem + Sparse::RING);  // [row] largest q . summary
    float* const lead_max = minit + BM;                                         // [sink or local block][row] its row max, log2 units
    uint8_t* const votes = reinterpret_cast<uint8_t*>(lead_max + Sparse::MAX_LEAD * BM);  // [parity of the step][wave]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ql = lane & 31;
    const int hh = lane >> 5;
    uint8_t* const Ks = sparse_smem;
    uint8_t* const Vs = Ks + S * T::BYTES;

    const auto [head, kv, i] = item_of(p, blockIdx.x);
    const int N = p.N;
    const int row0 = i * BM;
    const int last_row = min(N, row0 + BM) - 1;
    const int a_lo = row0 / BN, a_hi = last_row / BN;
    const int j_hi = p.causal ? a_hi : p.Tc - 1;
    const int nv = j_hi + 1;

    const uint16_t* Qg = p.Q + ((size_t)head * N) * D;
    const uint16_t* Kg = p.K + ((size_t)kv * N) * D;
    const uint16_t* Vg = p.V + ((size_t)kv * N) * D;
    const uint16_t* Rg = p.Krepr + ((size_t)kv * p.Tc) * D;

    const int qrow = row0 + 32 * wave + ql;
    const int qrow_c = min(qrow, N - 1);
    const int limit = p.causal ? qrow_c : N - 1;
    bf16x8 qf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(Qg + (size_t)qrow_c * D + 16 * kk + 8 * hh);

    // ---- requests, as in attn_frozen.hpp: a wave moves four adjacent pieces of a tile
    const int cp = lane % T::CH, pr0 = 16 * wave + lane / T::CH;  // (the row of its first piece)
    const uint32_t offK = (uint32_t)(pr0 * T::ROWB + ((cp ^ T::k_mix(pr0)) << 4));  // (four rows on: ^ 64)
    const uint32_t offV = (uint32_t)(pr0 * T::ROWB + ((cp ^ T::v_mix(pr0)) << 4));  // (the same for rows four apart)
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(sparse_smem) + wave * 4096);
    const uint32_t range = (uint32_t)min(N, nv * BN) * T::ROWB;
    const u32x4 rsrcK = tile_buffer((uint64_t)(uintptr_t)Kg, range), rsrcV = tile_buffer((uint64_t)(uintptr_t)Vg, range);
    // tile j (past the last visible one: zeros) to a slot
    auto request_k = [&](int j, int slot) __attribute__((always_inline)) {
        uint32_t o = offK;
        asm volatile("" : "+v"(o));  // (three instructions here, not three registers all along)
        request4_at(rsrcK, (uint32_t)j * T::BYTES, o, o ^ 64, o ^ 128, o ^ 192, lds0 + slot * T::BYTES);
    };
    auto request_v = [&](int j, int slot) __attribute__((always_inline)) {
        request4_at(rsrcV, (uint32_t)j * T::BYTES, offV, offV, offV, offV, lds0 + slot * T::BYTES);
    };

    // ---- q . summary and the sink and local blocks' row maxima: two tiles at a time, staged in the V slots
    const int n_sum = p.use_minit ? (nv + BN - 1) / BN : 0;
    const int n1 = min(p.n_sink, nv);
    const int lo2 = p.n_local > 0 ? max(max(0, a_lo - (p.n_local - 1)), n1) : nv, n2 = p.n_local > 0 ? max(0, min(a_hi, j_hi) + 1 - lo2) : 0;
    const int n_lead = n1 + n2, n0 = min(n1, 1), n_max = n_sum + n_lead - n0;  // (the scores of tile 0 are step 0's)
    auto lead_block = [&](int l) __attribute__((always_inline)) { return l < n1 ? l : lo2 + (l - n1); };
    auto mask = [&](int k, f32x16* st) __attribute__((always_inline)) {
        const int rel = limit - k * BN - 4 * hh;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) st[t][r] = (32 * t + 8 * (r >> 2) + (r & 3) <= rel) ? st[t][r] : -INFINITY;
    };
    auto lead_row_max = [&](int l, float r) __attribute__((always_inline)) {
        r = xhalf_max(r) * p.c;
        if (hh == 0) lead_max[l * BM + 32 * wave + ql] = r;
    };
    f32x16 sa[2], sb[2];
    float mx = -INFINITY, r0 = -INFINITY;
    request_k(0, 0);
    for (int t0 = 0; t0 == 0 || t0 < n_max; t0 += 2) {
        if (t0) __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int t = t0 + u;
            if (t < n_sum) load_tile<D, 4>(Rg, t * BN, nv, Vs + u * T::BYTES, false, wave, lane);  // (rows clamped to the visible blocks)
            else if (t < n_max) request_k(lead_block(n0 + t - n_sum), S + u);
        }
        wait_vm0_and_sync();
        if (t0 == 0) {
            request_k(1, 1);
            qk_tile_pipe<D>(Ks, qf, sa, ql, hh);
            mask(0, sa);
            r0 = tile_rowmax<false>(sa, 0, 0, hh);
            if (n0) lead_row_max(0, r0);
        }
#pragma unroll 1
        for (int u = 0; u < 2; ++u) {
            const int t = t0 + u;
            if (t >= n_max) break;
            qk_tile_pipe<D>(Vs + u * T::BYTES, qf, sb, ql, hh);
            if (t < n_sum) {
                mx = fmaxf(mx, tile_rowmax<false>(sb, 0, 0, hh));
            } else {
                const int l = n0 + t - n_sum;
                lead_row_max(l, tile_rowmax<true>(sb, lead_block(l) * BN, limit, hh));
            }
        }
    }
    mx = xhalf_max(mx);
    if (hh == 0) minit[32 * wave + ql] = mx;
    wait_vm0_and_sync();
    // ---- the sink and local blocks in order: kept where a row keeps them, and then part of the max.  A lane walks two of the 128 rows for the
    // decisions, which all waves take alike, and its own for its max
    float m2;
    uint32_t lead_kept = 0;
    {
        float m[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) m[e] = p.use_minit ? minit[lane + 64 * e] * p.c : -INFINITY;
        m2 = p.use_minit ? minit[32 * wave + ql] * p.c : -INFINITY;
        for (int l = 0; l < n_lead; ++l) {
            const float own = lead_max[l * BM + 32 * wave + ql];
            float mt[2];
            bool keeps = false;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                mt[e] = lead_max[l * BM + lane + 64 * e];
                keeps |= row0 + lane + 64 * e < N && mt[e] != -INFINITY && !(mt[e] < m[e] - p.thr2);
            }
            if (__builtin_amdgcn_ballot_w64(keeps) != 0) {
                lead_kept |= 1u << l;
#pragma unroll
                for (int e = 0; e < 2; ++e) m[e] = fmaxf(m[e], mt[e]);
                m2 = fmaxf(m2, own);
            }
        }
    }
    const float m_sub = finite_max(m2);

    uint8_t* const mrow = p.mask ? p.mask + ((size_t)head * p.Tr + i) * p.Tc : nullptr;
    if (mrow)
        for (int j = nv + tid; j < p.Tc; j += 256) mrow[j] = 2;

    // this wave's say on tile j, whose row max (of this lane's half) is r
    auto vote = [&](int j, float r) __attribute__((always_inline)) {
        const float mt = xhalf_max(r) * p.c;
        const bool row_keeps = (qrow < N) && (mt != -INFINITY) && !(mt < m2 - p.thr2);
        int keeps = __builtin_amdgcn_ballot_w64(row_keeps) != 0 ? 1 : 0;
        if (j < n1) keeps = (lead_kept >> j) & 1;
        else if (j >= lo2 && j < lo2 + n2) keeps = (lead_kept >> (n1 + j - lo2)) & 1;
        if (lane == 0) votes[(j & 1) * 4 + wave] = (uint8_t)keeps;
    };
    vote(0, r0);

    f32x16 ot[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) ot[db] = f32x16{0};
    float lsum = 0.f;
    uint32_t pk[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) pk[e] = 0;
    bool kept_before = false;  // tile k - 1 was kept
    uint64_t kept = 0;         // bit k & 63: tile k

    const int kbase = T::k_base(ql, hh), vbase = T::v_base(lane, hh);
    __syncthreads();

    using std::false_type;
    using std::true_type;
    auto slice = [&](int q, const f32x16* st, uint32_t* pk) __attribute__((always_inline)) {
        const int t = q >> 3, r = 2 * (q & 7);
        const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[t][r], p.c, -m_sub));
        const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[t][r + 1], p.c, -m_sub));
        lsum += e0;
        lsum += e1;
        pk[q] = pack_bf16(e0, e1);
    };
    // step k: scores of tile k in s0, P of tile k - 1 in pk; leaves the scores of tile k + 1 in s1 and P of tile k in pk.  MASKED: tile k + 1 may
    // need a mask.  LAST: there is none
    auto step = [&](int k, f32x16* s0, f32x16* s1, auto masked_c, auto last_c) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_c)::value, LAST = decltype(last_c)::value;
        const uint8_t* kt = Ks + ((k + 1) % S) * T::BYTES;
        const uint8_t* vt = Vs + ((k + 1) % S) * T::BYTES;
        bf16x8 f[4];
        auto ldk = [&](int x) __attribute__((always_inline)) {
            return *reinterpret_cast<const bf16x8*>(kt + (kbase ^ ((x >> 1) << 5)) + (x & 1) * 32 * T::ROWB);
        };
        auto ldv = [&](int x) __attribute__((always_inline)) {
            const uint8_t* a = vt + (vbase ^ ((x % DB) << 6)) + 16 * (x / DB) * T::ROWB;
            const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a));
            const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a + 8 * T::ROWB));
            const u32x2 a0 = __builtin_bit_cast(u32x2, v0), a1 = __builtin_bit_cast(u32x2, v1);
            const u32x4 aw = {a0[0], a0[1], a1[0], a1[1]};
            return __builtin_bit_cast(bf16x8, aw);
        };
        auto mfk = [&](int x) __attribute__((always_inline)) {
            s1[x & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[x & 3], qf[x >> 1], x < 2 ? f32x16{0} : s1[x & 1], 0, 0, 0);
            if (x + 4 < 16) f[x & 3] = ldk(x + 4);
        };
        const uint32_t v = *reinterpret_cast<const uint32_t*>(votes + (k & 1) * 4);  // the votes on tile k, behind P.V
        __builtin_amdgcn_s_setprio(1);
        if (kept_before) {
#pragma unroll
            for (int x = 0; x < 4; ++x) f[x] = ldv(x);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const int c = x / DB;
                const u32x4 pw = {pk[4 * c], pk[4 * c + 1], pk[4 * c + 2], pk[4 * c + 3]};
                ot[x % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[x & 3], __builtin_bit_cast(bf16x8, pw), ot[x % DB], 0, 0, 0);
                if (x + 4 < 16) f[x & 3] = ldv(x + 4);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!LAST) {
#pragma unroll
            for (int x = 0; x < 4; ++x) f[x] = ldk(x);
        }
        const bool keep = __builtin_amdgcn_readfirstlane((int)v) != 0;
        if (!LAST) request_k(k + 2, k % S);
        if (keep) request_v(k, S + k % S);
        __builtin_amdgcn_sched_barrier(0);
        if (keep) {
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                if (!LAST) mfk(x);
                slice(x, s0, pk);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else if (!LAST) {
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                mfk(x);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_s_setprio(0);
        if (!LAST) {
            if (MASKED) mask(k + 1, s1);
            vote(k + 1, tile_rowmax<false>(s1, 0, 0, hh));
        }
        kept |= (uint64_t)(keep ? 1 : 0) << (k & 63);
        if (mrow && wave == 0 && (LAST || (k & 63) == 63)) {  // the mask, 64 steps at a time (a store is waited for with the requests)
            const int j = (k & ~63) + lane;
            if (lane <= (k & 63)) mrow[j] = (kept >> lane) & 1 ? 0 : 1;
        }
        if ((k & 63) == 63) kept = 0;
        kept_before = keep;
        __builtin_amdgcn_s_waitcnt(0x0070);  // what was requested has landed; the vote is written, the slots are read
        __builtin_amdgcn_s_barrier();
    };
    int j_masked = min(p.causal ? a_lo : p.Tc, nv);  // first tile that needs masking
    if (N % BN) j_masked = min(j_masked, p.Tc - 1);
    int k = 0;
    for (; k + 2 <= j_masked - 1; k += 2) {  // (tile k + 1 is what a step may have to mask)
        step(k, sa, sb, false_type{}, false_type{});
        step(k + 1, sb, sa, false_type{}, false_type{});
    }
#pragma unroll 1
    for (; k < nv - 1; ++k) {
        step(k, sa, sb, true_type{}, false_type{});
#pragma unroll
        for (int t = 0; t < 2; ++t) sa[t] = sb[t];
    }
    step(k, sa, sb, true_type{}, true_type{});
    if (kept_before) pv_tile_pipe<D>(Vs + (k % S) * T::BYTES, pk, ot, lane, hh);

    store_output<D, 0, DB>(p, ot, m_sub, lsum, 0, head, qrow, hh);
}

}  // namespace
