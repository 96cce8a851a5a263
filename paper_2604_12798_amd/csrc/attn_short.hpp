// Alg. 1 on short sequences, and the rows of a call that do not fill a round of the ping-pong kernel (attn_pingpong.hpp): bf16,
// one 64-row query block per workgroup, the keys of a step split over KQ groups of two waves.
#pragma once
#include "common.hpp"
#include "summary.hpp"

namespace {

// ---------------------------------------------------------------------------------------------
// On a short sequence the fixed max of Alg. 1 costs more than it saves: a launch of its own for the summaries (3 - 5 us), one more
// tile product for them and for the sink and local blocks, and items long enough to pay for both.  Here every block's scores
// enter the max exactly (all blocks are what Alg. 1 calls special ones), each wave keeping a reference of its own, m2, the max plus
// kKeepMax, which it moves only when a row's max passes it, so that the rescale of O is rare; the weights are exp2(s - m2), at
// most 1, and sums of large values overflow no sooner than elsewhere.  The
// waves' sums are weighted by exp2(m2 - largest m2) when they meet in LDS.  The summaries, which the caller may want
// from the workspace, are written by workgroups behind the items, of the same launch.
//
// A step is 32 KQ keys; wave (rw, kq) multiplies the 32 keys of group kq with rows 32 rw .. 32 rw + 31, so all waves are busy however few
// rows an item has.  A wave's step: Q.K^T of the next step's keys with the row max and the first half of the weights of this
// one's dealt out between the MFMAs, then P.V with the second half.  K slots are requested two steps ahead, V slots one, the
// requests dealt out too (in front of the step they hold up its first MFMAs: 8 % of the time); one barrier per step.  A wave meets its keys in
// its first steps and only the last of them needs a mask, so there are two copies of a step's code and no branch between them.
// What bounds it: below 500 keys the launch and the chain of load latencies (4.6 us for an empty sequence); then a wave's own chain, 170
// instructions for 16 MFMAs: 0.5 us a step where a workgroup has a compute unit to itself, 1.06 to 1.13 for a step of each of two (64 keys and
// rows, d = 128, no mask).  Per score that is 1.05 to 1.17 times the ping-pong kernel's time in full rounds of long items, so those stay with that one.
// Measured on a single workgroup: slots deeper by one step or three change nothing, all eight fragments of K in front and the weights between the MFMAs
// of Q.K^T only cost 8 %.
// The first form waited in every step for the requests just made (see Q below), took a slot's place and its wrap from vector and scalar
// arithmetic (226 instructions) and moved the scores from one step to the next.
// KQ = 2: two workgroups per compute unit (80 KiB each at d = 128).  KQ = 4: one, for grids of no more items than compute units.
// Calls in us, first form / this: d = 128, 32 heads over 8, causal, N = 256 7.2 / 6.4, 512 10.0 / 8.8, 777 15.3 / 12.8, 1024 19.4 / 16.4; 8 heads, N =
// 1536 (KQ = 4) 17.5 / 14.6; no mask, 32 heads, N = 576 14.3 / 12.2; d = 64, 32 heads over 8, causal, N = 777 10.1 / 8.4, 1536 21.3 / 17.2.
constexpr float kKeepMax = 8.f;

template <int D, int KQ>
struct Short {
    static constexpr int KT = 32 * KQ;                       // keys per step
    static constexpr int SLOT = KT * Tile<D>::ROWB;          // of K or V
    static constexpr int NU = 2 * (D / 32);                  // units of O^T: eight registers, 16 features of a row
    static constexpr int LDS_BYTES = 5 * SLOT;  // three K and two V slots; at the end the partial O^T, max and l
    static_assert(2 * KQ * (NU * 2048 + 256) <= 5 * SLOT, "the partial sums have to fit the tiles' memory");
};

template <int D, int KQ>
__global__ __launch_bounds__(128 * KQ, 2) void attn_fwd_short_kernel(const Params p) {
    using T = Tile<D>;
    using F = Short<D, KQ>;
    constexpr int BM = 64, KK = D / 16, DB = D / 32, KT = F::KT, NU = F::NU, OWN = NU / KQ;
    constexpr int LI = F::SLOT / 1024 / (2 * KQ);  // load instructions per wave and slot
    constexpr int RPI = 1024 / T::ROWB;
    extern __shared__ __attribute__((aligned(16))) uint8_t short_smem[];
    uint8_t* const Ks = short_smem;
    uint8_t* const Vs = short_smem + 3 * F::SLOT;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = wave & 1, kq = wave >> 1;
    const int ql = lane & 31;
    const int hh = lane >> 5;
    const int id = blockIdx.x;
    if (id >= p.n_items) {  // the summaries, for the caller: a block of keys per wave
        const int w = (id - p.n_items) * 2 * KQ + wave;
        if (w < p.B * p.Hkv * p.Tc) summary_of_block<D>(p.K, const_cast<uint16_t*>(p.Krepr), w / p.Tc, w % p.Tc, p.N, p.N, p.Tc, BN, lane);
        return;
    }
    const auto [head, kv, i] = item_of(p, id);
    const int N = p.N;
    const int row0 = p.row_base + i * BM;
    const int n_vis = p.causal ? min(N, row0 + BM) : N;  // keys that any row sees
    const int n_steps = (n_vis + KT - 1) / KT;

    // ---- requests: a wave moves LI adjacent pieces (1 KiB of whole rows) of the K and of the V slot, by buffer loads whose buffer is
    // the head's keys: rows past the end of the sequence are out of its range and LDS gets zeros.  The slot's place is the loads' scalar
    // offset, so that a request costs three scalar instructions beside them
    const int r_own = RPI * LI * wave + lane / T::CH, cp = lane % T::CH;
    uint32_t offK[LI];
#pragma unroll
    for (int u = 0; u < LI; ++u) offK[u] = (uint32_t)(r_own * T::ROWB + ((cp ^ T::k_mix(r_own + RPI * u)) << 4));
    const uint32_t offV = (uint32_t)(r_own * T::ROWB + ((cp ^ T::v_mix(r_own)) << 4));  // (the same for all pieces)
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)(short_smem + wave * LI * 1024));
    const uint32_t bytes = (uint32_t)N * T::ROWB;  // (launched for fewer than 2^32)
    const u32x4 rsrcK = tile_buffer((uint64_t)(uintptr_t)(p.K + (size_t)kv * N * D), bytes), rsrcV = tile_buffer((uint64_t)(uintptr_t)(p.V + (size_t)kv * N * D), bytes);
    // K or V of step s (at = s * SLOT bytes) into the slot whose number among all five is `slot`
    auto request_k = [&](uint32_t at, uint32_t slot) __attribute__((always_inline)) {
        if constexpr (LI == 4) request4_at(rsrcK, at, offK[0], offK[1], offK[2], offK[3], lds0 + slot * F::SLOT);
        else request2_at(rsrcK, at, offK[0], offK[1], lds0 + slot * F::SLOT);
    };
    auto request_v = [&](uint32_t at, uint32_t slot) __attribute__((always_inline)) {
        if constexpr (LI == 4) request4_at(rsrcV, at, offV, offV, offV, offV, lds0 + slot * F::SLOT);
        else request2_at(rsrcV, at, offV, offV, lds0 + slot * F::SLOT);
    };

    const int qrow0 = row0 + 32 * rw, qrow = qrow0 + ql;
    const int qrow_c = min(qrow, N - 1);
    const int limit = p.causal ? qrow_c : N - 1;
    const int k_last = p.causal ? min(N - 1, qrow0 + 31) : N - 1;  // last key that any row of the wave sees
    // Q goes through LDS too (the second V slot, which step 0 is the first to write): whole rows, and no load whose result the compiler has
    // to wait for.  (With Q loaded to registers it waited for them, on the path that skips the first Q.K^T, inside every step, and so for all
    // requests of K and V in flight.)
    {
        const u32x4 rsrcQ = tile_buffer((uint64_t)(uintptr_t)(p.Q + ((size_t)head * N + row0) * D), (uint32_t)min(N - row0, BM) * T::ROWB);
        if (RPI * LI * wave < BM) {
            if constexpr (LI == 4) request4_at(rsrcQ, 0, offK[0], offK[1], offK[2], offK[3], lds0 + 4 * F::SLOT);
            else request2_at(rsrcQ, 0, offK[0], offK[1], lds0 + 4 * F::SLOT);
        }
    }
    request_k(0, 0);
    request_k(F::SLOT, 1);
    request_v(0, 3);
    request_k(2 * F::SLOT, 2);

    f32x16 ot[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) ot[db] = f32x16{0};
    float m2 = -INFINITY, lsum = 0.f;
    // fragment addresses: a slot is a constant offset
    uint32_t ka[KK], va[DB];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) ka[kk] = lds_addr(Ks) + (((T::k_base(ql, hh) ^ (kk << 5))) + 32 * kq * T::ROWB);
#pragma unroll
    for (int db = 0; db < DB; ++db) va[db] = lds_addr(Vs) + ((T::v_base(lane, hh) ^ (db << 6)) + 32 * kq * T::ROWB);
    auto ld_k = [&](uint32_t slot, int kk) __attribute__((always_inline)) { return *(lds_frag)(ka[kk] + slot); };
    auto ld_v = [&](uint32_t slot, int f) __attribute__((always_inline)) {
        const uint32_t a = va[f % DB] + (slot + 16 * (f / DB) * T::ROWB);
        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(a));
        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(a + 8 * T::ROWB));
        const u32x2 a0 = __builtin_bit_cast(u32x2, v0), a1 = __builtin_bit_cast(u32x2, v1);
        const u32x4 aw = {a0[0], a0[1], a1[0], a1[1]};
        return __builtin_bit_cast(bf16x8, aw);
    };
    __builtin_amdgcn_s_waitcnt(0x0F70 | (3 * LI));  // Q and K of step 0 have landed
    __syncthreads();
    bf16x8 qf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[kk] = *(lds_frag)(lds_addr(Vs) + F::SLOT + (T::k_base(ql, hh) ^ (kk << 5)) + 32 * rw * T::ROWB);
    f32x16 sa = f32x16{0}, sb;
    if (32 * kq <= k_last) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld_k(0, kk), qf[kk], sa, 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0x0070 | LI);  // K of step 1 and V of step 0; Q has been read
    __syncthreads();

    // step s (at = s * SLOT): softmax of its scores st and P.V, with Q.K^T of step s + 1 (NEXT), whose scores go to sn, in front.  slot_k,
    // slot_v: byte offsets of K of step s + 1 in the K slots and of V of step s in the V slots; to_k, to_v: the slots that are written
    auto step = [&](int s, uint32_t at, f32x16& st, f32x16& sn, uint32_t slot_k, uint32_t slot_v, uint32_t to_k, uint32_t to_v, auto next_c, auto masked_c)
                    __attribute__((always_inline)) {
        constexpr bool NEXT = decltype(next_c)::value, MASKED = decltype(masked_c)::value;
        bf16x8 fr[4];
        constexpr int H = KK / 2;
        if (NEXT) {
#pragma unroll
            for (int e = 0; e < 4; ++e) fr[e] = ld_k(slot_k, e);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (MASKED) {
            const int rel = limit - (s * KT + 32 * kq) - 4 * hh;
#pragma unroll
            for (int r = 0; r < 16; ++r) st[r] = (8 * (r >> 2) + (r & 3) <= rel) ? st[r] : -INFINITY;
        }
        float mx = fmaxf(fmaxf(st[0], st[1]), st[2]);
        // the first half of Q.K^T with the row max dealt out between
#pragma unroll
        for (int e = 0; e < H; ++e) {
            if (NEXT) {
                sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[e & 3], qf[e], e == 0 ? f32x16{0} : sn, 0, 0, 0);
                if (e + 4 < KK) fr[e & 3] = ld_k(slot_k, e + 4);
            }
            if (e + 4 >= KK) fr[e & 3] = ld_v(slot_v, e + 4 - KK);
            if (e == 1) request_v(at + F::SLOT, to_v);
#pragma unroll
            for (int q = 6 * e / H; q < 6 * (e + 1) / H; ++q) mx = fmaxf(fmaxf(mx, st[3 + 2 * q]), st[4 + 2 * q]);
            if (NEXT) __builtin_amdgcn_sched_barrier(0);
        }
        // (the third operand saves the two instructions that would quiet signalling NaNs first)
        mx = fmaxf(mx, st[15]);
        const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        const float m_tile = __builtin_fmaf(fmaxf(fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1])), -INFINITY), p.c, kKeepMax);
        if (__builtin_amdgcn_ballot_w64(!(m_tile <= m2 + kKeepMax)) != 0) {
            const float m_new = fmaxf(m2, m_tile);
            const float msub = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m2 - msub);
            lsum *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db) ot[db] *= alpha;
            m2 = m_new;
        }
        const float msub = m2 == -INFINITY ? 0.f : m2;
        uint32_t pk[8];
        auto slice = [&](int q) __attribute__((always_inline)) {
            const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[2 * q], p.c, -msub));
            const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[2 * q + 1], p.c, -msub));
            lsum += e0;
            lsum += e1;
            pk[q] = pack_bf16(e0, e1);
        };
        __builtin_amdgcn_sched_barrier(0);
        // the second half with the first 16 weights
#pragma unroll
        for (int e = H; e < KK; ++e) {
            if (NEXT) {
                sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[e & 3], qf[e], sn, 0, 0, 0);
                if (e + 4 < KK) fr[e & 3] = ld_k(slot_k, e + 4);
            }
            if (e + 4 >= KK) fr[e & 3] = ld_v(slot_v, e + 4 - KK);
#pragma unroll
            for (int q = 4 * (e - H) / H; q < 4 * (e - H + 1) / H; ++q) slice(q);
            if (NEXT) __builtin_amdgcn_sched_barrier(0);
        }
        auto pf = [&](int c) __attribute__((always_inline)) {
            const u32x4 pw = {pk[4 * c], pk[4 * c + 1], pk[4 * c + 2], pk[4 * c + 3]};
            return __builtin_bit_cast(bf16x8, pw);
        };
        // P.V of the first 16 keys with the other 16 weights, then of those
#pragma unroll
        for (int f = 0; f < DB; ++f) {
            ot[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[f & 3], pf(0), ot[f], 0, 0, 0);
            if (f + 4 < 2 * DB) fr[f & 3] = ld_v(slot_v, f + 4);
            if (f == 0) request_k(at + 3 * F::SLOT, to_k);
#pragma unroll
            for (int q = 4 + 4 * f / DB; q < 4 + 4 * (f + 1) / DB; ++q) slice(q);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int f = 0; f < DB; ++f) ot[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[(f + DB) & 3], pf(1), ot[f], 0, 0, 0);
    };
    using std::false_type;
    using std::true_type;
    auto next_step = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0x0070 | LI);  // all requests but K of step s + 3, and the reads of the slots that are written next
        __builtin_amdgcn_s_barrier();
    };
    const int n_own = k_last < 32 * kq ? 0 : (k_last - 32 * kq) / KT + 1;  // steps that this wave has keys in: the first ones
    int s = 0;
    uint32_t at = 0;
    // six steps in a row bring the slots back to where they were (three of K, two of V), so that each step's are constants
    for (;;) {
        auto one = [&](auto j_c) __attribute__((always_inline)) {  // (as a function with a result: a break behind each step made the compiler spill)
            constexpr int J = decltype(j_c)::value;
            if (s >= n_own - 1) return false;
            step(s, at, J & 1 ? sb : sa, J & 1 ? sa : sb, (J + 1) % 3 * F::SLOT, J % 2 * F::SLOT, J % 3, 3 + (J + 1) % 2, true_type{}, false_type{});
            next_step();
            ++s;
            at += F::SLOT;
            return true;
        };
        if (!one(std::integral_constant<int, 0>{})) break;
        if (!one(std::integral_constant<int, 1>{})) break;
        if (!one(std::integral_constant<int, 2>{})) break;
        if (!one(std::integral_constant<int, 3>{})) break;
        if (!one(std::integral_constant<int, 4>{})) break;
        if (!one(std::integral_constant<int, 5>{})) break;
    }
    if (n_own > 0) {
        if (s & 1) sa = sb;
        step(s, at, sa, sb, 0, s % 2 * F::SLOT, s % 3, 3 + (s + 1) % 2, false_type{}, true_type{});
        next_step();
        ++s;
        at += F::SLOT;
    }
    for (; s < n_steps; ++s, at += F::SLOT) {
        request_v(at + F::SLOT, 3 + (s + 1) % 2);
        request_k(at + 3 * F::SLOT, s % 3);
        next_step();
    }
    wait_vm0_and_sync();  // (the requests past the last step write zeros)

    // ---- the groups add their sums: each takes OWN units of O^T, the others' shares weighted by exp2(m - largest m)
    float* const ex = reinterpret_cast<float*>(short_smem);
    float* const xml = reinterpret_cast<float*>(short_smem + 2 * KQ * NU * 2048);  // [wave][max, l][32 rows]
    const float l_own = xhalf_sum(lsum);
    if (hh == 0) {
        xml[wave * 64 + ql] = m2;
        xml[wave * 64 + 32 + ql] = l_own;
    }
#pragma unroll
    for (int u = 0; u < NU; ++u)
        if (u / OWN != kq) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const f32x16& o = ot[u >> 1];
                const int r = 8 * (u & 1) + 4 * e;
                *reinterpret_cast<f32x4*>(ex + (((wave * NU + u) * 2 + e) * 64 + lane) * 4) = f32x4{o[r], o[r + 1], o[r + 2], o[r + 3]};
            }
        }
    __syncthreads();
    float m = -INFINITY, w[KQ], l = 0.f;
#pragma unroll
    for (int k = 0; k < KQ; ++k) m = fmaxf(m, xml[(2 * k + rw) * 64 + ql]);
    const float msub = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int k = 0; k < KQ; ++k) {
        w[k] = __builtin_amdgcn_exp2f(xml[(2 * k + rw) * 64 + ql] - msub);
        l += w[k] * xml[(2 * k + rw) * 64 + 32 + ql];
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    auto finish = [&](auto kq_c) __attribute__((always_inline)) {
        constexpr int KO = decltype(kq_c)::value;
        if (qrow < N && p.LSE && KO == 0 && hh == 0)
            p.LSE[(size_t)head * N + qrow] = l > 0.f ? (m + __builtin_amdgcn_logf(l)) * kLn2 : -INFINITY;
        uint16_t* const Og = p.O + ((size_t)head * N + qrow_c) * D;
#pragma unroll
        for (int v = 0; v < OWN; ++v) {
            constexpr int U0 = KO * OWN;
            const int u = U0 + v;
            float o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = 0.f;
#pragma unroll
            for (int k = 0; k < KQ; ++k)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    f32x4 x;
                    if (k == KO) {
                        const f32x16& own = ot[u >> 1];
                        const int r = 8 * (u & 1) + 4 * e;
                        x = f32x4{own[r], own[r + 1], own[r + 2], own[r + 3]};
                    } else {
                        x = *reinterpret_cast<const f32x4*>(ex + ((((2 * k + rw) * NU + u) * 2 + e) * 64 + lane) * 4);
                    }
#pragma unroll
                    for (int c = 0; c < 4; ++c) o[4 * e + c] = __builtin_fmaf(w[k], x[c], o[4 * e + c]);
                }
            // the lane pair (l, l ^ 32) trades runs of four features for runs of eight, as in store_output
            const uint32_t a0 = pack_bf16(o[0] * inv, o[1] * inv), a1 = pack_bf16(o[2] * inv, o[3] * inv);
            const uint32_t b0 = pack_bf16(o[4] * inv, o[5] * inv), b1 = pack_bf16(o[6] * inv, o[7] * inv);
            const auto r0 = __builtin_amdgcn_permlane32_swap(a0, b0, false, false);
            const auto r1 = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
            if (qrow < N) *reinterpret_cast<u32x4*>(Og + 32 * (u >> 1) + 16 * (u & 1) + 8 * hh) = u32x4{r0[0], r1[0], r0[1], r1[1]};
        }
    };
    if constexpr (KQ == 4) {
        if (kq == 0) finish(std::integral_constant<int, 0>{});
        else if (kq == 1) finish(std::integral_constant<int, 1>{});
        else if (kq == 2) finish(std::integral_constant<int, 2>{});
        else finish(std::integral_constant<int, 3>{});
    } else {
        if (kq == 0) finish(std::integral_constant<int, 0>{});
        else finish(std::integral_constant<int, 1>{});
    }
}

}  // namespace
