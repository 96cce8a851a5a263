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
// its first steps and only the last of them needs a mask, so there are two copies of a step and no branch between
// them (with one the compiler moved O between registers in every step: 93 us for 82 at 32 heads, N = 2048, no mask).
// What bounds it: below 500 keys the launch and the chain of load latencies (4.3 - 5.3 us for an empty sequence); then the two waves of
// a SIMD, 2500 cycles for 64 rows x 128 keys against 1024 of MFMA, and the 64 KiB of tiles they take (twice the bytes per row of
// the 128-row kernels), which is why longer sequences stay with those.
// KQ = 2: two workgroups per compute unit (80 KiB each at d = 128).  KQ = 4: one, for grids of no more items than compute units.
// Calls in us, without it and with it: d = 128, 32 heads over 8, causal, N = 200 14.4 / 7.3, 512 18.5 / 10.3, 777 22.2 / 15.2, 1024 24.4 /
// 17.5; 8 heads over 2, N = 2048 33.2 / 20.6 (KQ = 4); 160 heads, N = 320 36.7 / 19.3; d = 64, 32 heads over 8, N = 777 15.3 / 10.2.
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
    const int g = p.Hq / p.Hkv, G = p.B * p.Hkv;
    const int id = blockIdx.x;
    if (id >= p.n_items) {  // the summaries, for the caller: a block of keys per wave
        const int w = (id - p.n_items) * 2 * KQ + wave;
        if (w < G * p.Tc) summary_of_block<D>(p.K, const_cast<uint16_t*>(p.Krepr), w / p.Tc, w % p.Tc, p.N, p.N, p.Tc, BN, lane);
        return;
    }
    // items: late (long) query blocks first; the KV heads congruent mod 8 on one XCD, as in the other kernels
    int b, h, i;
    {
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
    b = __builtin_amdgcn_readfirstlane(b);
    h = __builtin_amdgcn_readfirstlane(h);
    i = __builtin_amdgcn_readfirstlane(i);
    const int hkv = __builtin_amdgcn_readfirstlane(h / g);
    const int N = p.N;
    const int row0 = p.row_base + i * BM;
    const int n_vis = p.causal ? min(N, row0 + BM) : N;  // keys that any row sees
    const int n_steps = (n_vis + KT - 1) / KT;

    const uint16_t* Qg = p.Q + ((size_t)(b * p.Hq + h) * N) * D;
    const uint16_t* Kg = p.K + ((size_t)(b * p.Hkv + hkv) * N) * D;
    const uint16_t* Vg = p.V + ((size_t)(b * p.Hkv + hkv) * N) * D;

    // ---- requests: a wave moves LI adjacent pieces (1 KiB of whole rows) of the K and of the V slot, by buffer loads whose buffer is
    // the slot's keys: rows past the end of the sequence are out of its range and LDS gets zeros
    const int r_own = RPI * LI * wave + lane / T::CH, cp = lane % T::CH;
    uint32_t offK[LI], offV[LI];
#pragma unroll
    for (int u = 0; u < LI; ++u) {
        offK[u] = (uint32_t)(r_own * T::ROWB + ((cp ^ T::k_mix(r_own + RPI * u)) << 4));
        offV[u] = (uint32_t)(r_own * T::ROWB + ((cp ^ T::v_mix(r_own + RPI * u)) << 4));
    }
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)(short_smem + wave * LI * 1024));
    auto request = [&](const uint16_t* base, int s, const uint32_t* o, uint32_t at) __attribute__((always_inline)) {
        const uint64_t a = (uint64_t)(uintptr_t)base + (uint64_t)(uint32_t)s * (uint32_t)F::SLOT;
        const uint32_t bytes = min(max(N - s * KT, 0), KT) * T::ROWB;
        if constexpr (LI == 4) request4(a, bytes, o[0], o[1], o[2], o[3], lds0 + at);
        else request2(a, bytes, o[0], o[1], lds0 + at);
    };
    auto request_k = [&](int s) __attribute__((always_inline)) { request(Kg, s, offK, (uint32_t)(s % 3) * F::SLOT); };
    auto request_v = [&](int s) __attribute__((always_inline)) { request(Vg, s, offV, (uint32_t)(3 + (s & 1)) * F::SLOT); };

    const int qrow0 = row0 + 32 * rw, qrow = qrow0 + ql;
    const int qrow_c = min(qrow, N - 1);
    const int limit = p.causal ? qrow_c : N - 1;
    const int k_last = p.causal ? min(N - 1, qrow0 + 31) : N - 1;  // last key that any row of the wave sees
    bf16x8 qf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
        qf[kk] = *reinterpret_cast<const bf16x8*>(Qg + (size_t)qrow_c * D + 16 * kk + 8 * hh);
    request_k(0);
    request_k(1);
    request_v(0);
    request_k(2);

    f32x16 ot[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) ot[db] = f32x16{0};
    float m2 = -INFINITY, lsum = 0.f;
    const int kbase = T::k_base(ql, hh) + 32 * kq * T::ROWB, vbase = T::v_base(lane, hh) + 32 * kq * T::ROWB;
    auto ld_k = [&](const uint8_t* kt, int kk) __attribute__((always_inline)) { return *reinterpret_cast<const bf16x8*>(kt + (kbase ^ (kk << 5))); };
    auto ld_v = [&](const uint8_t* vt, int f) __attribute__((always_inline)) {
        const uint8_t* a = vt + (vbase ^ ((f % DB) << 6)) + 16 * (f / DB) * T::ROWB;
        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a));
        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a + 8 * T::ROWB));
        const u32x2 a0 = __builtin_bit_cast(u32x2, v0), a1 = __builtin_bit_cast(u32x2, v1);
        const u32x4 aw = {a0[0], a0[1], a1[0], a1[1]};
        return __builtin_bit_cast(bf16x8, aw);
    };
    __builtin_amdgcn_s_waitcnt(0x0F70 | (3 * LI));  // K of step 0 has landed
    __syncthreads();
    f32x16 st = f32x16{0};
    if (32 * kq <= k_last) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld_k(Ks, kk), qf[kk], st, 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70 | LI);  // K of step 1 and V of step 0
    __syncthreads();

    // step s: softmax of its scores and P.V, with Q.K^T of step s + 1 (NEXT) in front
    auto step = [&](int s, auto next_c, auto masked_c) __attribute__((always_inline)) {
        constexpr bool NEXT = decltype(next_c)::value, MASKED = decltype(masked_c)::value;
        const int c0 = s * KT + 32 * kq;
        const uint8_t* const kt = Ks + ((s + 1) % 3) * F::SLOT;
        const uint8_t* const vt = Vs + (s & 1) * F::SLOT;
        bf16x8 fr[4];
        constexpr int H = KK / 2;
        if (NEXT) {
#pragma unroll
            for (int e = 0; e < 4; ++e) fr[e] = ld_k(kt, e);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (MASKED) {
            const int rel = limit - c0 - 4 * hh;
#pragma unroll
            for (int r = 0; r < 16; ++r) st[r] = (8 * (r >> 2) + (r & 3) <= rel) ? st[r] : -INFINITY;
        }
        f32x16 sn = f32x16{0};
        float mx[2] = {st[0], st[1]};
        // the first half of Q.K^T with the row max dealt out between
#pragma unroll
        for (int e = 0; e < H; ++e) {
            if (NEXT) {
                sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[e & 3], qf[e], sn, 0, 0, 0);
                if (e + 4 < KK) fr[e & 3] = ld_k(kt, e + 4);
            }
            if (e + 4 >= KK) fr[e & 3] = ld_v(vt, e + 4 - KK);
            if (e == 1) request_v(s + 1);
#pragma unroll
            for (int r = 2 + 14 * e / H; r < 2 + 14 * (e + 1) / H; ++r) mx[r & 1] = fmaxf(mx[r & 1], st[r]);
            if (NEXT) __builtin_amdgcn_sched_barrier(0);
        }
        const float m_new = fmaxf(m2, __builtin_fmaf(xhalf_max(fmaxf(mx[0], mx[1])), p.c, kKeepMax));
        if (__builtin_amdgcn_ballot_w64(!(m_new <= m2 + kKeepMax)) != 0) {
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
                if (e + 4 < KK) fr[e & 3] = ld_k(kt, e + 4);
            }
            if (e + 4 >= KK) fr[e & 3] = ld_v(vt, e + 4 - KK);
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
            if (f + 4 < 2 * DB) fr[f & 3] = ld_v(vt, f + 4);
            if (f == 0) request_k(s + 3);
#pragma unroll
            for (int q = 4 + 4 * f / DB; q < 4 + 4 * (f + 1) / DB; ++q) slice(q);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int f = 0; f < DB; ++f) ot[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[(f + DB) & 3], pf(1), ot[f], 0, 0, 0);
        if (NEXT) st = sn;
    };
    using std::false_type;
    using std::true_type;
    auto next_step = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0x0070 | LI);  // all requests but K of step s + 3, and the reads of the slots that are written next
        __builtin_amdgcn_s_barrier();
    };
    const int n_own = k_last < 32 * kq ? 0 : (k_last - 32 * kq) / KT + 1;  // steps that this wave has keys in: the first ones
    int s = 0;
    for (; s < n_own - 1; ++s) {
        step(s, true_type{}, false_type{});
        next_step();
    }
    if (n_own > 0) {
        step(s, false_type{}, true_type{});
        next_step();
        ++s;
    }
    for (; s < n_steps; ++s) {
        request_v(s + 1);
        request_k(s + 3);
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
            p.LSE[(size_t)(b * p.Hq + h) * N + qrow] = l > 0.f ? (m + __builtin_amdgcn_logf(l)) * kLn2 : -INFINITY;
        uint16_t* const Og = p.O + ((size_t)(b * p.Hq + h) * N + qrow_c) * D;
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
