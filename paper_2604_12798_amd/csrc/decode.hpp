// Decode kernels: one query token per head against a growing key/value cache.
#pragma once
#include "common.hpp"

namespace {

// ---------------------------------------------------------------------------------------------
// Decode: one query token per head against a key/value cache, the keys split over workgroups.
// A wave carries the Hq / Hkv (<= 32) query heads of one KV head as the columns of its score tile
// (unused columns repeat the last head).  Two small kernels:
//   decode_split_kernel  per (KV head, key range): sum exp(s - m) and sum exp(s - m) v over the range, m its running row
//                        max (the rescale of the sums is branched over in every tile that does not raise it)
//   decode_merge_kernel  per query head: the ranges' partial sums, each weighted by exp(m_range - max m), added, divided
// With one range per head (n_splits = 1) the first kernel writes O and LSE itself.
// A fixed max from the block summaries and the sink / local blocks, which the prefill kernels gain from, costs a decode step
// time: it has to be known before the first range starts, so a kernel of its own went over the summaries in front of the
// split kernel (3.5 - 5 us of a step), to save vector work that is hidden under the reads anyway.  Here a range needs
// nothing from another one before the merge.  (Seeding each range's max from its own summaries was measured too: the same
// time, and the largest weights of a row are then rounded to bf16, which they are not when the max is exact.)
// The work is HBM bound (K and V are read once), so the score and P.V helpers of the prefill kernels are enough; what matters
// is how the tiles are fetched: into registers, with non-temporal loads, one tile ahead, and from there into the two LDS
// tiles a wave owns (see decode_split_kernel).
struct DecodeParams {
    const uint16_t* Q;      // [B, Hq, d]
    const uint16_t* K;      // [B, Hkv, n_cap, d]
    const uint16_t* V;
    // partial results of range r of batch entry b and head h in slot (first(b) + r) * Hq + h, where first(b) counts the
    // ranges of the entries before b (b * n_splits when every entry has n_splits ranges)
    float* pm;              // [B * n_splits * Hq]     the range's max, log2 units
    float* lpart;           // [B * n_splits * Hq]     sum of exp
    float* opart;           // [B * n_splits * Hq, d]  sum of exp * v
    uint16_t* O;            // [B, Hq, d]
    float* LSE;             // [B, Hq] or null
    int B, Hq, Hkv, n_cap, n_keys, n_splits;
    int g, per;  // query heads per KV head; tiles of a range where the batch has one length
    const int* seq_lens;    // null, or [B] device array: valid keys per batch entry (clamped to [1, n_cap]) instead of n_keys
    float c;
};

// What the entries of a batch have: one length; lengths of their own and n_splits ranges each; lengths of their own and ranges
// dealt out by length.
enum Lens { LENS_ONE = 0, LENS_FIXED = 1, LENS_DEALT = 2 };

// Keys of batch entry b.
__device__ __forceinline__ int decode_keys(const DecodeParams& p, int b) {
    return p.seq_lens ? min(max(p.seq_lens[b], 1), p.n_cap) : p.n_keys;
}

// Which tiles a range covers when every entry of the batch has a length of its own (LENS_DEALT).  The B * n_splits ranges are dealt
// to the entries by length, so that all are about equally long (a fixed number per entry leaves the ranges of short entries
// idle: the kernel took 52 us at 16 entries of 200 to 8192 keys, it takes 30): `per` tiles a range, the smallest value found
// from the even share upwards, in steps of an eighth, for which the entries' ranges fit into B * n_splits.  Every wave works
// this out by itself, from up to DEAL_MAX_B / 64 entries in each lane.  It is not done where that costs more than it gives:
//   more entries, or above 64 of them more than eight ranges for each compute unit: there is a search in each of many waves, and
//     the number of ranges evens out what dealing would (search over the whole batch against n_splits ranges each, d = 128: 256
//     entries of up to 512 keys, 8 KV heads, two ranges 77 / 46 us; 1024 entries 523 / 154; 4096 entries 6060 / 608)
//   above 64 entries with ranges of a tile or two (256 entries of up to 128 keys, one KV head, two ranges, d = 64 11.5 / 7.2)
//   one range per entry: there is nothing to deal
// In between it is worth it: 128 entries of up to 8192 keys, one KV head, four ranges 25 us dealt, 57 not.
constexpr int DEAL_MAX_B = 256;
struct Ranges {
    int b, first, nb;  // an entry, the ranges of the entries before it, its own number of ranges
};
// the entry that range w of the list belongs to (b = -1: past the last range), or, with w < 0, the ranges of entry b
__device__ __forceinline__ Ranges varlen_find(const DecodeParams& p, int lane, int w, int b) {
    constexpr int E = DEAL_MAX_B / 64;
    int tiles[E], n[E], sum = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        tiles[e] = 64 * e + lane < p.B ? (decode_keys(p, 64 * e + lane) + BN - 1) / BN : 0;
        sum += tiles[e];  // (256 entries of 2^25 tiles at most: a sum past 2^31 would not fit the GPU)
    }
    const int slots = p.B * p.n_splits;
    int per = max(1, (wave_sum(sum) + slots - 1) / slots);
    for (;; per += max(1, per >> 3)) {  // (ends where per passes the longest entry, with one range for each, or before)
        int ranges = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            n[e] = 64 * e < p.B ? (tiles[e] + per - 1) / per : 0;
            ranges += n[e];
        }
        if (wave_sum(ranges) <= slots) break;
    }
    Ranges out = {-1, 0, 0};
    int before = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (64 * e < p.B && out.b < 0) {
            const int upto = before + wave_prefix(n[e]);
            const uint64_t found = __builtin_amdgcn_ballot_w64(n[e] > 0 && (w >= 0 ? w >= upto - n[e] && w < upto : 64 * e + lane == b));
            if (found) {
                const int l = __builtin_ctzll(found);
                out.b = 64 * e + l;
                out.nb = __builtin_amdgcn_readlane(n[e], l);
                out.first = __builtin_amdgcn_readlane(upto, l) - out.nb;
            }
            before = __builtin_amdgcn_readlane(upto, 63);
        }
    }
    return out;
}

// One 64-row tile, global -> registers with the tile mover's lane mapping (every instruction covers whole rows, 1 KiB
// contiguous; the swizzle is applied on the global side), and registers -> LDS at the positions the LDS-direct mover
// writes.  The loads are non-temporal: the cache is streamed through once per step and is larger than L2 and the
// memory-side cache, and plain loads, which allocate there, cost 12 % of the stream's rate (LDS-direct loads another 7 %).
// They are buffer loads whose buffer is the tile: rows past the last key are out of its range and give zeros, and a lane's offset
// repeats every four instructions (offs[u & 3]), so a load costs no vector instruction, in a ragged tile as in a whole one
// (against 64-bit addresses per lane, with the rows of every range's first tile clamped, and divisions for what the host knows: steps of
// 4 x 8 heads of 32768 keys 89.5 / 86.9 us, 8 x 16 heads of 4001 keys, d = 64, 27.7 / 27.3, 16 sequences of up to 8192 keys 1.2 % faster).
template <int D>
__device__ __forceinline__ void tile_lane_offsets(bool is_v, int lane, uint32_t* offs) {
    using T = Tile<D>;
    constexpr int RPI = 1024 / T::ROWB;
    const int cp = lane % T::CH;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int rr = RPI * u + lane / T::CH;
        const int ch = cp ^ (is_v ? T::v_mix(rr) : T::k_mix(rr));
        offs[u] = (uint32_t)((lane / T::CH) * T::ROWB + ch * 16);
    }
}
template <int D>
__device__ __forceinline__ void tile_to_regs(const uint16_t* base, int tile, int n_keys, const uint32_t* offs, u32x4* r) {
    using T = Tile<D>;
    constexpr int NI = BN / (1024 / T::ROWB);
    uint8_t* const tb = const_cast<uint8_t*>(reinterpret_cast<const uint8_t*>(base) + (size_t)tile * T::BYTES);
    const int bytes = __builtin_amdgcn_readfirstlane(min(max(n_keys - tile * BN, 0), BN) * T::ROWB);  // (scalar, whatever unit the clamp runs on)
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(tb, 0, bytes, 0x00020000);
#pragma unroll
    for (int u = 0; u < NI; ++u) r[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, offs[u & 3], u * 1024, 2));
}
template <int D>
__device__ __forceinline__ void regs_to_tile(uint8_t* dst, int lane, const u32x4* r) {
    using T = Tile<D>;
    constexpr int NI = BN / (1024 / T::ROWB);
#pragma unroll
    for (int u = 0; u < NI; ++u) *reinterpret_cast<u32x4*>(dst + u * 1024 + lane * 16) = r[u];
}

// A workgroup is W waves that share one range, a wave taking a contiguous part of it.  The tiles are staged through registers:
// while tile t is worked on, V(t + 1) and K(t + 1), then K(t + 2), are in flight
// in registers (the accumulation registers: loads and LDS writes take them directly), each requested one tile ahead of
// its use, and LDS holds only the two tiles being read (32 KiB a wave at d = 128).  The LDS executes a wave's instructions in
// order: a tile is written over its predecessor behind the last read of that one, without a wait.  The steady loop runs
// over whole tiles and has no branch between a load and its use, so that the compiler's wait counts stay exact (a load
// that sits behind a branch makes it wait for everything at the join); the last one to three tiles, among them a
// ragged one, take the same body with the missing requests compiled out.
// (64-wide heads: half the bytes per tile and half the registers, so twice the waves per SIMD keep the same number of bytes
// in flight.)
template <int D, int W, int LENS>
__global__ __launch_bounds__(64 * W, D == 64 ? 2 : 1) void decode_split_kernel(const DecodeParams p) {
    using T = Tile<D>;
    constexpr int KK = D / 16, DB = D / 32;
    constexpr int NI = BN / (1024 / T::ROWB);
    constexpr int OROW = D + 4;  // row of the exchange of partial sums, in floats: padded against bank conflicts
    static_assert(32 * OROW * 4 + 64 * 4 <= 2 * T::BYTES, "the exchange has to fit the tiles' memory");
    __shared__ __attribute__((aligned(16))) uint8_t smem[W * 2 * T::BYTES];  // (up to 128 KiB; of fixed size, so no limit has to be raised for it)
    const int lane = threadIdx.x & 63, ql = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* const Ks = smem + wave * 2 * T::BYTES;
    uint8_t* const Vs = Ks + T::BYTES;
    // (lengths that differ and are not dealt out: all heads of an entry start together, so that no long one starts late)
    const int g = p.g, hkv = LENS == LENS_FIXED ? blockIdx.y : blockIdx.z;
    int b = LENS == LENS_FIXED ? blockIdx.z : blockIdx.y, r = blockIdx.x, nb = p.n_splits;  // batch entry, its range, the number of its ranges
    const int w = b * p.n_splits + r;  // range of the batch's list
    if (LENS == LENS_DEALT) {
        const Ranges rg = varlen_find(p, lane, w, 0);
        if (rg.b < 0) return;  // (the same in all waves of the workgroup)
        b = rg.b; r = w - rg.first; nb = rg.nb;
    }
    const size_t slot = (size_t)w * p.Hq + hkv * g;
    const int n_keys = LENS == LENS_ONE ? p.n_keys : __builtin_amdgcn_readfirstlane(decode_keys(p, b));
    const int Tc = (n_keys + BN - 1) / BN, per = LENS == LENS_ONE ? p.per : (Tc + nb - 1) / nb;
    const int r0 = r * per, r1 = min(Tc, r0 + per);  // its tiles
    const int share = (max(r1 - r0, 0) + W - 1) / W;
    const int t_lo = r0 + wave * share, t_hi = min(r1, t_lo + share);
    const int t_whole = min(t_hi, n_keys / BN);  // tiles below this index are whole
    const size_t bh = (size_t)b * p.Hkv + hkv;
    const uint16_t* Kg = p.K + bh * p.n_cap * D;
    const uint16_t* Vg = p.V + bh * p.n_cap * D;
    uint32_t offk[4], offv[4];
    tile_lane_offsets<D>(false, lane, offk);
    tile_lane_offsets<D>(true, lane, offv);
    bf16x8 qf[KK];
    {
        const int h = hkv * g + min(ql, g - 1);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            qf[kk] = *reinterpret_cast<const bf16x8*>(p.Q + ((size_t)b * p.Hq + h) * D + 16 * kk + 8 * hh);
    }
    f32x16 ot[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) ot[db] = f32x16{0};
    float m2 = -INFINITY, lsum = 0.f;
    u32x4 rk[NI], rv[NI];
    // tile t.  On entry K(t) is in LDS, rv holds V(t) and, requested after it, rk holds K(t + 1) (HASK1).
    // HASV1 / HASK2: tiles t + 1 / t + 2 exist; FULL: tile t is whole
    auto body = [&](int t, auto hasv1_c, auto hask1_c, auto hask2_c, auto full_c) __attribute__((always_inline)) {
        constexpr bool HASV1 = decltype(hasv1_c)::value, HASK1 = decltype(hask1_c)::value, HASK2 = decltype(hask2_c)::value;
        constexpr bool FULL = decltype(full_c)::value;
        f32x16 st[2];
        uint32_t pk[16];
        qk_tile_pipe<D>(Ks, qf, st, ql, hh);
        // (a ragged tail is masked)
        softmax_tile<true, !FULL, DB, true, true>(st, pk, ot, m2, lsum, p.c, t * BN, n_keys - 1, hh, 0.f);
        __builtin_amdgcn_sched_barrier(0);  // (requests and LDS writes go out where they are written, not where the scheduler likes them)
        regs_to_tile<D>(Vs, lane, rv);  // V(t) has landed when only K(t + 1) is still out
        if (HASV1) tile_to_regs<D>(Vg, t + 1, n_keys, offv, rv);
        __builtin_amdgcn_sched_barrier(0);
        pv_tile_pipe<D>(Vs, pk, ot, lane, hh);
        __builtin_amdgcn_sched_barrier(0);
        if (HASK1) regs_to_tile<D>(Ks, lane, rk);  // K(t + 1) has landed when only V(t + 1) is still out
        if (HASK2) tile_to_regs<D>(Kg, t + 2, n_keys, offk, rk);
        __builtin_amdgcn_sched_barrier(0);
    };
    using Y = std::true_type;
    using N_ = std::false_type;
    if (t_lo < t_hi) {
        tile_to_regs<D>(Kg, t_lo, n_keys, offk, rk);
        tile_to_regs<D>(Vg, t_lo, n_keys, offv, rv);
        __builtin_amdgcn_sched_barrier(0);
        regs_to_tile<D>(Ks, lane, rk);
        __builtin_amdgcn_sched_barrier(0);
        int t = t_lo;
        if (t + 2 < t_whole) {  // (the request for K(t + 1) is not behind a branch of its own: see above)
            tile_to_regs<D>(Kg, t + 1, n_keys, offk, rk);
            do {  // tiles t + 1 and t + 2 are whole and inside the range
                body(t, Y{}, Y{}, Y{}, Y{});
                ++t;
            } while (t + 2 < t_whole);
        } else if (t + 1 < t_hi) {
            tile_to_regs<D>(Kg, t + 1, n_keys, offk, rk);
        }
        if (t + 2 < t_hi) body(t++, Y{}, Y{}, Y{}, N_{});  // (at most one: t_hi <= t_whole + 1)
        if (t + 1 < t_hi) body(t++, Y{}, Y{}, N_{}, N_{});
        body(t, N_{}, N_{}, N_{}, N_{});
    }
    // the waves' sums meet in LDS (in the tiles' memory; each wave writes its own part, behind its own last reads)
    float* const ox = reinterpret_cast<float*>(Ks);
    const float l = xhalf_sum(lsum);
    if (ql < g) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
                *reinterpret_cast<f32x4*>(ox + ql * OROW + 32 * db + 8 * q4 + 4 * hh) =
                    f32x4{ot[db][4 * q4], ot[db][4 * q4 + 1], ot[db][4 * q4 + 2], ot[db][4 * q4 + 3]};
        if (hh == 0) {
            ox[32 * OROW + ql] = m2;
            ox[32 * OROW + 32 + ql] = l;
        }
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < g * (D / 4); idx += 64 * W) {
        const int col = idx / (D / 4), c4 = idx - col * (D / 4);
        const float* const x0 = reinterpret_cast<const float*>(smem);
        constexpr int WS = 2 * T::BYTES / 4;  // floats from one wave's part to the next
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < W; ++w) m = fmaxf(m, x0[w * WS + 32 * OROW + col]);
        const float msub = m == -INFINITY ? 0.f : m;
        float lt = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float a = W == 1 ? 1.f : __builtin_amdgcn_exp2f(x0[w * WS + 32 * OROW + col] - msub);
            lt += a * x0[w * WS + 32 * OROW + 32 + col];
            o += a * *reinterpret_cast<const f32x4*>(x0 + w * WS + col * OROW + 4 * c4);
        }
        if (p.n_splits == 1) {  // the only range: this is the result
            const size_t row = (size_t)b * p.Hq + hkv * g + col;
            const float inv = lt > 0.f ? 1.f / lt : 0.f;
            *reinterpret_cast<u32x2*>(p.O + row * D + 4 * c4) = u32x2{pack_bf16(o[0] * inv, o[1] * inv), pack_bf16(o[2] * inv, o[3] * inv)};
            if (p.LSE && c4 == 0) p.LSE[row] = lt > 0.f ? (m + __builtin_amdgcn_logf(lt)) * kLn2 : -INFINITY;
        } else {
            *reinterpret_cast<f32x4*>(p.opart + (slot + col) * D + 4 * c4) = o;
            if (c4 == 0) {
                p.pm[slot + col] = m;
                p.lpart[slot + col] = lt;
            }
        }
    }
}

// One workgroup per query head: D / 4 threads read a partial row (16 bytes each), 1024 / D rows at a time and up to four such
// rounds in flight, each group of threads with a running max of its own; the groups meet in LDS.  The order of the sums is
// fixed.  (One thread per output element walking the ranges one by one took 8.6 us for 32 heads of 32
// ranges and 6.3 us for 128 heads of 16, a chain of load latencies; with loads behind branches and a division in front this took 3.0 and
// 5.0, now 2.7 and 4.8.  Only the rounds that the ranges fill: steps of 6400 heads of two ranges of 100 keys, four rounds of loads for
// each / one, d = 64 16.8 / 14.4, d = 128 29.2 / 26.8.)
template <int D, bool DEALT>
__global__ __launch_bounds__(256) void decode_merge_kernel(const DecodeParams p) {
    constexpr int C4 = D / 4, NG = 256 / C4;
    __shared__ float xo[NG][D], xm[NG], xl[NG];
    const int h = blockIdx.x, b = blockIdx.y, row = b * p.Hq + h;
    const int c4 = threadIdx.x % C4, gr = threadIdx.x / C4;
    int first = b * p.n_splits, nb = p.n_splits;
    if (DEALT) {
        const Ranges rg = varlen_find(p, threadIdx.x & 63, -1, b);
        first = rg.first;
        nb = rg.nb;
    }
    const float* const pm0 = p.pm + (size_t)first * p.Hq + h;
    const float* const pl0 = p.lpart + (size_t)first * p.Hq + h;
    const float* const po0 = p.opart + ((size_t)first * p.Hq + h) * D + 4 * c4;
    float m = -INFINITY, l = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    // U rounds from range s0 on (every group makes them, and a load past the last range reads the last one again: no load sits behind a branch)
    auto rounds = [&](int s0, auto u_c) __attribute__((always_inline)) {
        constexpr int U = decltype(u_c)::value;
        float pm[U], pl[U];
        f32x4 po[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t at = (size_t)min(s0 + u * NG + gr, nb - 1) * p.Hq;
            pm[u] = pm0[at];
            pl[u] = pl0[at];
            po[u] = *reinterpret_cast<const f32x4*>(po0 + at * D);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = s0 + u * NG + gr < nb;
            pm[u] = live ? pm[u] : -INFINITY;
            pl[u] = live ? pl[u] : 0.f;
            po[u] = live ? po[u] : f32x4{0.f, 0.f, 0.f, 0.f};
        }
        float mn = m;
#pragma unroll
        for (int u = 0; u < U; ++u) mn = fmaxf(mn, pm[u]);
        const float msub = mn == -INFINITY ? 0.f : mn;
        const float a0 = __builtin_amdgcn_exp2f(m - msub);
#pragma unroll
        for (int u = 0; u < U; ++u) {  // (which product of the first two is rounded is spelled out: the same bits however many rounds there are)
            const float a = __builtin_amdgcn_exp2f(pm[u] - msub);
            l = u == 0 ? __builtin_fmaf(l, a0, a * pl[u]) : __builtin_fmaf(a, pl[u], l);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = u == 0 ? __builtin_fmaf(o[e], a0, a * po[u][e]) : __builtin_fmaf(a, po[u][e], o[e]);
        }
        m = mn;
    };
    using std::integral_constant;
    if (nb <= NG) rounds(0, integral_constant<int, 1>{});
    else if (nb <= 2 * NG) rounds(0, integral_constant<int, 2>{});
    else
        for (int s0 = 0; s0 < nb; s0 += 4 * NG) rounds(s0, integral_constant<int, 4>{});
    *reinterpret_cast<f32x4*>(&xo[gr][4 * c4]) = o;
    if (c4 == 0) { xm[gr] = m; xl[gr] = l; }
    __syncthreads();
    const int t = threadIdx.x;
    if (t >= D / 2) return;
    m = -INFINITY;
#pragma unroll
    for (int k = 0; k < NG; ++k) m = fmaxf(m, xm[k]);
    const float msub = m == -INFINITY ? 0.f : m;
    l = 0.f;
    float o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int k = 0; k < NG; ++k) {
        const float a = __builtin_amdgcn_exp2f(xm[k] - msub);
        l += a * xl[k];
        o0 += a * xo[k][2 * t];
        o1 += a * xo[k][2 * t + 1];
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    *reinterpret_cast<uint32_t*>(p.O + (size_t)row * D + 2 * t) = pack_bf16(o0 * inv, o1 * inv);
    if (p.LSE && t == 0) p.LSE[row] = l > 0.f ? (m + __builtin_amdgcn_logf(l)) * kLn2 : -INFINITY;
}

}  // namespace
