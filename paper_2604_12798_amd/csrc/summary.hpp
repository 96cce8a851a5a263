// Key-block summary pre-passes (sabsmax and the ablated representations).
#pragma once
#include "common.hpp"

namespace {

// ---------------------------------------------------------------------------------------------
// Key-block summary (Alg. 1, first loop): per dimension the element of largest magnitude of the block's keys with its
// sign, ties to the positive value.  HBM bound: K is read once.  One WAVE per key block, four blocks per workgroup:
// a lane owns one 16-byte chunk of every RG-th row, issues the loads of ROWS rows together, none behind a branch, reduces in registers,
// and the RG lanes of a chunk combine through lane exchanges: no LDS, no barrier, 256 bytes per lane in flight at d = 128 with ROWS = 64.
// A launch for a few blocks (a decode step's) is a chain of latencies: with eight predicated loads at a time and exchanges through the
// LDS unit it took 3.6 us for 8 blocks of 2048 keys' cache and 4.6 for 128 at d = 64, now 3.0 and 3.9 (an empty kernel takes 1.5);
// 4 x 8 heads of 32768 keys 5.0 / 4.8.
// Works on bf16 bit patterns, two to a dword: the key (magnitude << 1) | (sign ? 0 : 1) orders elements by magnitude
// and, at equal magnitude, puts the positive one on top, so the pick is an unsigned 16-bit maximum of keys.
typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
__device__ inline uint32_t sabs_key(uint32_t x) { return ((x << 1) & 0xfffefffeu) | ((~x >> 15) & 0x00010001u); }
__device__ inline uint32_t sabs_unkey(uint32_t k) { return ((k >> 1) & 0x7fff7fffu) | ((~k & 0x00010001u) << 15); }
__device__ inline uint32_t key_max(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

// max of keys with the lane 8, 16 or 32 further (which trades places with it)
template <int M>
__device__ __forceinline__ uint32_t key_max_across(uint32_t x) {
    if constexpr (M == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return key_max(r[0], r[1]);
    } else if constexpr (M == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return key_max(r[0], r[1]);
    } else {
        static_assert(M == 8, "rotations within rows of 16 lanes");
        return key_max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false));  // row_ror:8
    }
}

// N = row stride of one head's key array (its capacity), n_valid = keys present, Tc = block stride of
// one head's summary array.  bh and j are the same for all lanes; `live`: write the result.
template <int D, int ROWS = BN>
__device__ __forceinline__ void summary_of_block(const uint16_t* __restrict__ K, uint16_t* __restrict__ R, int bh, int j, int N,
                                                 int n_valid, int Tc, int block_n, int lane, bool live = true) {
    constexpr int CH = D / 8;        // 16-byte chunks per row
    constexpr int RG = 64 / CH;      // rows a wave reads at once
    constexpr int NL = ROWS / RG;    // such reads in flight
    const int ch = lane % CH, rg = lane / CH;
    const int c0 = j * block_n, c1 = min(n_valid, c0 + block_n);
    const uint8_t* base = reinterpret_cast<const uint8_t*>(K) + ((size_t)bh * N + c0) * (2 * D);
    const uint32_t zero_key = sabs_key(0u);  // +0: the smallest magnitude, already the positive one
    u32x4 acc = {zero_key, zero_key, zero_key, zero_key};
    for (int r0 = c0; r0 < c1; r0 += ROWS, base += ROWS * 2 * D) {
        u32x4 x[NL];
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            // (past the end the last row is read again, which changes no maximum: no load sits behind a branch.  Non-temporal: a
            // streaming read; 10 % faster at 64 MiB of keys, no change to the attention kernel behind it)
            const uint32_t r = (uint32_t)min(rg + u * RG, c1 - 1 - r0);
            x[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + (r * (2 * D) + ch * 16)));
        }
#pragma unroll
        for (int u = 0; u < NL; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = key_max(acc[e], sabs_key(x[u][e]));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if constexpr (CH == 8) acc[e] = key_max_across<8>(acc[e]);
        acc[e] = key_max_across<32>(key_max_across<16>(acc[e]));
    }
    if (rg == 0 && live) {
        const u32x4 out = {sabs_unkey(acc[0]), sabs_unkey(acc[1]), sabs_unkey(acc[2]), sabs_unkey(acc[3])};
        *reinterpret_cast<u32x4*>(R + ((size_t)bh * Tc + j) * D + ch * 8) = out;
    }
}

// Rows loaded together at d = 128: 64, but no more than a short block has, or than half of what its last round would read twice, and 16 where the
// rows are more than the memory-side cache holds: a stream from memory is the faster for fewer loads at once.  us with 64 / so: 4 x 8 heads of 32768 keys,
// blocks of 8 104 / 49, of 16 57 / 44, of 64 44.7 / 41.9, of 128 42.9 / 41.9, of 256 42.1 (16 rows 47.5); 4 x 8 of 4096, of 32 6.0 / 5.3, of 96 7.45 / 6.3, of 64 4.95 (16 rows
// 5.5); 3 x 8 of 16384, of 64 15.9 / 15.8, 6 x 8 of 16384, of 128 31.2 (16 rows 32.3).  (d = 64 reads 64 rows with eight loads: no length gains.)
__host__ __device__ inline bool many_rows(int block_n, long long rows) { return block_n <= 128 && rows > (block_n <= 64 ? 7 << 16 : 7 << 17); }
template <typename F>
__host__ inline void with_rows(int d, int block_n, long long rows, F launch) {
    using std::integral_constant;
    if (d == 64) launch(integral_constant<int, 64>{}, integral_constant<int, 64>{});
    else if (block_n <= 16) launch(integral_constant<int, 128>{}, integral_constant<int, 16>{});
    else if ((block_n - 1) % 64 < 32) launch(integral_constant<int, 128>{}, integral_constant<int, 32>{});
    else if (many_rows(block_n, rows)) launch(integral_constant<int, 128>{}, integral_constant<int, 16>{});
    else launch(integral_constant<int, 128>{}, integral_constant<int, 64>{});
}

// j0 = first block to (re)compute and n_blocks their number: a growing cache recomputes only the blocks that received keys.
template <int D, int ROWS>
__global__ __launch_bounds__(256) void kblock_summary_kernel(const uint16_t* __restrict__ K, uint16_t* __restrict__ R,
                                                             int N, int n_valid, int Tc, int block_n, int j0, int n_blocks) {
    // (a wave without a block does the last one again and writes nothing: no branch in front of the loads, whose latency is all there is of a
    // launch for a few blocks)
    const int lane = threadIdx.x & 63, jb = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    summary_of_block<D, ROWS>(K, R, blockIdx.y, j0 + min(jb, n_blocks - 1), N, n_valid, Tc, block_n, lane, jb < n_blocks);
}

// With per-sequence lengths (device arrays indexed by batch entry, Hkv heads each) the host does not know which blocks received
// keys.  The kernel counts them, and its waves walk the list of them in order of memory, a block at a time: reads bound it when
// there is much to do, a launch and the count when there is little.
// E = 1, 4: up to 64 E entries, E in each lane of every wave.  E = 0: more; the entries are dealt out to the threads of a workgroup,
// and two levels of sums in LDS lead to the thread that has an item's entry (16 waves to a workgroup, as each counts the batch).
// Before: one wave for every block of the capacity, most of them with nothing to do, then a fixed number of waves for every head,
// most of them idle where the heads have different numbers of blocks.  In us (first / second / now), d = 128, 8 KV heads:
//   a new key in each of 128 caches of 8192 rows 44 / 3.7 / 4.7; 32768 new rows in one of 128 and a key in the others 96 / 285 / 14;
//   in every fourth 368 / 710 / 392; in all 1424 / 1521 / 1501 (waves that stay lose the order of memory, a wave for each block keeps it)
constexpr int APPEND_WAVES = 8192;  // eight to a SIMD
template <int D, int ROWS, int E>
__global__ __launch_bounds__(E ? 256 : 1024) void kblock_summary_varlen_kernel(const uint16_t* __restrict__ K, uint16_t* __restrict__ R,
                                                                               int B, int Hkv, int N, int Tc, int block_n,
                                                                               const int* __restrict__ old_len,
                                                                               const int* __restrict__ new_len, int n_wg) {
    constexpr int NW = E ? 4 : 16, T = 64 * NW, C = E ? E : 1;
    __shared__ int upto[E ? 1 : T], wave_upto[16];  // blocks of one head: of the entries of the threads, of the waves up to one
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int j0[C], n_valid[C], n[C], up[C];  // of entries in each lane: first block, keys, number of blocks, the same up to the entry
    auto look_at = [&](int b, int e) __attribute__((always_inline)) {
        n[e] = j0[e] = n_valid[e] = 0;
        if (b < B) {
            n_valid[e] = min(max(new_len[b], 0), N);
            j0[e] = min(max(old_len[b], 0), n_valid[e]) / block_n;
            n[e] = (n_valid[e] + block_n - 1) / block_n - j0[e];
        }
    };
    int total = 0;
    if (E) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            look_at(64 * e + lane, e);
            up[e] = total + wave_prefix(n[e]);
            total = __builtin_amdgcn_readlane(up[e], 63);
        }
    } else {
        int own = 0;
        for (int b = threadIdx.x; b < B; b += T) {
            look_at(b, 0);
            own += n[0];
        }
        const int sum = wave_prefix(own);
        if (lane == 63) wave_upto[wave] = sum;
        __syncthreads();
        const int waves_upto = wave_prefix(lane < NW ? wave_upto[lane] : 0);
        __syncthreads();
        const int before = wave ? __builtin_amdgcn_readlane(waves_upto, wave - 1) : 0;
        upto[E ? 0 : threadIdx.x] = before + sum;
        if (lane == 63) wave_upto[wave] = before + sum;
        __syncthreads();
        total = __builtin_amdgcn_readlane(waves_upto, NW - 1);
    }
    total *= Hkv;
    const bool many = many_rows(block_n, (long long)total * block_n);
    for (int item = blockIdx.x * NW + wave; item < total; item += n_wg * NW) {
        int bh = 0, j = 0, nv = 0;
        // the item's entry: b0 + l * stride, l the first lane whose sum lies behind the item
        auto found = [&](int e, int b0, int stride) __attribute__((always_inline)) {
            const int l = __builtin_ctzll(__builtin_amdgcn_ballot_w64(item < up[e] * Hkv) | (1ull << 63));
            const int nb = __builtin_amdgcn_readlane(n[e], l), rem = item - (__builtin_amdgcn_readlane(up[e], l) - nb) * Hkv, h = rem / nb;
            bh = (b0 + l * stride) * Hkv + h;
            j = __builtin_amdgcn_readlane(j0[e], l) + (rem - h * nb);
            nv = __builtin_amdgcn_readlane(n_valid[e], l);
        };
        if (E) {
            bool done = false;
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (!done && item < __builtin_amdgcn_readlane(up[e], 63) * Hkv) {
                    found(e, 64 * e, 1);
                    done = true;
                }
        } else {
            const int w = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < NW && wave_upto[lane & (NW - 1)] * Hkv <= item));
            const int t = 64 * w + __builtin_popcountll(__builtin_amdgcn_ballot_w64(upto[E ? 0 : (64 * w + lane) & (T - 1)] * Hkv <= item));
            look_at(t + lane * T, 0);  // (the thread's entries, one to a lane: no more than 64 of a batch of at most 65535)
            up[0] = (t ? upto[E ? 0 : t - 1] : 0) + wave_prefix(n[0]);
            found(0, t, T);
        }
        if (D == 128 && ROWS == 64 && many) summary_of_block<D, 16>(K, R, bh, j, N, nv, Tc, block_n, lane);
        else summary_of_block<D, ROWS>(K, R, bh, j, N, nv, Tc, block_n, lane);
    }
}

// The three ablated block representations (ablation of the k_repr construction): per dimension the
// maximum (mode 1), the mean (mode 2: fp32 sum in a fixed order, rounded to bf16) or the largest
// magnitude without its sign (mode 3).  Not on the hot path: one thread per (row group, 8 dims).
template <int D>
__global__ __launch_bounds__(256) void kblock_summary_alt_kernel(const uint16_t* __restrict__ K, uint16_t* __restrict__ R,
                                                                 int N, int Tc, int block_n, int mode) {
    constexpr int CH = D / 8;
    constexpr int RG = 256 / CH;
    __shared__ float part[RG][D];
    const int j = blockIdx.x, bh = blockIdx.y;
    const int ch = threadIdx.x % CH, rg = threadIdx.x / CH;
    const int c0 = j * block_n, c1 = min(N, c0 + block_n);
    const uint16_t* base = K + (size_t)bh * N * D;
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = mode == 1 ? -INFINITY : 0.f;
    for (int r = c0 + rg; r < c1; r += RG) {
        const u32x4 x = *reinterpret_cast<const u32x4*>(base + (size_t)r * D + ch * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = __uint_as_float(((x[e >> 1] >> (16 * (e & 1))) & 0xffffu) << 16);
            acc[e] = mode == 1 ? fmaxf(acc[e], v) : (mode == 2 ? acc[e] + v : fmaxf(acc[e], fabsf(v)));
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) part[rg][ch * 8 + e] = acc[e];
    __syncthreads();
    if (rg == 0) {
        const int nrg = min(RG, c1 - c0);  // row groups that saw at least one row
        uint32_t out[4];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float a = acc[e];
            for (int q = 1; q < nrg; ++q) {
                const float v = part[q][ch * 8 + e];
                a = mode == 2 ? a + v : fmaxf(a, v);
            }
            if (mode == 2) a /= (float)(c1 - c0);
            const uint32_t bits = pack_bf16(a, 0.f) & 0xffffu;
            out[e >> 1] = (e & 1) ? (out[e >> 1] | (bits << 16)) : bits;
        }
        *reinterpret_cast<u32x4*>(R + ((size_t)bh * Tc + j) * D + ch * 8) = u32x4{out[0], out[1], out[2], out[3]};
    }
}

}  // namespace
