// C ABI of libvfa.so (declared in vfa.h): argument checks, kernel selection and launches.  The kernels live in the
// headers included below and are compiled for gfx950 in this translation unit, except attn_vsa_pp_kernel (vsa_pp.hip).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>
#include <atomic>

#include "vfa.h"

#include "common.hpp"
#include "attn_generic.hpp"
#include "attn_pingpong.hpp"
#include "attn_frozen.hpp"
#include "attn_short.hpp"
#include "attn_sparse.hpp"
#include "vsa_pp.hpp"
#include "summary.hpp"
#include "decode.hpp"
#include "fp8.hpp"
#include "mx4.hpp"

namespace {

// ---------------------------------------------------------------------------------------------
// host side
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Workgroups of 256 threads that one launch can have: of 2^32 work-items or more HIP runs a part, without an error
constexpr long long kMaxWorkgroups256 = (1LL << 24) - 1;

int check_common(const void* Q, const void* K, const void* V, void* O, const float* LSE, int B, int Hq, int Hkv,
                 int N, int d, int block_m, int block_n) {
    if (B < 0 || N < 0 || Hq <= 0 || Hkv <= 0 || d <= 0 || block_m <= 0 || block_n <= 0) return VFA_ERR_INVALID_ARG;
    if (Hq % Hkv != 0) return VFA_ERR_INVALID_ARG;
    if (d != 64 && d != 128) return VFA_ERR_UNSUPPORTED;
    if (!(block_n == 64 && (block_m == 64 || block_m == 128))) return VFA_ERR_UNSUPPORTED;
    if (B == 0 || N == 0) return VFA_OK;
    if (!Q || !K || !V || !O) return VFA_ERR_INVALID_ARG;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O)) return VFA_ERR_INVALID_ARG;
    if (LSE && (reinterpret_cast<uintptr_t>(LSE) & 3u)) return VFA_ERR_INVALID_ARG;
    const long long wgs = (long long)B * Hq * ceil_div(N, block_m);
    if (wgs > 0x7fffffffLL || (long long)B * Hq * N > 0x7fffffffLL) return VFA_ERR_UNSUPPORTED;
    return VFA_OK;
}

// Host-side caches.  Everything the library remembers between calls is a per-device fact that any thread would
// compute to the same value (a CU count, "this kernel's LDS limit has been raised", the address of the device
// array below), held in atomics: two threads that race on a first call both do the lookup and store the same thing.
constexpr int kMaxDevices = 64;

int current_device() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return -1;
    return dev;
}

// number of compute units of the current device (0 if the query fails), looked up once per device
int cu_count() {
    static std::atomic<int> cached[kMaxDevices];
    const int dev = current_device();
    if (dev < 0) return 0;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = -1;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n > 0 ? n : 0;
}

// Opt the kernels that need more than 64 KiB of LDS in to it: all of them on the first attention call on a device, whatever call
// that is, so that no later one, which may be a captured one, has to (idempotent, so a race only repeats it).
template <typename KernelT>
bool raise_lds_limit(KernelT kernel, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
}
template <int D, int KS>
bool raise_frozen() {
    return raise_lds_limit(&attn_fwd_frozen_kernel<D, KS, false>, Frozen<D, KS>::LDS_BYTES) &&
           raise_lds_limit(&attn_fwd_frozen_kernel<D, KS, true>, Frozen<D, KS>::LDS_BYTES);
}
template <int D, int KQ>
bool raise_short() { return raise_lds_limit(&attn_fwd_short_kernel<D, KQ>, Short<D, KQ>::LDS_BYTES); }
template <int MODE>
bool raise_pp() {
    return raise_lds_limit(&attn_fwd_pp_kernel<MODE, false>, pp_lds_bytes<false>()) &&
           raise_lds_limit(&attn_fwd_pp_kernel<MODE, true>, pp_lds_bytes<true>());
}
bool raise_lds_limits() {
    static std::atomic<unsigned char> done[kMaxDevices];
    const int dev = current_device();
    if (dev < 0) return false;
    if (done[dev].load(std::memory_order_acquire)) return true;
    if (!raise_short<64, 2>() || !raise_short<64, 4>() || !raise_short<128, 2>() || !raise_short<128, 4>()) return false;
    if (!raise_lds_limit(&attn_sparse_kernel, Sparse::LDS_BYTES)) return false;
    if (!raise_frozen<64, 1>() || !raise_frozen<64, 2>() || !raise_frozen<128, 2>() || !raise_pp<MODE_VFA>() || !raise_pp<MODE_FA>() ||
        !raise_pp<MODE_FA_LAZY>() || !raise_pp<MODE_FA_SOFTEXP>() || vfa_detail_vsa_pp_raise_lds() != 0)
        return false;
    done[dev].store(1, std::memory_order_release);
    return true;
}
// rows [row_base, N) of every head; `summaries`: with the workgroups that write them to p.Krepr
template <int D, int KQ>
int launch_short(Params p, int row_base, bool summaries, hipStream_t s) {
    p.row_base = row_base;
    p.Tr = ceil_div(p.N - row_base, 64);
    p.n_items = p.B * p.Hq * p.Tr;
    // KV heads that are no multiple of eight.  In one order for all, an XCD meets every head that is its number mod 8 in the workgroups' order, and reads
    // their keys in turn: lists for the eights where those are more than its L2 (4 MB) holds together.  Causal calls otherwise keep the one order, since
    // long items of a list's later KV heads start behind the short ones of its first.  us, one order / lists: d = 128, causal, 144 heads over
    // 36, N = 2204 278 / 207, 98 heads, N = 2560 405 / 193, no mask, 141 over 47, N = 1407 313 / 160; d = 64, causal, 174 over 87, N = 1024 73 / 41;
    // 2 and 5 MB: d = 128, 40 over 20, N = 698 12.2 / 14.6, d = 64, 136 over 34, N = 1090 33.8 / 37.4.  1200 shapes: in the mean 0.3 % over the faster one at d = 128, 0.6 at
    // d = 64, lines of 4 MB 0.5 and 1.1
    const int heads = p.B * p.Hq, met = min(p.B * p.Hkv, ceil_div(heads, heads & 1 ? 1 : heads & 2 ? 2 : heads & 4 ? 4 : 8));  // (KV heads an XCD meets)
    set_items(p, !p.causal || (double)met * p.N * 4 * D > (D == 128 ? 2.5e6 : 6e6));
    const long long wgs = p.n_items + (summaries ? ((long long)p.B * p.Hkv * p.Tc + 2 * KQ - 1) / (2 * KQ) : 0);
    attn_fwd_short_kernel<D, KQ><<<dim3((unsigned)wgs), 128 * KQ, Short<D, KQ>::LDS_BYTES, s>>>(p);
    return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
}
template <int D, int KS>
int launch_frozen(Params p, int row_base, int block_m, hipStream_t s) {  // rows [row_base, N) of every head
    p.row_base = row_base;
    p.Tr = ceil_div(p.N - row_base, 128);
    const dim3 grid((unsigned)(p.B * p.Hq * p.Tr));
    if (block_m == 64 && p.causal) attn_fwd_frozen_kernel<D, KS, true><<<grid, 256 * KS, Frozen<D, KS>::LDS_BYTES, s>>>(p);
    else attn_fwd_frozen_kernel<D, KS, false><<<grid, 256 * KS, Frozen<D, KS>::LDS_BYTES, s>>>(p);
    return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
}

// The ping-pong kernel under a causal mask, with a list of items for each XCD (KV heads in eights): the tiles of its busiest workgroup over the
// average.  A workgroup takes one item of each round, the rounds in alternating directions (attn_pingpong.hpp), so an XCD's only KV head, or
// whole KV heads to a round, even out, and a long item of a later KV head on top of other long ones does not.  Four tiles for an
// item's start and end; 1 beyond 16 rounds, where little is left of it.
double pp_unevenness(const Params& p, bool head_pairs, int n_cu) {
    const int g = p.Hq / p.Hkv, units = head_pairs ? g / 2 : g, rows = head_pairs ? 128 : 256, Ti = ceil_div(p.N, rows);
    const int slots = n_cu / 8;
    const long long len = (long long)p.B * p.Hkv / 8 * units * Ti;
    constexpr int MAX_SLOTS = 64;
    if (slots < 1 || slots > MAX_SLOTS || len <= slots || len > 16LL * slots) return 1.0;
    int load[MAX_SLOTS] = {}, at = 0, step = 1, most = 0;  // (the slot of the next item; a round ends where it would leave the slots)
    long long all = 0;
    for (long long y = 0; y < len;) {
        for (int i = Ti; i > 0 && y < len; --i) {
            const int tiles = ceil_div(min(p.N, i * rows), BN) + 4;
            for (int u = 0; u < units; ++u, ++y) {
                most = max(most, load[at] += tiles);
                all += tiles;
                if (at + step < 0 || at + step >= slots) step = -step;
                else at += step;
            }
        }
    }
    return (double)most * slots / all;
}

// Alg. 1 on the kernel for short sequences (attn_short.hpp): 0 = no, else its groups of keys.  `items` are blocks of 64 rows, `rounds` those of
// the other kernels' items (two blocks of 128 rows at d = 128).  Its items are a quarter as long as the ping-pong kernel's, need no launch for the
// summaries and start alone, so it wins on few tiles, on few items and where the others' rounds are poorly filled; in full rounds of long items
// those are 1.05 to 1.15 times faster.  The lines lie where they meet.  6900 shapes of 7 to 96 tiles, 3 to 580 heads, any number to a KV head, against neither,
// two and four groups: in the mean 0.4 % over the fastest.  Slower than without it by more than 3 %: 45, by more than 5 %: ten, the worst of them d = 128, causal, 512
// heads, N = 1266 1.08, 21 heads, N = 4519 1.08, 24 heads, N = 4096 1.06 and d = 64, 44 heads, N = 3644 1.07.  us, theirs / this one:
//   four groups, from ten tiles on, for no more items than units (at d = 128 the summaries' workgroups counted, since one fills a
//     unit), against two: d = 128, 4 heads, N = 4096 35.3 / 29.9, 8 heads, N = 1024 12.3 / 11.5; causal, few long heads, whose items are uneven: up to
//     four per unit at d = 64 (12 heads, N = 4096 35.5 / 34.3), 1.9 at d = 128 (8 heads, N = 3600 39.8 / 35.5; 16 heads, N = 1536 18.5 / 18.0); d = 64, no
//     mask, long ones, up to two per unit (4 heads, N = 6144 neither 57.0, two 59.8, four 55.0)
//   d = 64, causal: any with 8 items per unit (32 heads, N = 5541, 11 per unit 168 / 156), 57 tiles with 16 (44 heads, N = 3644 1.07 times slower, 64 heads, N =
//     3735 163.5 / 150.6), 46 beyond (256 heads, N = 2361 259 / 239, 512 heads, N = 2560 0.96)
//   d = 64, no mask: four items per unit, any tiles, or 48 where they fill their rounds to within a quarter; eight, 48 or 26; 32 or 20 beyond
//     (40 heads over 10, N = 3072 0.97, 256 heads, N = 1536 0.97, 209 heads, N = 1820 239 / 215)
//   d = 128, causal, KV heads in eights: by how uneven the ping-pong kernel's workgroups come out (pp_unevenness), the less the more tiles.  Even
//     groups of heads: 64 over 8, N = 2048 (1.0) 76.8 / 80.8, 32 over 8, N = 3328 (1.1) 93.6 / 100.7, 32 over 16, N = 3328 (1.8) 129.8 / 100.2; 64 over 16, N = 3600 246 / 225; odd ones,
//     whose items cover two diagonals: 128 heads, N = 2048 162 / 170, N = 3072 320 / 346, 24 heads, N = 5000 218 / 171, 48 heads, N = 5632 381 / 401
//   d = 128, causal, other numbers of KV heads, whose list for the whole chip starts with all long items: 88 tiles with 1.5 rounds, 34 to 14 with
//     more (36 heads over 9, N = 2254 62.7 / 57.8), odd groups 90, 52 to 38 (126 over 42, N = 2048 165 / 158, N = 3077 1.06 times faster and not taken)
//   d = 128, no mask: rounds filled to within a quarter 18 tiles (128 heads over 32, N = 1536 147 / 154), others 72 to 14, the more rounds the fewer (12 over 4, N =
//     2062 39.6 / 34.8; 48 heads, N = 1800 104 / 90; 74 over 37, N = 1920 169 / 151)
//   more than four sink or local blocks: never
int short_groups(const Params& p, int d, int n_cu) {
    const long long heads = (long long)p.B * p.Hq, items = heads * p.Tc;  // (of 64 rows)
    if (n_cu <= 0 || p.n_sink > 4 || p.n_local > 4 || p.Tc > 96) return 0;
    if (items + ((long long)p.B * p.Hkv * p.Tc + 3) / 4 > kMaxWorkgroups256) return 0;  // (with the summaries' workgroups; four groups are for few items)
    const int Tc = p.Tc, g = p.Hq / p.Hkv, kv_heads = p.B * p.Hkv, blocks = ceil_div(p.N, 128);
    const double per_cu = (double)items / n_cu;
    const bool few_heads = p.causal && 16 * heads <= n_cu;
    if (d == 64) {
        if (Tc >= 10 && (per_cu <= 1 || (few_heads && per_cu <= 4) || (!p.causal && Tc >= 48 && per_cu <= 2))) return 4;
        if (p.causal) return Tc <= (per_cu <= 8 ? 96 : per_cu <= 16 ? 57 : 46) ? 2 : 0;
        const double rounds = (double)(heads * blocks) / (2 * n_cu);
        const bool full = ceil(rounds) - rounds < 0.25;
        return Tc <= (per_cu <= 4 ? (full ? 48 : 96) : per_cu <= 8 ? (full ? 26 : 48) : (full ? 20 : 32)) ? 2 : 0;
    }
    const long long summary_wgs = ((long long)kv_heads * Tc + 7) / 8;
    if (Tc >= 10 && Tc <= 64 && (items + summary_wgs <= n_cu || (few_heads && Tc >= 16 && per_cu <= 1.9))) return 4;
    const bool even = (g & 1) == 0;  // (pairs of heads, else of blocks)
    const double rounds = (double)(even ? heads / 2 * blocks : heads * ((blocks + 1) / 2)) / n_cu, idle = ceil(rounds) - rounds;
    int upto;
    if (!p.causal) {
        if (idle < 0.25) upto = rounds < 6 ? 18 : 10;
        else upto = rounds < 0.5 ? 72 : rounds < 0.75 ? 42 : rounds < 2 ? 34 : rounds < 4 ? 28 : rounds < 6 ? 20 : 14;
    } else if (rounds <= 1.2) {
        upto = 96;
    } else if ((kv_heads & 7) == 0) {
        const double uneven = log(pp_unevenness(p, even, n_cu));
        if (even) return uneven > 0.40 - (rounds < 5 ? 11.5 : rounds < 8 ? 8 : 6) / Tc ? 2 : 0;
        return uneven > 0.32 - (rounds < 5 || rounds >= 8 ? 10 : 7.5) / Tc ? 2 : 0;
    } else if (even) {
        upto = rounds <= 1.5 ? 88 : rounds < 5 ? 34 : rounds < 8 ? 30 : rounds < 12 ? 22 : 14;
    } else {
        upto = rounds <= 1.5 ? 90 : rounds < 4 ? 52 : rounds < 8 ? 46 : 38;
    }
    return Tc <= upto ? 2 : 0;
}

// Without a causal mask all items are equally long, and what is left of them after whole rounds of the ping-pong kernel takes as long
// as a round: the first row of that rest, which then runs on a kernel of finer items (a head's last rows: no more than one item per
// compute unit, of 64 rows with the keys split four ways, attn_short.hpp, else, where the items are long, of 128 rows, attn_frozen.hpp), or 0.
// In us, before / after: 16 heads, N = 5000 (one round and 904 rows) 222 / 197; 24 heads, N = 3000 141 / 119; 32 heads, N = 3000
// (rest on attn_frozen.hpp) 149 / 144; 48 heads, N = 1751 96 / 101 with that, so only above 32 tiles.
int tail_row(const Params& p, int n_cu, bool head_pairs) {
    if (p.causal || p.n_sink > 4 || p.n_local > 4 || n_cu <= 0 || p.Tc <= 12 || p.N > 1 << 23) return 0;  // (the last: attn_short.hpp's offsets)
    const long long heads = (long long)p.B * p.Hq, per_band = head_pairs ? heads / 2 : heads;  // items of `band` rows
    const int band = head_pairs ? 128 : 256;
    const long long rounds = per_band * ceil_div(p.N, band) / n_cu, bands = rounds * n_cu / per_band, rows = bands * band;
    if (rounds == 0 || rows >= p.N || 10 * bands * per_band < 9 * rounds * n_cu) return 0;
    const int rest = p.N - (int)rows;
    return heads * ceil_div(rest, 64) <= n_cu || (p.Tc > 32 && heads * ceil_div(rest, 128) <= n_cu) ? (int)rows : 0;
}

// Which kernel Alg. 1's calls that are not short ones run on at d = 128: true = attn_frozen.hpp (items of 128 rows, a third to a half cheaper than the
// ping-pong kernel's items of 256), false = attn_pingpong.hpp (one and a half times the rate once the compute units are full).
//   up to one 128-row item per compute unit: the ping-pong kernel would leave half of them idle (us, ping-pong / frozen: 32 heads, N =
//     1024 31.7 / 24.6; most such calls are short ones by now)
//   two to 2.9 per compute unit, all equally long (no causal mask) and of more than twelve tiles: three rounds of short items
//     against two of long ones (16 heads, N = 5000 241 / 227).  Where the third round is nearly full or the items are short it is
//     the other way round (256 heads, N = 300 38.2 / 42.5; 32 heads, N = 3000 155 / 160; 160 heads, N = 512 47 / 49.5).  Between
//     one and two it is two rounds against one (N = 3072: 89 against 76 us), above three four against two, and under a causal mask
//     the ping-pong kernel's long items find short ones to pair with
//   many sink / local blocks: their scores are computed twice in attn_frozen.hpp
bool prefer_frozen(const Params& p, int n_cu, bool has_tail) {
    const long long items = (long long)p.B * p.Hq * p.Tr;
    if (p.n_sink > 4 || p.n_local > 4 || n_cu <= 0) return false;
    return items <= n_cu || (!p.causal && p.Tc > 12 && items > 2LL * n_cu && 10 * items <= 29LL * n_cu && !has_tail);
}

// Calls with block_m = 64 and without skipping, d = 128, that are not short ones (`p` in blocks of 128 rows): true = items of 64 rows on the generic
// kernel, two to a compute unit, false = blocks of 128 rows.  The short items run at 50 to 80 % of the rate, waste fewer rows and
// take less to start, which is more for short sequences only (generic / other us):
//   Alg. 1, one round of at most four tiles (32 heads, N = 64 9.6 / 10.7, N = 256 14.3 / 14.8; N = 300 15.4 / 15.1).  With
//     `frozen` (the other choice is attn_frozen.hpp) and no more than one of its items per compute unit, only there
//   no causal mask, up to 14 tiles, where they need no more rounds (the baseline, 96 heads, N = 777 54.9 / 59.3; two rounds
//     against one, N = 512 37 / 24; 16 tiles, 32 heads 35.0 / 33.2)
//   under a causal mask, which evens out the rounds: Alg. 1 up to ten tiles and one and a quarter rounds (96 heads, N = 320 19.7 /
//     22.1; two rounds, N = 640 46.0 / 47.6 and 64 heads, N = 1024 43 / 36), the baselines, which have no max to find in front, up to
//     16 and two and a half (128 heads, N = 384 17.1 / 21.8; 96 heads, N = 777 40.9 / 45.4, N = 1024 57.5 / 47.4)
// 645 shapes of each, against the generic kernel alone: slower by more than 2 % are Alg. 1, causal, 96 heads, N = 640 to 768 (3.5
// to 6.3 %) and 72 heads, N = 777 (6.7 %), and the baseline, 128 heads, N = 700 (10 %); the mean is 27 and 13 % faster.  (Alg. 1's of
// four tiles, and its causal ones, are those with many sink or local blocks and vfa_variant_fwd's: the rest are short ones by now.)
bool prefer_rows64(const Params& p, int n_cu, bool head_pairs, bool frozen, bool baseline) {
    if (n_cu <= 0) return false;
    const long long heads = (long long)p.B * p.Hq, items = heads * p.Tc, slots = 2LL * n_cu;
    if (!baseline && p.Tc <= 4) return items <= slots;
    if (frozen && heads * p.Tr <= n_cu) return false;
    if (p.causal) return baseline ? p.Tc <= 16 && 2 * items <= 5 * slots : p.Tc <= 10 && 4 * items <= 5 * slots;
    const long long pairs = head_pairs ? heads / 2 * p.Tr : heads * ((p.Tr + 1) / 2);
    return p.Tc <= 14 && (items + slots - 1) / slots <= (pairs + n_cu - 1) / n_cu;
}

// Alg. 2 at d = 128, block_m = 128 runs on attn_sparse_kernel where a block meets enough tiles for what that one does before its main
// loop: the scores of every sink and local block but tile 0, which the loop takes again.  us on the other kernels / there:
//   one sink and one local block (two such tiles): 32/8 heads, N = 256 15.2 / 15.4, 512 21.5 / 20.4, 2048 67 / 58, 8000 555 / 502;
//   four and four (eight): 32/8 heads, N = 512 22.8 / 24.5, 777 30.2 / 31.0, 2048 66.8 / 65.9, 4096 174 / 163, 32768 (8 heads) 2231 / 1935;
//   none: N = 256 14.5 / 13.3, 512 20.6 / 18.2;
// with several items to a workgroup's place the other kernel hides its own ends, and it takes a longer loop: 128/8 heads, N = 1024, one
// and one 64.2 / 65.4, four and four 65.7 / 74.8; 64/8 heads, N = 4096, four and four 316.6 / 315.9.
// 1500 shapes of 2 to 300 tiles, up to 4 and 4 blocks, 0 to 90 % dropped: masks are the same on all; 0.91 to 0.97 of the other kernels' time in the mean; slower by more than 3 % are three
// (118 heads over 59, N = 1536 111.5 / 116.3, 99 over 33, N = 1536 94.6 / 98.1, 110 over 55, N = 2056 191 / 198).
bool prefer_sparse(const Params& p, int n_cu) {
    const long long items = (long long)p.B * p.Hq * p.Tr;
    if (p.n_sink > 4 || p.n_local > 4 || items > kMaxWorkgroups256 || p.N > 1 << 23) return false;  // (its LDS; a launch; 32-bit offsets)
    const int again = (p.n_sink > 1 ? p.n_sink - 1 : 0) + (p.n_local > 0 ? p.n_local + 1 : 0);
    return (p.causal ? p.Tc + 2 : 2 * p.Tc) >= (items > 2 * n_cu ? 10 : 4) * again;  // (twice a block's tiles, on average)
}

// Otherwise (more than four sink or local blocks, above all): the generic kernel up to this many tokens (causal; half as many
// non-causal), the ping-pong kernel above.  In the generic kernel a workgroup drops a tile alone (the ping-pong kernel's interval
// is short only where both of its groups drop theirs), and the ends of a work item cost no more than its middle; the ping-pong
// kernel's steps overlap better and don't fetch V for a dropped tile.  Generic / ping-pong us, 32/8 heads, 20 to 40 % of the tiles
// dropped: N = 8000 511 / 560, 10000 784 / 847, 16384 1863 / 1884, 64K (8 heads) 7147 / 6290; with nothing dropped 8000 583 / 614,
// 10000 881 / 919, 12200 1262 / 1268, 16384 2262 / 2169; 8/1 heads 10000 268 / 290, 16384 515 / 493; with 98 % dropped 10200
// 535 / 532; four batches of N = 8000 1901 / 2386.  Non-causal: N = 4096 264 / 286, 5000 395 / 454, 6100 547 / 550, nothing dropped
// 655 / 643.
constexpr int VSA_GENERIC_MAX_N = 10240;

// `fixed_max`: Alg. 1 as written on all rows (no kernel that takes every block's scores into the max)
template <int MODE>
int launch_fwd(const Params& p, int d, int block_m, hipStream_t s, bool fixed_max = false) {
    (void)hipGetLastError();
    if (!raise_lds_limits()) return VFA_ERR_HIP;
    const int g = p.Hq / p.Hkv;
    const bool ablation = p.order_asc || p.all_special || p.rowskip || p.Qrepr || (MODE == MODE_VSA && p.tau2 >= 0.f);
    // ping-pong kernel: head pairs when the heads per KV head are even; otherwise (MHA, odd groups) pairs of
    // adjacent query blocks; for VSA only where each block still meets its tiles in Alg. 2's order
    // (causal, at most one local block), since the skip decisions depend on the max at the time of the visit
    const bool head_pairs = (g & 1) == 0;
    // Without skipping, block_m decides only which blocks count as local ones, and a larger set of exact-max blocks is as good:
    // nearly everything runs in blocks of 128 rows then (d = 128 in blocks of 64, N = 4096: 219 us on the generic kernel, 131 here)
    Params q = p;
    if (MODE != MODE_VSA && !ablation) q.Tr = ceil_div(p.N, 128);
    bool rows64 = false;
    int tail = 0;  // rows [0, tail) run on the ping-pong kernel, those behind them on another one
    if constexpr (MODE == MODE_VFA) {
        if (!ablation && d == 64 && p.n_sink <= 4 && p.n_local <= 4) {
            // two groups to an item while there is no more than one item per compute unit (32 heads, N = 777: 12.4 against 13.6 us;
            // N = 4096: 95 against 87)
            const long long items = (long long)q.B * q.Hq * q.Tr;
            if (items <= cu_count()) return launch_frozen<64, 2>(q, 0, block_m, s);
            // (more than one launch can have: the generic kernel, whose workgroups have half as many threads at block_m = 64)
            if (items <= kMaxWorkgroups256) return launch_frozen<64, 1>(q, 0, block_m, s);
        }
        if (!ablation && d == 128) {
            if (!fixed_max) tail = tail_row(q, cu_count(), head_pairs);
            const bool frozen = prefer_frozen(q, cu_count(), tail > 0);
            rows64 = block_m == 64 && prefer_rows64(q, cu_count(), head_pairs, frozen, false);
            if (frozen && !rows64) return launch_frozen<128, 2>(q, 0, block_m, s);
            if (rows64) tail = 0;
        }
    }
    if constexpr (MODE == MODE_VSA) {
        if (!ablation && d == 128 && block_m == 128 && prefer_sparse(p, cu_count())) {
            set_items(q, false);  // (lists for the eights of KV heads: 1.01 times slower in the mean of 500 shapes, 142 heads, N = 500 34.4 / 53.2 us)
            attn_sparse_kernel<<<dim3((unsigned)(p.B * p.Hq * p.Tr)), 256, Sparse::LDS_BYTES, s>>>(q);
            return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
        }
    }
    if constexpr (is_fa(MODE)) {
        rows64 = d == 128 && block_m == 64 && prefer_rows64(q, cu_count(), head_pairs, false, true);
    }
    if (d == 128 && (block_m == 128 || MODE != MODE_VSA) && !ablation && !rows64 &&
        (MODE != MODE_VSA || (p.N > (p.causal ? VSA_GENERIC_MAX_N : VSA_GENERIC_MAX_N / 2) && (head_pairs || (p.causal && p.n_local <= 1))))) {
        q.pair_blocks = head_pairs ? 0 : 1;
        if (tail) q.Tr = tail / 128;
        unsigned n_wg = (unsigned)(head_pairs ? q.B * (q.Hq / 2) * q.Tr : q.B * q.Hq * ((q.Tr + 1) / 2));
        // One workgroup fills a CU (128 KiB of LDS), so with more work items than CUs the kernel runs one
        // persistent workgroup per CU over a static share of the items: the next item starts without a
        // workgroup launch (worth about 1 % at N = 16K and 30 % at N = 4K, measured).
        const int n_cu = cu_count();
        if (n_cu > 0 && (n_cu & 7) == 0 && n_wg > (unsigned)n_cu) {
            q.persist = n_cu;
            n_wg = (unsigned)n_cu;
        }
        if constexpr (MODE == MODE_VSA) {
            return vfa_detail_vsa_pp_launch(&q, sizeof(q), n_wg, s) == 0 ? VFA_OK : VFA_ERR_HIP;
        } else {
            if (block_m == 64 && p.causal) attn_fwd_pp_kernel<MODE, true><<<dim3(n_wg), 512, pp_lds_bytes<true>(), s>>>(q);
            else attn_fwd_pp_kernel<MODE, false><<<dim3(n_wg), 512, pp_lds_bytes<false>(), s>>>(q);
            if (hipGetLastError() != hipSuccess) return VFA_ERR_HIP;
            if constexpr (MODE == MODE_VFA) {
                if (tail && (long long)p.B * p.Hq * ceil_div(p.N - tail, 64) <= n_cu) return launch_short<128, 4>(p, tail, false, s);
                if (tail) return launch_frozen<128, 2>(p, tail, block_m, s);
            }
            return VFA_OK;
        }
    }
    const dim3 grid((unsigned)(p.B * p.Hq * p.Tr));
    if ((long long)p.B * p.Hq * p.Tr > kMaxWorkgroups256 * 128 / block_m) return VFA_ERR_HIP;  // (two threads to a row of a block)
    if constexpr (MODE == MODE_VSA) {
        if (!ablation) {
            if (d == 128 && block_m == 128) attn_fwd_kernel<128, 4, MODE, true><<<grid, 256, 0, s>>>(p);
            else if (d == 128 && block_m == 64) attn_fwd_kernel<128, 2, MODE, true><<<grid, 128, 0, s>>>(p);
            else if (d == 64 && block_m == 128) attn_fwd_kernel<64, 4, MODE, true><<<grid, 256, 0, s>>>(p);
            else if (d == 64 && block_m == 64) attn_fwd_kernel<64, 2, MODE, true><<<grid, 128, 0, s>>>(p);
            else return VFA_ERR_UNSUPPORTED;
            return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
        }
    }
    if (d == 128 && block_m == 64) {
        attn_fwd_kernel<128, 2, MODE><<<grid, 128, 0, s>>>(p);
        return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
    }
    if constexpr (!is_fa(MODE)) {  // (the baselines take the ping-pong kernel for every such call)
        if (d == 128 && block_m == 128) {
            attn_fwd_kernel<128, 4, MODE><<<grid, 256, 0, s>>>(p);
            return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
        }
    }
    if (d == 64 && block_m == 128) attn_fwd_kernel<64, 4, MODE><<<grid, 256, 0, s>>>(p);
    else if (d == 64 && block_m == 64) attn_fwd_kernel<64, 2, MODE><<<grid, 128, 0, s>>>(p);
    else return VFA_ERR_UNSUPPORTED;
    return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
}

int summary_launch(const void* K, void* Krepr, int B, int Hkv, int N, int d, int block_n, int repr_mode, hipStream_t s) {
    const int Tc = ceil_div(N, block_n);
    const dim3 grid((unsigned)Tc, (unsigned)(B * Hkv));
    const dim3 grid4((unsigned)ceil_div(Tc, 4), (unsigned)(B * Hkv));  // sabsmax: one wave per block, four to a workgroup
    const uint16_t* k = (const uint16_t*)K;
    uint16_t* r = (uint16_t*)Krepr;
    (void)hipGetLastError();
    if (repr_mode == 0) {
        with_rows(d, block_n, (long long)B * Hkv * N, [&](auto d_c, auto rows_c) {
            kblock_summary_kernel<decltype(d_c)::value, decltype(rows_c)::value><<<grid4, 256, 0, s>>>(k, r, N, N, Tc, block_n, 0, Tc);
        });
    } else {
        if (d == 128) kblock_summary_alt_kernel<128><<<grid, 256, 0, s>>>(k, r, N, Tc, block_n, repr_mode);
        else kblock_summary_alt_kernel<64><<<grid, 256, 0, s>>>(k, r, N, Tc, block_n, repr_mode);
    }
    return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
}

int vfa_vsa_common(int mode, const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int Hq, int Hkv,
                   int N, int d, int block_m, int block_n, int causal, int n_sink, int n_local, int use_minit,
                   float softmax_scale, float thr_nats, unsigned char* skip_mask, void* workspace,
                   size_t workspace_bytes, void* stream, int repr_mode = 0, int reorder = 1, int freeze = 1,
                   int rowskip = 0, float lazy_tau = -1.f, int q_repr_mode = 0, bool variant = false) {
    int rc = check_common(Q, K, V, O, LSE, B, Hq, Hkv, N, d, block_m, block_n);
    if (rc != VFA_OK) return rc;
    if (n_sink < 0 || n_local < 0) return VFA_ERR_INVALID_ARG;
    if (!use_minit && n_sink + n_local == 0 && freeze) return VFA_ERR_INVALID_ARG;
    // ascending order, no seed, no sink block: a query block whose first key block is not one of its local ones would
    // meet a frozen tile with the max still at -inf
    if (!use_minit && !reorder && n_sink == 0 && freeze) return VFA_ERR_INVALID_ARG;
    if (repr_mode < 0 || repr_mode > 3) return VFA_ERR_INVALID_ARG;
    if (q_repr_mode < 0 || q_repr_mode > 3 || (q_repr_mode && use_minit != 1)) return VFA_ERR_INVALID_ARG;
    if (!(lazy_tau < 0.f) && !isfinite(lazy_tau)) return VFA_ERR_INVALID_ARG;   // negative = off; NaN / inf rejected
    if (lazy_tau != lazy_tau) return VFA_ERR_INVALID_ARG;
    if ((rowskip || lazy_tau >= 0.f) && (mode != MODE_VSA || freeze)) return VFA_ERR_INVALID_ARG;
    if (mode == MODE_VSA && !(thr_nats > 0.f && isfinite(thr_nats))) return VFA_ERR_INVALID_ARG;
    if (!isfinite(softmax_scale)) return VFA_ERR_INVALID_ARG;
    if (use_minit < 0 || use_minit > 2) return VFA_ERR_INVALID_ARG;
    if (B == 0 || N == 0) return VFA_OK;
    const size_t krepr_bytes = vfa_workspace_bytes(B, Hkv, N, d, block_n);
    if (use_minit) {
        const size_t need = krepr_bytes + (q_repr_mode ? vfa_workspace_bytes(B, Hq, N, d, block_m) : 0);
        if (!workspace || !aligned16(workspace) || workspace_bytes < need) return VFA_ERR_INVALID_ARG;
        if ((long long)B * (q_repr_mode ? Hq : Hkv) > 65535) return VFA_ERR_UNSUPPORTED;
    }
    hipStream_t s = (hipStream_t)stream;
    const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / sqrtf((float)d);
    Params p{};
    p.Q = (const uint16_t*)Q; p.K = (const uint16_t*)K; p.V = (const uint16_t*)V;
    p.Krepr = (const uint16_t*)workspace; p.O = (uint16_t*)O; p.LSE = LSE; p.mask = skip_mask;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.N = N; p.Tr = ceil_div(N, block_m); p.Tc = ceil_div(N, block_n);
    p.causal = causal ? 1 : 0; p.n_sink = n_sink; p.n_local = n_local; p.use_minit = use_minit ? 1 : 0;
    p.order_asc = reorder ? 0 : 1; p.all_special = freeze ? 0 : 1;
    p.rowskip = rowskip ? 1 : 0; p.tau2 = lazy_tau >= 0.f ? lazy_tau : -1.f;
    p.c = scale * kLog2e;
    p.thr2 = thr_nats * kLog2e;
    if (mode == MODE_VFA && !variant) {  // (the ablation's calls differ in the max they fix, so all of them fix one)
        const int groups = short_groups(p, d, cu_count());
        if (groups) {
            (void)hipGetLastError();
            if (!raise_lds_limits()) return VFA_ERR_HIP;
            const bool sums = use_minit == 1;
            if (d == 64) return groups == 4 ? launch_short<64, 4>(p, 0, sums, s) : launch_short<64, 2>(p, 0, sums, s);
            return groups == 4 ? launch_short<128, 4>(p, 0, sums, s) : launch_short<128, 2>(p, 0, sums, s);
        }
    }
    void* qrepr = nullptr;
    if (use_minit == 1) {
        rc = summary_launch(K, workspace, B, Hkv, N, d, block_n, repr_mode, s);
        if (rc != VFA_OK) return rc;
        if (q_repr_mode) {  // the same reductions over the query blocks: 1 = unsigned absmax, 2 = sabsmax, 3 = mean
            static const int kSummaryMode[4] = {0, 3, 0, 2};
            qrepr = (char*)workspace + krepr_bytes;
            rc = summary_launch(Q, qrepr, B, Hq, N, d, block_m, kSummaryMode[q_repr_mode], s);
            if (rc != VFA_OK) return rc;
        }
    }
    p.Qrepr = (const uint16_t*)qrepr;
    return mode == MODE_VSA ? launch_fwd<MODE_VSA>(p, d, block_m, s) : launch_fwd<MODE_VFA>(p, d, block_m, s, variant);
}

int fa_common(int mode, const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int Hq, int Hkv,
              int N, int d, int block_m, int block_n, int causal, float softmax_scale, float tau, void* stream) {
    int rc = check_common(Q, K, V, O, LSE, B, Hq, Hkv, N, d, block_m, block_n);
    if (rc != VFA_OK) return rc;
    if (!isfinite(softmax_scale)) return VFA_ERR_INVALID_ARG;
    if (B == 0 || N == 0) return VFA_OK;
    Params p{};
    p.Q = (const uint16_t*)Q; p.K = (const uint16_t*)K; p.V = (const uint16_t*)V;
    p.O = (uint16_t*)O; p.LSE = LSE;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.N = N; p.Tr = ceil_div(N, block_m); p.Tc = ceil_div(N, block_n);
    p.causal = causal ? 1 : 0;
    const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / sqrtf((float)d);
    p.c = scale * kLog2e;
    p.tau2 = tau;  // tau is already a count of factors of two: tau * ln 2 nats = tau in the log2 domain
    if (mode == MODE_FA_SOFTEXP) return launch_fwd<MODE_FA_SOFTEXP>(p, d, block_m, (hipStream_t)stream);
    if (mode == MODE_FA_LAZY) return launch_fwd<MODE_FA_LAZY>(p, d, block_m, (hipStream_t)stream);
    return launch_fwd<MODE_FA>(p, d, block_m, (hipStream_t)stream);
}

int decode_common(const void* Q, const void* K, const void* V, const void* Krepr, void* O, float* LSE, int B, int Hq,
                  int Hkv, int n_cap, int n_keys, const int* seq_lens, int d, int block_n, int n_sink, int n_local,
                  int use_minit, int n_splits, float softmax_scale, void* workspace, size_t workspace_bytes, void* stream);

}  // namespace

// The one device array of the library: the partial sums of vfa_decode_noalloc_fwd's key ranges (what the
// workspace argument carries in vfa_decode_fwd).  Every device the library is used on holds its own copy, at
// its own address, until the process ends.  In host code the name below is only a handle for
// hipGetSymbolAddress: the kernels receive the address that call returns, never the name.
static __device__ __align__(256) unsigned char scratch[VFA_DECODE_NOALLOC_MAX_BYTES];

namespace {

// device address of `scratch` on the calling thread's current device; looked up on the first call per device
void* scratch_address() {
    static std::atomic<void*> addr[kMaxDevices];
    const int dev = current_device();
    if (dev < 0) return nullptr;
    void* ptr = addr[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return nullptr;
        }
        addr[dev].store(ptr, std::memory_order_release);
    }
    return ptr;
}

}  // namespace

extern "C" {

size_t vfa_workspace_bytes(int B, int Hkv, int N, int d, int block_n) {
    if (B <= 0 || Hkv <= 0 || N <= 0 || d <= 0 || block_n <= 0) return 0;
    const size_t bytes = (size_t)B * Hkv * ceil_div(N, block_n) * d * 2;
    return (bytes + 255) & ~(size_t)255;
}

int vfa_kblock_summary(const void* K, void* Krepr, int B, int Hkv, int N, int d, int block_n, void* stream) {
    return vfa_kblock_summary_mode(K, Krepr, B, Hkv, N, d, block_n, 0, stream);
}

int vfa_kblock_summary_mode(const void* K, void* Krepr, int B, int Hkv, int N, int d, int block_n, int repr_mode,
                            void* stream) {
    if (B < 0 || N < 0 || Hkv <= 0 || block_n <= 0) return VFA_ERR_INVALID_ARG;
    if (repr_mode < 0 || repr_mode > 3) return VFA_ERR_INVALID_ARG;
    if (d != 64 && d != 128) return VFA_ERR_UNSUPPORTED;
    if (B == 0 || N == 0) return VFA_OK;
    if (!K || !Krepr || !aligned16(K) || !aligned16(Krepr)) return VFA_ERR_INVALID_ARG;
    if ((long long)B * Hkv > 65535) return VFA_ERR_UNSUPPORTED;
    return summary_launch(K, Krepr, B, Hkv, N, d, block_n, repr_mode, (hipStream_t)stream);
}

int fa_baseline_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int Hq, int Hkv, int N,
                    int d, int block_m, int block_n, int causal, float softmax_scale, void* stream) {
    return fa_common(MODE_FA, Q, K, V, O, LSE, B, Hq, Hkv, N, d, block_m, block_n, causal, softmax_scale, 0.f, stream);
}

int fa_lazy_rescale_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int Hq, int Hkv,
                        int N, int d, int block_m, int block_n, int causal, float softmax_scale, float rescale_tau,
                        void* stream) {
    if (!(rescale_tau >= 0.f && isfinite(rescale_tau))) return VFA_ERR_INVALID_ARG;
    return fa_common(MODE_FA_LAZY, Q, K, V, O, LSE, B, Hq, Hkv, N, d, block_m, block_n, causal, softmax_scale, rescale_tau,
                     stream);
}

int fa_lazy_rescale_softexp_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int Hq, int Hkv,
                                int N, int d, int block_m, int block_n, int causal, float softmax_scale,
                                float rescale_tau, void* stream) {
    if (!(rescale_tau >= 0.f && isfinite(rescale_tau))) return VFA_ERR_INVALID_ARG;
    return fa_common(MODE_FA_SOFTEXP, Q, K, V, O, LSE, B, Hq, Hkv, N, d, block_m, block_n, causal, softmax_scale,
                     rescale_tau, stream);
}

int vfa_attn_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int Hq, int Hkv, int N,
                 int d, int block_m, int block_n, int causal, int n_sink, int n_local, int use_minit,
                 float softmax_scale, void* workspace, size_t workspace_bytes, void* stream) {
    return vfa_vsa_common(MODE_VFA, Q, K, V, O, LSE, B, Hq, Hkv, N, d, block_m, block_n, causal, n_sink, n_local,
                          use_minit, softmax_scale, 0.f, nullptr, workspace, workspace_bytes, stream);
}

int vsa_attn_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int Hq, int Hkv, int N,
                 int d, int block_m, int block_n, int causal, int n_sink, int n_local, int use_minit,
                 float softmax_scale, float skip_threshold_nats, unsigned char* skip_mask, void* workspace,
                 size_t workspace_bytes, void* stream) {
    return vfa_vsa_common(MODE_VSA, Q, K, V, O, LSE, B, Hq, Hkv, N, d, block_m, block_n, causal, n_sink, n_local,
                          use_minit, softmax_scale, skip_threshold_nats, skip_mask, workspace, workspace_bytes, stream);
}

int vfa_variant_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE, int B, int Hq, int Hkv, int N,
                    int d, int block_m, int block_n, int causal, int n_sink, int n_local, int use_minit, int repr_mode,
                    int q_repr_mode, int reorder, int freeze, int rowskip, float lazy_rescale_tau, float softmax_scale,
                    float skip_threshold_nats, unsigned char* skip_mask, void* workspace, size_t workspace_bytes,
                    void* stream) {
    const bool skipping = skip_threshold_nats != 0.f;
    return vfa_vsa_common(skipping ? MODE_VSA : MODE_VFA, Q, K, V, O, LSE, B, Hq, Hkv, N, d, block_m, block_n, causal,
                          n_sink, n_local, use_minit, softmax_scale, skip_threshold_nats, skipping ? skip_mask : nullptr,
                          workspace, workspace_bytes, stream, repr_mode, reorder, freeze, rowskip, lazy_rescale_tau,
                          q_repr_mode, true);
}

int vfa_kblock_summary_append(const void* K, void* Krepr, int B, int Hkv, int n_cap, int n_old, int n_new, int d,
                              int block_n, void* stream) {
    if (B < 0 || Hkv <= 0 || n_cap < 0 || block_n <= 0) return VFA_ERR_INVALID_ARG;
    if (n_old < 0 || n_new < n_old || n_new > n_cap) return VFA_ERR_INVALID_ARG;
    if (d != 64 && d != 128) return VFA_ERR_UNSUPPORTED;
    if (B == 0 || n_new == n_old) return VFA_OK;
    if (!K || !Krepr || !aligned16(K) || !aligned16(Krepr)) return VFA_ERR_INVALID_ARG;
    if ((long long)B * Hkv > 65535) return VFA_ERR_UNSUPPORTED;
    const int j0 = n_old / block_n, j1 = ceil_div(n_new, block_n);  // blocks [j0, j1) received keys
    const int tc_cap = ceil_div(n_cap, block_n);
    const dim3 grid((unsigned)ceil_div(j1 - j0, 4), (unsigned)(B * Hkv));
    hipStream_t s = (hipStream_t)stream;
    (void)hipGetLastError();
    with_rows(d, block_n, (long long)B * Hkv * (n_new - j0 * block_n), [&](auto d_c, auto rows_c) {
        kblock_summary_kernel<decltype(d_c)::value, decltype(rows_c)::value><<<grid, 256, 0, s>>>((const uint16_t*)K, (uint16_t*)Krepr, n_cap, n_new, tc_cap, block_n,
                                                                                                j0, j1 - j0);
    });
    return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
}

size_t vfa_decode_workspace_bytes(int B, int Hq, int d, int n_splits) {
    if (B <= 0 || Hq <= 0 || d <= 0 || n_splits <= 0) return 0;
    const size_t bytes = (size_t)B * Hq * n_splits * (2 + (size_t)d) * sizeof(float);
    return (bytes + 255) & ~(size_t)255;
}

int vfa_decode_fwd(const void* Q, const void* K, const void* V, const void* Krepr, void* O, float* LSE, int B, int Hq,
                   int Hkv, int n_cap, int n_keys, int d, int block_n, int n_sink, int n_local, int use_minit,
                   int n_splits, float softmax_scale, void* workspace, size_t workspace_bytes, void* stream) {
    if (n_keys < 1 || n_keys > n_cap) return VFA_ERR_INVALID_ARG;
    return decode_common(Q, K, V, Krepr, O, LSE, B, Hq, Hkv, n_cap, n_keys, nullptr, d, block_n, n_sink, n_local, use_minit,
                         n_splits, softmax_scale, workspace, workspace_bytes, stream);
}

int vfa_decode_noalloc_fwd(const void* Q, const void* K, const void* V, const void* Krepr, void* O, float* LSE, int B,
                           int Hq, int Hkv, int n_cap, int n_keys, int d, int block_n, int n_sink, int n_local,
                           int use_minit, int n_splits, float softmax_scale, void* stream) {
    if (n_keys < 1 || n_keys > n_cap) return VFA_ERR_INVALID_ARG;
    if (B < 0 || Hq <= 0 || d <= 0 || n_splits < 1) return VFA_ERR_INVALID_ARG;
    if (B == 0) return VFA_OK;
    // (rows * (2 + d) floats, in 64-bit arithmetic: the size check must not itself overflow)
    if ((unsigned long long)B * (unsigned long long)Hq * (unsigned long long)n_splits * (2ull + (unsigned long long)d) * 4ull >
        (unsigned long long)VFA_DECODE_NOALLOC_MAX_BYTES)
        return VFA_ERR_TOO_LARGE;
    void* const ws = scratch_address();
    if (!ws) return VFA_ERR_HIP;
    return decode_common(Q, K, V, Krepr, O, LSE, B, Hq, Hkv, n_cap, n_keys, nullptr, d, block_n, n_sink, n_local, use_minit,
                         n_splits, softmax_scale, ws, VFA_DECODE_NOALLOC_MAX_BYTES, stream);
}

int vfa_decode_varlen_fwd(const void* Q, const void* K, const void* V, const void* Krepr, void* O, float* LSE, int B,
                          int Hq, int Hkv, int n_cap, const int* seq_lens, int d, int block_n, int n_sink, int n_local,
                          int use_minit, int n_splits, float softmax_scale, void* workspace, size_t workspace_bytes,
                          void* stream) {
    if (B > 0 && (!seq_lens || (reinterpret_cast<uintptr_t>(seq_lens) & 3u))) return VFA_ERR_INVALID_ARG;
    return decode_common(Q, K, V, Krepr, O, LSE, B, Hq, Hkv, n_cap, n_cap, seq_lens, d, block_n, n_sink, n_local, use_minit,
                         n_splits, softmax_scale, workspace, workspace_bytes, stream);
}

int vfa_kblock_summary_append_varlen(const void* K, void* Krepr, int B, int Hkv, int n_cap, const int* old_lens,
                                     const int* new_lens, int d, int block_n, void* stream) {
    if (B < 0 || Hkv <= 0 || n_cap < 0 || block_n <= 0) return VFA_ERR_INVALID_ARG;
    if (d != 64 && d != 128) return VFA_ERR_UNSUPPORTED;
    if (B == 0 || n_cap == 0) return VFA_OK;
    if (!K || !Krepr || !old_lens || !new_lens || !aligned16(K) || !aligned16(Krepr)) return VFA_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(old_lens) | reinterpret_cast<uintptr_t>(new_lens)) & 3u) return VFA_ERR_INVALID_ARG;
    if ((long long)B * Hkv > 65535) return VFA_ERR_UNSUPPORTED;
    const int tc_cap = ceil_div(n_cap, block_n);
    hipStream_t s = (hipStream_t)stream;
    (void)hipGetLastError();
    auto launch = [&](auto d_c, auto rows_c, auto e_c) {
        constexpr int E = decltype(e_c)::value, NW = E ? 4 : 16;
        const long long wgs = min(((long long)B * Hkv * tc_cap + NW - 1) / NW, (long long)(APPEND_WAVES / NW));
        kblock_summary_varlen_kernel<decltype(d_c)::value, decltype(rows_c)::value, E><<<(unsigned)wgs, 64 * NW, 0, s>>>(
            (const uint16_t*)K, (uint16_t*)Krepr, B, Hkv, n_cap, tc_cap, block_n, old_lens, new_lens, (int)wgs);
    };
    with_rows(d, block_n, 0, [&](auto d_c, auto rows_c) {  // (the kernel counts the rows)
        if (B <= 64) launch(d_c, rows_c, std::integral_constant<int, 1>{});
        else if (B <= 256) launch(d_c, rows_c, std::integral_constant<int, 4>{});
        else launch(d_c, rows_c, std::integral_constant<int, 0>{});
    });
    return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
}

}  // extern "C"

namespace {
int decode_common(const void* Q, const void* K, const void* V, const void* Krepr, void* O, float* LSE, int B, int Hq,
                  int Hkv, int n_cap, int n_keys, const int* seq_lens, int d, int block_n, int n_sink, int n_local,
                  int use_minit, int n_splits, float softmax_scale, void* workspace, size_t workspace_bytes, void* stream) {
    if (B < 0 || Hq <= 0 || Hkv <= 0 || n_cap <= 0 || d <= 0 || block_n <= 0) return VFA_ERR_INVALID_ARG;
    if (Hq % Hkv != 0 || n_sink < 0 || n_local < 0 || n_splits < 1 || n_splits > 4096) return VFA_ERR_INVALID_ARG;
    if (use_minit != 0 && use_minit != 1) return VFA_ERR_INVALID_ARG;
    if (!use_minit && n_sink + n_local == 0) return VFA_ERR_INVALID_ARG;
    if (!isfinite(softmax_scale)) return VFA_ERR_INVALID_ARG;
    if ((d != 64 && d != 128) || block_n != BN || Hq / Hkv > 32) return VFA_ERR_UNSUPPORTED;
    if (B == 0) return VFA_OK;
    if (!Q || !K || !V || !O || !workspace || (use_minit && !Krepr)) return VFA_ERR_INVALID_ARG;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O) || !aligned16(workspace) ||
        (use_minit && !aligned16(Krepr)))
        return VFA_ERR_INVALID_ARG;
    if (LSE && (reinterpret_cast<uintptr_t>(LSE) & 3u)) return VFA_ERR_INVALID_ARG;
    if (workspace_bytes < vfa_decode_workspace_bytes(B, Hq, d, n_splits)) return VFA_ERR_INVALID_ARG;
    if ((long long)B * Hkv > 65535 || (long long)B * Hq > 0x7fffffffLL) return VFA_ERR_UNSUPPORTED;
    DecodeParams p{};
    p.Q = (const uint16_t*)Q; p.K = (const uint16_t*)K; p.V = (const uint16_t*)V;
    p.O = (uint16_t*)O; p.LSE = LSE;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.n_cap = n_cap; p.n_keys = n_keys; p.seq_lens = seq_lens; p.n_splits = n_splits;
    const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / sqrtf((float)d);
    p.c = scale * kLog2e;
    const size_t rows = (size_t)B * Hq * n_splits;
    p.opart = (float*)workspace; p.pm = p.opart + rows * d; p.lpart = p.pm + rows;  // the 16-byte stores go first
    hipStream_t s = (hipStream_t)stream;
    // Waves per range: two tiles of 16 KiB in flight per wave at d = 128, of 8 KiB at d = 64, and what the reads need is about
    // 64 KiB in flight per compute unit.  At 512 ranges (two per compute unit) one wave each is enough at d = 128 (512 MiB:
    // 88.8 us against 92.9 with two) and four are best at d = 64 (125 MiB: 28.1 us against 29.4 with two and 33 with one);
    // a range with fewer tiles than waves leaves waves idle.  Lengths that differ and are not dealt out: the longest entries finish
    // last, with few others left beside them, so d = 64 keeps two waves (4096 entries of up to 8192 keys, one KV head, one range
    // 304 us with one wave, 270 with two; d = 128 does not gain)
    const int n_cu = cu_count() > 0 ? cu_count() : 256;
    (void)hipGetLastError();
    // One range for each KV head after all, its keys shared by as many waves as fill a compute unit (or half of one, for more heads
    // than units), which then writes the result: no partial sums, no second launch (2.4 us and more).  `heads` KV heads of
    // `all` tiles; us, n_splits ranges / one:
    //   few tiles: up to five at d = 128 (8 heads, 100 keys 12.5 / 9.6, 320 12.5 / 10.4, 640 12.5 / 13.1; 32 heads, 512 12.4 / 13.1), 16 at d = 64
    //     (32 heads, 1000 keys 12.1 / 11.3, 1500 12.0 / 13.8); more heads than units, half a unit each, 16 (360 heads, d = 128, 700 keys
    //     28.6 / 27.5, 1500 49.5 / 50.5)
    //   as many heads as nearly fill the units, or their halves: always (d = 128, 180 heads, 700 keys 17.7 / 14.3, 3000 53.5 / 44.2, 20000 319 /
    //     270; 224, 8000 141 / 140, 20000 344 / 331; 256, 3000 63.1 / 60.7, 20000 387 / 384; 400, 1500 56.2 / 50.6, 20000 658 / 611; 504, 20000
    //     747 / 743; d = 64, 180 heads, 20000 169 / 136; 480, 8000 152 / 153; but 128 heads, 3000 38.3 / 42.1, and three ranges to two
    //     units, which end together: 384 heads, 8000 240 / 248, 20000 577 / 600)
    //   lengths that differ, which n_splits ranges even out: `all` is the longest there may be (16 x 8 heads of up to 700 keys 14.4 / 16.0;
    //     32 x 8 16.5 / 16.4, of up to 1500 20.5 / 24.5; d = 64 12.7 / 11.0 and 12.8 / 14.6)
    const long long heads = (long long)B * Hkv;
    const int all = ceil_div(n_keys, BN);
    bool single = false;
    const bool half = heads > n_cu;  // two workgroups to a compute unit
    if (n_splits > 1 && heads <= 2LL * n_cu) {
        const bool filled = half ? 2 * heads > 3LL * n_cu : 10 * heads >= 7LL * n_cu;
        if (!seq_lens) single = filled || all <= (half || d == 64 ? 16 : 5);
        else single = all <= (d == 64 ? (half ? 16 : 12) : (filled && !half ? 11 : 5));
        if (single) p.n_splits = n_splits = 1;
    }
    const long long wgs = heads * n_splits;
    const int tiles = ceil_div(all, n_splits);
    p.g = Hq / Hkv; p.per = tiles;
    // (the lines are explained at varlen_find)
    const bool dealt = seq_lens && n_splits > 1 && (B <= 64 || (B <= DEAL_MAX_B && wgs <= 8LL * n_cu && all > 2 * n_splits));
    auto launch = [&](auto d_c, auto w_c) {
        constexpr int D = decltype(d_c)::value, W = decltype(w_c)::value;
        const dim3 grid((unsigned)n_splits, (unsigned)B, (unsigned)Hkv);
        if (!seq_lens) {
            decode_split_kernel<D, W, LENS_ONE><<<grid, 64 * W, 0, s>>>(p);
        } else {
            bool launched = false;
            if constexpr (W * D <= 256) {  // (more waves share a KV head's only range)
                if (dealt) decode_split_kernel<D, W, LENS_DEALT><<<grid, 64 * W, 0, s>>>(p);
                launched = dealt;
            }
            if (!launched) decode_split_kernel<D, W, LENS_FIXED><<<dim3((unsigned)n_splits, (unsigned)Hkv, (unsigned)B), 64 * W, 0, s>>>(p);
        }
        if (n_splits == 1) return;
        if (dealt) decode_merge_kernel<D, true><<<dim3((unsigned)Hq, (unsigned)B), 256, 0, s>>>(p);
        else decode_merge_kernel<D, false><<<dim3((unsigned)Hq, (unsigned)B), 256, 0, s>>>(p);
    };
    using std::integral_constant;
    if (single) {
        if (d == 128 && !half) launch(integral_constant<int, 128>{}, integral_constant<int, 4>{});
        else if (d == 128) launch(integral_constant<int, 128>{}, integral_constant<int, 2>{});
        else if (!half) launch(integral_constant<int, 64>{}, integral_constant<int, 8>{});
        else launch(integral_constant<int, 64>{}, integral_constant<int, 4>{});
    } else if (d == 128) {
        if (tiles >= 2 && wgs <= n_cu) launch(integral_constant<int, 128>{}, integral_constant<int, 2>{});
        else launch(integral_constant<int, 128>{}, integral_constant<int, 1>{});
    } else {
        if (tiles >= 4 && wgs <= 2LL * n_cu) launch(integral_constant<int, 64>{}, integral_constant<int, 4>{});
        else if ((tiles >= 2 && wgs <= 4LL * n_cu) || (seq_lens && !dealt && tiles >= 8)) launch(integral_constant<int, 64>{}, integral_constant<int, 2>{});
        else launch(integral_constant<int, 64>{}, integral_constant<int, 1>{});
    }
    return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
}
}  // namespace

namespace {
// Launches one of the quantising kernels over n8 runs of eight elements: `launch(chunks, stream, blocks)`.
// Runs of a thread: one while that gives no more than 2048 workgroups, eight to a compute unit (E4M3 / MXFP4, 2^20 elements
// 2.0 / 2.3 us, with four runs 2.5 / 3.2), then two (2^25: 15.7 / 18.0, one 16.1 / 18.4, four 16.1 / 19.3), four with
// non-temporal loads above 2^26 elements (2^27: 63 / 67, plain loads 69 / 67 with two), up to which the input may still be in
// the memory-side cache, written by the kernel before (2^26: plain 29.1 / 32.5, non-temporal 33.8 / 35.8)
template <typename F>
int quantize_launch(long long n8, F launch) {
    const int chunks = n8 <= 256 * 2048 ? 1 : (n8 <= 1LL << 23 ? 2 : 4);
    const long long blocks = (n8 + 256 * chunks - 1) / (256 * chunks);
    if (blocks > 0x7fffffffLL) return VFA_ERR_UNSUPPORTED;
    (void)hipGetLastError();
    if (chunks == 1) launch(std::integral_constant<int, 1>{}, std::false_type{}, (unsigned)blocks);
    else if (chunks == 2) launch(std::integral_constant<int, 2>{}, std::false_type{}, (unsigned)blocks);
    else launch(std::integral_constant<int, 4>{}, std::true_type{}, (unsigned)blocks);
    return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
}
}  // namespace

extern "C" {

size_t vfa_fp8_v_bytes(int B, int Hkv, int N) {
    if (B <= 0 || Hkv <= 0 || N <= 0) return 0;
    return (size_t)B * Hkv * ceil_div(N, BN) * Tile8::VBYTES;
}

int vfa_fp8_quantize(const void* X, void* X8, long long n, float inv_scale, void* stream) {
    if (n < 0 || (n & 7) || !(inv_scale > 0.f) || !isfinite(inv_scale)) return VFA_ERR_INVALID_ARG;
    if (n == 0) return VFA_OK;
    if (!X || !X8 || !aligned16(X) || (reinterpret_cast<uintptr_t>(X8) & 7u)) return VFA_ERR_INVALID_ARG;
    const long long n8 = n / 8;
    return quantize_launch(n8, [&](auto chunks, auto stream_c, unsigned blocks) {
        fp8_quantize_kernel<decltype(chunks)::value, decltype(stream_c)::value><<<blocks, 256, 0, (hipStream_t)stream>>>((const uint16_t*)X, (uint8_t*)X8, n8, inv_scale);
    });
}

int vfa_fp8_pack_v(const void* V, void* Vt, int B, int Hkv, int N, int d, float inv_scale, void* stream) {
    if (B < 0 || Hkv <= 0 || N < 0 || !(inv_scale > 0.f) || !isfinite(inv_scale)) return VFA_ERR_INVALID_ARG;
    if (d != 128) return VFA_ERR_UNSUPPORTED;
    if (B == 0 || N == 0) return VFA_OK;
    if (!V || !Vt || !aligned16(V) || !aligned16(Vt)) return VFA_ERR_INVALID_ARG;
    if ((long long)B * Hkv > 65535) return VFA_ERR_UNSUPPORTED;
    const int Tc = ceil_div(N, BN);
    (void)hipGetLastError();
    fp8_pack_v_kernel<<<dim3((unsigned)Tc, (unsigned)(B * Hkv)), 256, 0, (hipStream_t)stream>>>((const uint16_t*)V, (uint8_t*)Vt,
                                                                                              N, Tc, inv_scale);
    return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
}

}  // extern "C"

namespace {

int fp8_common(int frozen, bool noexp, const void* Q8, const void* K8, const void* Vt8, void* O, float* LSE, int B, int Hq,
               int Hkv, int N, int d, int block_m, int block_n, int causal, int n_sink, int n_local, int use_minit,
               float softmax_scale, float descale_q, float descale_k, float descale_v, void* workspace,
               size_t workspace_bytes, void* stream) {
    if (B < 0 || N < 0 || Hq <= 0 || Hkv <= 0 || d <= 0 || block_m <= 0 || block_n <= 0) return VFA_ERR_INVALID_ARG;
    if (Hq % Hkv != 0 || (frozen != 0 && frozen != 1)) return VFA_ERR_INVALID_ARG;
    if (!(descale_q > 0.f && descale_k > 0.f && descale_v > 0.f) || !isfinite(descale_q * descale_k) || !isfinite(descale_v) ||
        !isfinite(softmax_scale))
        return VFA_ERR_INVALID_ARG;
    if (frozen) {
        if (n_sink < 0 || n_local < 0 || use_minit < 0 || use_minit > 2) return VFA_ERR_INVALID_ARG;
        if (!use_minit && n_sink + n_local == 0) return VFA_ERR_INVALID_ARG;
    }
    if (d != 128 || block_m != 128 || block_n != BN) return VFA_ERR_UNSUPPORTED;
    if (B == 0 || N == 0) return VFA_OK;
    if (!Q8 || !K8 || !Vt8 || !O || !aligned16(Q8) || !aligned16(K8) || !aligned16(Vt8) || !aligned16(O)) return VFA_ERR_INVALID_ARG;
    if (LSE && (reinterpret_cast<uintptr_t>(LSE) & 3u)) return VFA_ERR_INVALID_ARG;
    const int Tc = ceil_div(N, BN), Tr = ceil_div(N, block_m);
    if ((long long)B * Hq * Tr > kMaxWorkgroups256 || (long long)B * Hq * N > 0x7fffffffLL || (long long)B * Hkv > 65535)
        return VFA_ERR_UNSUPPORTED;
    const bool minit = frozen && use_minit;
    if (minit && (!workspace || !aligned16(workspace) || workspace_bytes < (size_t)B * Hkv * Tc * 128)) return VFA_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    Fp8Params p{};
    p.Q = (const uint8_t*)Q8; p.K = (const uint8_t*)K8; p.Vt = (const uint8_t*)Vt8; p.Krepr = (const uint8_t*)workspace;
    p.O = (uint16_t*)O; p.LSE = LSE;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.N = N; p.Tr = Tr; p.Tc = Tc;
    p.causal = causal ? 1 : 0; p.n_sink = n_sink; p.n_local = n_local; p.use_minit = minit ? 1 : 0;
    const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / sqrtf((float)d);
    p.c = scale * descale_q * descale_k * kLog2e;
    p.descale_v = descale_v;
    p.headroom = frozen ? 4.f : 0.f;
    // Alg. 1 with the factor between code products and log2-domain scores a power of two (the caller's choice
    // of descale_q decides): that factor moves into the MFMA's block scale and the frozen max into its
    // accumulator start
    bool fold = false;
    if (frozen) {
        int ex = 0;
        const float mant = frexpf(p.c, &ex);  // p.c = mant * 2^ex, mant in [0.5, 1)
        if (fabsf(mant - 0.5f) <= 0x1p-18f && ex - 1 >= -100 && ex - 1 <= 100) {
            fold = true;
            p.scale_a = (int)((uint32_t)(127 + ex - 1) * 0x01010101u);
            p.c = 1.f;
        }
    }
    if (noexp && !fold) return VFA_ERR_INVALID_ARG;  // (before anything is launched)
    (void)hipGetLastError();
    if (minit && use_minit == 1) {
        fp8_kblock_summary_kernel<<<dim3((unsigned)Tc, (unsigned)(B * Hkv)), 256, 0, s>>>((const uint8_t*)K8, (uint8_t*)workspace, N, Tc);
        if (hipGetLastError() != hipSuccess) return VFA_ERR_HIP;
    }
    const dim3 grid((unsigned)(B * Hq * Tr));
    if (noexp) attn_fp8_kernel<MODE_VFA, true, true><<<grid, 256, 0, s>>>(p);
    else if (fold) attn_fp8_kernel<MODE_VFA, true><<<grid, 256, 0, s>>>(p);
    else if (frozen) attn_fp8_kernel<MODE_VFA, false><<<grid, 256, 0, s>>>(p);
    else attn_fp8_kernel<MODE_FA, false><<<grid, 256, 0, s>>>(p);
    return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
}

}  // namespace

extern "C" {

int vfa_fp8_attn_fwd(int frozen, const void* Q8, const void* K8, const void* Vt8, void* O, float* LSE, int B, int Hq, int Hkv,
                     int N, int d, int block_m, int block_n, int causal, int n_sink, int n_local, int use_minit,
                     float softmax_scale, float descale_q, float descale_k, float descale_v, void* workspace,
                     size_t workspace_bytes, void* stream) {
    return fp8_common(frozen, false, Q8, K8, Vt8, O, LSE, B, Hq, Hkv, N, d, block_m, block_n, causal, n_sink, n_local, use_minit,
                      softmax_scale, descale_q, descale_k, descale_v, workspace, workspace_bytes, stream);
}

int vfa_fp8_attn_noexp_fwd(const void* Q8, const void* K8, const void* Vt8, void* O, float* LSE, int B, int Hq, int Hkv, int N,
                           int d, int block_m, int block_n, int causal, int n_sink, int n_local, int use_minit,
                           float softmax_scale, float descale_q, float descale_k, float descale_v, void* workspace,
                           size_t workspace_bytes, void* stream) {
    return fp8_common(1, true, Q8, K8, Vt8, O, LSE, B, Hq, Hkv, N, d, block_m, block_n, causal, n_sink, n_local, use_minit,
                      softmax_scale, descale_q, descale_k, descale_v, workspace, workspace_bytes, stream);
}

size_t vfa_mxfp4_workspace_bytes(int B, int Hkv, int N) {
    if (B <= 0 || Hkv <= 0 || N <= 0) return 0;
    const size_t bytes = (size_t)B * Hkv * ceil_div(N, BN) * (128 + 4);
    return (bytes + 255) & ~(size_t)255;
}

int vfa_mxfp4_quantize(const void* X, void* X4, void* XS, long long n, float pre_scale, void* stream) {
    if (n < 0 || (n & 31) || !(pre_scale > 0.f) || !isfinite(pre_scale)) return VFA_ERR_INVALID_ARG;
    if (n == 0) return VFA_OK;
    if (!X || !X4 || !XS || !aligned16(X) || (reinterpret_cast<uintptr_t>(X4) & 3u)) return VFA_ERR_INVALID_ARG;
    const long long n8 = n / 8;
    return quantize_launch(n8, [&](auto chunks, auto stream_c, unsigned blocks) {
        mx4_quantize_kernel<decltype(chunks)::value, decltype(stream_c)::value><<<blocks, 256, 0, (hipStream_t)stream>>>((const uint16_t*)X, (uint8_t*)X4, (uint8_t*)XS, n8, pre_scale);
    });
}

}  // extern "C"

namespace {

int mx4_common(int frozen, bool noexp, const void* Q4, const void* QS, const void* K4, const void* KS, const void* Vt8, void* O,
               float* LSE, int B, int Hq, int Hkv, int N, int d, int block_m, int block_n, int causal, int n_sink,
               int n_local, int use_minit, float softmax_scale, float descale_v, void* workspace,
               size_t workspace_bytes, void* stream) {
    if (B < 0 || N < 0 || Hq <= 0 || Hkv <= 0 || d <= 0 || block_m <= 0 || block_n <= 0) return VFA_ERR_INVALID_ARG;
    if (Hq % Hkv != 0 || (frozen != 0 && frozen != 1)) return VFA_ERR_INVALID_ARG;
    if (!(descale_v > 0.f) || !isfinite(descale_v) || !isfinite(softmax_scale)) return VFA_ERR_INVALID_ARG;
    if (frozen) {
        if (n_sink < 0 || n_local < 0 || use_minit < 0 || use_minit > 2) return VFA_ERR_INVALID_ARG;
        if (!use_minit && n_sink + n_local == 0) return VFA_ERR_INVALID_ARG;
    }
    if (d != 128 || block_m != 128 || block_n != BN) return VFA_ERR_UNSUPPORTED;
    if (B == 0 || N == 0) return VFA_OK;
    if (!Q4 || !QS || !K4 || !KS || !Vt8 || !O) return VFA_ERR_INVALID_ARG;
    if (!aligned16(Q4) || !aligned16(K4) || !aligned16(Vt8) || !aligned16(O)) return VFA_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(QS) & 3u) || (reinterpret_cast<uintptr_t>(KS) & 3u)) return VFA_ERR_INVALID_ARG;
    if (LSE && (reinterpret_cast<uintptr_t>(LSE) & 3u)) return VFA_ERR_INVALID_ARG;
    const int Tc = ceil_div(N, BN), Tr = ceil_div(N, block_m);
    if ((long long)B * Hq * Tr > kMaxWorkgroups256 || (long long)B * Hq * N > 0x7fffffffLL || (long long)B * Hkv > 65535)
        return VFA_ERR_UNSUPPORTED;
    const bool minit = frozen && use_minit;
    if (minit && (!workspace || !aligned16(workspace) || workspace_bytes < vfa_mxfp4_workspace_bytes(B, Hkv, N)))
        return VFA_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    uint8_t* const repr = (uint8_t*)workspace;
    uint8_t* const repr_s = repr ? repr + (size_t)B * Hkv * Tc * 128 : nullptr;  // (a multiple of 128: dword aligned)
    {
        const float sc = softmax_scale > 0.f ? softmax_scale : 1.0f / sqrtf((float)d);
        if (noexp && !(fabsf(sc * kLog2e - 1.f) <= 0x1p-18f)) return VFA_ERR_INVALID_ARG;  // (before anything is launched)
    }
    (void)hipGetLastError();
    if (minit && use_minit == 1) {
        mx4_kblock_summary_kernel<<<dim3((unsigned)Tc, (unsigned)(B * Hkv)), 256, 0, s>>>((const uint8_t*)K4, (const uint8_t*)KS,
                                                                                         repr, repr_s, N, Tc);
        if (hipGetLastError() != hipSuccess) return VFA_ERR_HIP;
    }
    Mx4Params p{};
    p.Q = (const uint8_t*)Q4; p.Qs = (const uint8_t*)QS; p.K = (const uint8_t*)K4; p.Ks = (const uint8_t*)KS;
    p.Vt = (const uint8_t*)Vt8; p.Krepr = repr; p.KreprS = repr_s;
    p.O = (uint16_t*)O; p.LSE = LSE;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.N = N; p.Tr = Tr; p.Tc = Tc;
    p.causal = causal ? 1 : 0; p.n_sink = n_sink; p.n_local = n_local; p.use_minit = minit ? 1 : 0;
    const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / sqrtf((float)d);
    p.c = scale * kLog2e;
    p.descale_v = descale_v;
    p.headroom = frozen ? 4.f : 0.f;
    // Alg. 1 with the scores already in log2 units (the caller multiplied Q by scale * log2(e) before quantising
    // and passes softmax_scale = ln 2): nothing is left to multiply, and the frozen max becomes the accumulators' start
    const bool fold = frozen && fabsf(p.c - 1.f) <= 0x1p-18f;
    if (fold) p.c = 1.f;
    const dim3 grid((unsigned)(B * Hq * Tr));
    if (noexp) attn_mx4_kernel<MODE_VFA, true, true><<<grid, 256, 0, s>>>(p);
    else if (fold) attn_mx4_kernel<MODE_VFA, true><<<grid, 256, 0, s>>>(p);
    else if (frozen) attn_mx4_kernel<MODE_VFA, false><<<grid, 256, 0, s>>>(p);
    else attn_mx4_kernel<MODE_FA, false><<<grid, 256, 0, s>>>(p);
    return hipGetLastError() == hipSuccess ? VFA_OK : VFA_ERR_HIP;
}

}  // namespace

extern "C" {

int vfa_mxfp4_attn_fwd(int frozen, const void* Q4, const void* QS, const void* K4, const void* KS, const void* Vt8, void* O,
                       float* LSE, int B, int Hq, int Hkv, int N, int d, int block_m, int block_n, int causal, int n_sink,
                       int n_local, int use_minit, float softmax_scale, float descale_v, void* workspace,
                       size_t workspace_bytes, void* stream) {
    return mx4_common(frozen, false, Q4, QS, K4, KS, Vt8, O, LSE, B, Hq, Hkv, N, d, block_m, block_n, causal, n_sink, n_local,
                      use_minit, softmax_scale, descale_v, workspace, workspace_bytes, stream);
}

int vfa_mxfp4_attn_noexp_fwd(const void* Q4, const void* QS, const void* K4, const void* KS, const void* Vt8, void* O,
                             float* LSE, int B, int Hq, int Hkv, int N, int d, int block_m, int block_n, int causal,
                             int n_sink, int n_local, int use_minit, float softmax_scale, float descale_v, void* workspace,
                             size_t workspace_bytes, void* stream) {
    return mx4_common(1, true, Q4, QS, K4, KS, Vt8, O, LSE, B, Hq, Hkv, N, d, block_m, block_n, causal, n_sink, n_local,
                      use_minit, softmax_scale, descale_v, workspace, workspace_bytes, stream);
}

const char* vfa_strerror(int code) {
    switch (code) {
        case VFA_OK: return "ok";
        case VFA_ERR_INVALID_ARG: return "invalid argument";
        case VFA_ERR_UNSUPPORTED: return "unsupported shape (d must be 64 or 128; blocks 64x64 or 128x64)";
        case VFA_ERR_HIP: return "HIP launch error";
        case VFA_ERR_TOO_LARGE: return "problem needs more scratch than the library's fixed device array holds (use the entry point that takes a workspace)";
        default: return "unknown error code";
    }
}

}  // extern "C"
