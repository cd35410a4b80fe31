// Seed Location Checker kernels for gfx950: compaction of the seed location
// filter bitmask into the list of surviving locations, and the alignment check
// of the survivors (edit distance of the read within its bin's span).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "grim_device.h"
#include "grim_internal.h"

namespace grim {

// ------------------------------------------------- seed location checker
// Survivor compaction (Section "Integration with a Full Read Mapper": the Seed
// Location Checker reads the filter bitmask and fetches only the passing
// locations).  Three launches: per-block popcounts, one-block exclusive scan
// of the block totals, then the emit pass lists each block's passing pairs in
// LDS, in order, and writes them one survivor per thread: every store is
// coalesced and a thread's bin ids are fetched side by side.  What bounds it is
// those fetches (at 1.5 % passing, some 1e7 lines of cand_bin, most of 1.5 GB
// moved).  Measured on 8.3e8 pairs of 4M reads, 12.4M survivors: 21 + 11 + 237 us;
// one thread walking each 128 pairs, its reads searched by two threads a block
// and 1024 totals scanned at a time, took 40 + 38 + 517.  5.6e5 pairs, 7.4e4
// survivors: 4 + 3 + 9 us (4 + 5 + 43).
constexpr int kCompactWpt = 4;                       // bitmask words per thread
constexpr int kCompactWpb = 256 * kCompactWpt;       // words per block

__device__ __forceinline__ uint32_t mask_word(const uint32_t *bits, uint64_t w, uint64_t n_pairs)
{
    uint32_t x = bits[w];
    const uint64_t end = (w + 1) * 32;
    if (end > n_pairs)
        x &= (n_pairs & 31) ? ((1u << (n_pairs & 31)) - 1u) : 0u;
    return x;
}

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *lds, uint32_t *total)
{
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
        const uint32_t y = __shfl_up(incl, s);
        if (lane >= s)
            incl += y;
    }
    if (lane == 63)
        lds[wv] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
        if (i < wv)
            before += lds[i];
        all += lds[i];
    }
    __syncthreads();
    *total = all;
    return before + incl - v;
}

// N words of the bitmask from w0 on (0 past its end) and their popcount.
template <int N>
__device__ __forceinline__ uint32_t load_mask(const uint32_t *__restrict__ bits, uint64_t w0,
                                              uint64_t n_words, uint64_t n_pairs, uint32_t (&x)[N])
{
    uint32_t c = 0;
    if ((w0 + N) * 32 <= n_pairs) {
        __builtin_memcpy(x, bits + w0, sizeof(x));   // one load, 4-byte aligned
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j)
            x[j] = (w0 + j < n_words) ? mask_word(bits, w0 + j, n_pairs) : 0u;
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
        c += __popc(x[j]);
    return c;
}

// Popcounts of kCountBlocks emit blocks, one per wavefront at a time, their
// loads side by side.
constexpr int kCountBlocks = 8;

__global__ __launch_bounds__(256) void compact_count_kernel(const uint32_t *__restrict__ bits,
                                                            uint64_t n_words, uint64_t n_pairs,
                                                            uint64_t n_blocks,
                                                            uint64_t *__restrict__ block_sums)
{
    const int lane = threadIdx.x & 63;
    const uint64_t b0 = ((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * (kCountBlocks / 4);
#pragma unroll
    for (int i = 0; i < kCountBlocks / 4; ++i) {
        const uint64_t b = b0 + i;
        if (b >= n_blocks)
            return;
        uint32_t x[4][kCompactWpt], c = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            c += load_mask<kCompactWpt>(bits, b * kCompactWpb + (uint64_t)(j * 64 + lane) * kCompactWpt, n_words,
                           n_pairs, x[j]);
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1)
            c += __shfl_xor(c, m);
        if (lane == 0)
            block_sums[b] = c;
    }
}

// One workgroup: in-place exclusive scan of n block totals; *n_out = sum.  Up to
// 32768 totals at a time go through LDS (one pad word per 32), so that global
// loads and stores are contiguous while each thread scans consecutive ones: one
// round of loads and one block scan where 1024 at a time took 25 (38 us; 11 now).
constexpr uint32_t kScanRound = 1024 * 32;

__global__ __launch_bounds__(1024) void compact_scan_kernel(uint64_t *sums, uint64_t n, uint64_t *n_out)
{
    __shared__ uint32_t v[kScanRound + kScanRound / 32];   // a block holds 32768 pairs at most
    __shared__ uint32_t part[16];
    const uint32_t t = threadIdx.x;
    const int lane = t & 63, wv = t >> 6;
    auto at = [](uint32_t i) { return i + (i >> 5); };
    uint64_t carry = 0;
    for (uint64_t base = 0; base < n; base += kScanRound) {
        const uint32_t m = n - base < kScanRound ? (uint32_t)(n - base) : kScanRound;
        const uint32_t k = (m + 1023) / 1024;   // consecutive totals per thread
#pragma unroll 8
        for (uint32_t i = t; i < m; i += 1024)
            v[at(i)] = (uint32_t)sums[base + i];
        __syncthreads();
        const uint32_t lo = min(t * k, m), hi = min(lo + k, m);
        uint32_t mine = 0;
        for (uint32_t i = lo; i < hi; ++i)
            mine += v[at(i)];
        uint32_t incl = mine;
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) {
            const uint32_t y = __shfl_up(incl, s);
            if (lane >= s)
                incl += y;
        }
        if (lane == 63)
            part[wv] = incl;
        __syncthreads();
        uint32_t before = incl - mine, all = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < wv)
                before += part[w];
            all += part[w];
        }
        for (uint32_t i = lo; i < hi; ++i) {
            const uint32_t x = v[at(i)];
            v[at(i)] = before;
            before += x;
        }
        __syncthreads();
        for (uint32_t i = t; i < m; i += 1024)
            sums[base + i] = carry + v[at(i)];
        carry += all;
        __syncthreads();   // v and part are written again
    }
    if (t == 0)
        *n_out = carry;
}

// Read holding pair k: the last r in [lo, hi] with off[r] <= k (off[lo] <= k).
template <typename Off>
__device__ __forceinline__ uint64_t read_of(const Off *off, uint64_t lo, uint64_t hi, uint64_t k)
{
    while (lo < hi) {
        const uint64_t mid = (lo + hi + 1) >> 1;
        if ((uint64_t)off[mid] <= k)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// A workgroup covers WPB words of the bitmask: a whole block of the count pass
// (32768 pairs), or a quarter or a sixteenth of one where there are too few blocks
// to fill the chip, and then counts the words before its own in the block itself.  Its
// passing pairs are listed in LDS kEmitList at a time (about 490 a block at
// 1.5 %), and the offsets of the reads they belong to, relative to its first
// pair, are staged there when there are at most kStageReads of them.
constexpr int kStageReads = 2048;
constexpr int kEmitList = 4096;
constexpr int kEmitRow = 4;       // survivors per thread whose bin ids load together
constexpr int kEmitSmall = 64;    // words of the smaller workgroups
constexpr int kEmitMiddle = 256;

template <int WPB>
__global__ __launch_bounds__(256) void compact_emit_kernel(
    const uint32_t *__restrict__ bits, uint64_t n_words, uint64_t n_pairs,
    const uint64_t *__restrict__ block_off, const uint64_t *__restrict__ cand_off, uint64_t n_reads,
    const uint32_t *__restrict__ cand_bin, uint64_t cap, uint64_t *__restrict__ surv_pair,
    uint32_t *__restrict__ surv_read, uint32_t *__restrict__ surv_bin)
{
    constexpr int WPT = WPB >= 256 ? WPB / 256 : 1;   // words per thread
    constexpr uint32_t kPairs = WPB * 32;
    constexpr int kSub = kCompactWpb / WPB;           // workgroups per block
    __shared__ uint32_t lds[4];
    __shared__ uint32_t stage[kStageReads];
    __shared__ uint16_t list[kEmitList];
    __shared__ uint64_t range[2];
    const int t = threadIdx.x;
    const uint64_t w_first = (uint64_t)blockIdx.x * WPB, p_first = w_first * 32;
    const uint64_t block = blockIdx.x / kSub;
    uint32_t x[WPT] = {};
    const uint32_t c =
        t * WPT < WPB ? load_mask<WPT>(bits, w_first + t * WPT, n_words, n_pairs, x) : 0u;
    uint32_t ahead = 0;   // survivors of the block before this workgroup's words
    if (kSub > 1) {
        uint32_t one = 0, y[1];
        for (uint64_t w = block * kCompactWpb + t; w < w_first; w += 256)
            one += load_mask<1>(bits, w, n_words, n_pairs, y);
        block_exclusive_scan(one, lds, &ahead);
    }
    uint32_t total;
    const uint32_t before = block_exclusive_scan(c, lds, &total);
    if (total == 0 || n_reads == 0)
        return;
    // reads of the workgroup's first and last pair, a wavefront each
    const uint64_t p_end = p_first + kPairs < n_pairs ? p_first + kPairs : n_pairs;
    if (t < 128) {
        const uint64_t r = wave_read_of(cand_off, n_reads, t < 64 ? p_first : p_end - 1, t & 63);
        if ((t & 63) == 0)
            range[t >> 6] = r;
    }
    __syncthreads();
    const uint64_t r_lo = range[0];
    const uint64_t n_own = range[1] >= r_lo ? range[1] - r_lo + 1 : 1;
    const bool staged = n_own <= (uint64_t)kStageReads;
    if (staged)
        for (uint32_t i = t; i < n_own; i += 256) {
            const uint64_t o = cand_off[r_lo + i];
            stage[i] = o <= p_first ? 0u : o - p_first < kPairs ? (uint32_t)(o - p_first) : kPairs;
        }
    const uint64_t pos0 = block_off[block] + ahead;
    for (uint32_t at = 0; at < total; at += kEmitList) {
        if (before < at + kEmitList && before + c > at) {
            uint32_t rank = before - at;   // wraps for survivors listed before
#pragma unroll
            for (int j = 0; j < WPT; ++j)
                for (uint32_t m = x[j]; m; m &= m - 1, ++rank)
                    if (rank < (uint32_t)kEmitList)
                        list[rank] = (uint16_t)((t * WPT + j) * 32 + (__ffs(m) - 1));
        }
        __syncthreads();
        const uint32_t n = min(total - at, (uint32_t)kEmitList);
        for (uint32_t i0 = t; i0 < n; i0 += 256 * kEmitRow) {
            uint32_t rel[kEmitRow], bin[kEmitRow];
#pragma unroll
            for (int u = 0; u < kEmitRow; ++u) {
                const uint32_t i = i0 + u * 256;
                rel[u] = i < n ? list[i] : list[i0];
                bin[u] = cand_bin[p_first + rel[u]];
            }
#pragma unroll
            for (int u = 0; u < kEmitRow; ++u) {
                const uint32_t i = i0 + u * 256;
                const uint64_t pos = pos0 + at + i;
                if (i < n && pos < cap) {
                    const uint64_t r =
                        staged ? r_lo + read_of(stage, 0, n_own - 1, rel[u])
                               : read_of(cand_off, r_lo, r_lo + n_own - 1, p_first + rel[u]);
                    surv_pair[pos] = p_first + rel[u];
                    surv_read[pos] = (uint32_t)r;
                    surv_bin[pos] = bin[u];
                }
            }
        }
        __syncthreads();   // the list is written again
    }
}

hipError_t launch_compact(hipStream_t s, const uint32_t *bits, uint64_t n_pairs,
                          const uint64_t *cand_off, uint64_t n_reads, const uint32_t *cand_bin,
                          uint64_t cap, uint64_t *surv_pair, uint32_t *surv_read,
                          uint32_t *surv_bin, uint64_t *n_out, uint64_t *block_sums)
{
    const uint64_t n_words = (n_pairs + 31) / 32;
    const uint64_t nb = (n_words + kCompactWpb - 1) / kCompactWpb;
    if (nb == 0) {
        hipLaunchKernelGGL(compact_scan_kernel, dim3(1), dim3(1024), 0, s, block_sums, 0, n_out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(compact_count_kernel, dim3((uint32_t)((nb + kCountBlocks - 1) / kCountBlocks)),
                       dim3(256), 0, s, bits, n_words, n_pairs, nb, block_sums);
    hipLaunchKernelGGL(compact_scan_kernel, dim3(1), dim3(1024), 0, s, block_sums, nb, n_out);
    // Sixteenths below 128 blocks (4.2e6 pairs), quarters below 512 (1.7e7).  All three
    // launches, whole blocks / quarters / sixteenths: 4.3e6 pairs at 1.5 % passing 14 /
    // 14 / 15 us, with all of them 194 / 46 / 34; 8e6 14 / 14 / 19 and 194 / 52 / 43;
    // 1.6e7 16 / 16 / 32 and 210 / 89 / 95; 2.4e7 20 / 22 / 44 and 236 / 130 / 137.
    auto emit = [&](auto kernel, uint64_t words) {
        hipLaunchKernelGGL(kernel, dim3((uint32_t)((n_words + words - 1) / words)), dim3(256), 0, s,
                           bits, n_words, n_pairs, block_sums, cand_off, n_reads, cand_bin, cap,
                           surv_pair, surv_read, surv_bin);
    };
    if (nb < 128)
        emit(compact_emit_kernel<kEmitSmall>, kEmitSmall);
    else if (nb < 512)
        emit(compact_emit_kernel<kEmitMiddle>, kEmitMiddle);
    else
        emit(compact_emit_kernel<kCompactWpb>, kCompactWpb);
    return hipGetLastError();
}

uint64_t compact_blocks(uint64_t n_pairs)
{
    const uint64_t n_words = (n_pairs + 31) / 32;
    return (n_words + kCompactWpb - 1) / kCompactWpb;
}


// ---------------------------------------------------- alignment check
// Smallest edit distance between a surviving read and any substring of its
// bin's span (free start and end in the reference), i.e. whether the
// location really holds the read within E edits.  Computed with Myers'
// bit-parallel approximate-matching recurrence (G. Myers, J. ACM 46(3), 1999)
// on one long bit vector per column: row i of the dynamic-programming
// column is bit i of a vector of 32-bit words, and the addition and the
// one-row shifts carry from word to word.  One thread per survivor; the
// vertical deltas live in registers, the read's match masks in LDS.
//
// The read fills the vector from the bottom: the rows above it match every
// base and start with vertical delta 0, so they repeat the free boundary row
// (distance 0 at every column, nothing carried out of them), and the read's
// last row is always bit 31 of the last word.  A wavefront therefore runs the
// words from the first one any of its lanes needs to the last, with no
// per-lane branching inside a column.

// 16 read bases starting at base position pos (any alignment; may start
// before the array, whose words count as 0 there and past its end), first
// base in the top bits.
__device__ __forceinline__ uint32_t read_window(const uint32_t *__restrict__ w, uint64_t nw,
                                                int64_t pos)
{
    const int64_t wi = pos >> 4;   // floor, also for negative positions
    const uint32_t sh = (uint32_t)(pos & 15) << 1;
    const uint32_t w0 = wi >= 0 && (uint64_t)wi < nw ? w[wi] : 0u;
    const uint32_t w1 = wi + 1 >= 0 && (uint64_t)(wi + 1) < nw ? w[wi + 1] : 0u;
    return (uint32_t)((((uint64_t)w0 << 32) | w1) >> (32 - sh));
}

// The same for a position inside the array, without branches: bases past the
// array's end come out as anything.
__device__ __forceinline__ uint32_t read_window_in(const uint32_t *__restrict__ w, uint64_t nw,
                                                   uint64_t pos)
{
    const uint64_t wi = pos >> 4;
    const uint32_t sh = (uint32_t)(pos & 15) << 1;
    const uint32_t w0 = w[wi], w1 = w[wi + 1 < nw ? wi + 1 : wi];
    return sh ? __builtin_amdgcn_alignbit(w0, w1, 32 - sh) : w0;
}

// Bits 0, 2, ..., 30 of x gathered into bits 0..15.
__device__ __forceinline__ uint32_t even_bits(uint32_t x)
{
    x = (x | (x >> 1)) & 0x33333333u;
    x = (x | (x >> 2)) & 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    return (x | (x >> 8)) & 0x0000FFFFu;
}

// Three-input bitwise function as gfx950's v_bitop3_b32 immediate: the truth
// table of f read off f(0xF0, 0xCC, 0xAA) (operands a, b, c in that order).
template <uint32_t IMM>
__device__ __forceinline__ uint32_t bitop3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, IMM);
}
constexpr uint32_t kXorOr = ((0xF0u ^ 0xCCu) | 0xAAu) & 0xFFu;   // (a ^ b) | c
constexpr uint32_t kOrNor = (0xF0u | ~(0xCCu | 0xAAu)) & 0xFFu;  // a | ~(b | c)

// The column scan over words S..NW-1 of every lane (S is the same for the
// whole wavefront).  peq_t points at this thread's match masks (64-bit pairs
// of words, base-major, 256 threads apart); rp/wsh locate the span
// in the packed reference.  Returns the smallest distance at the read's last
// row over the span's columns (L when the span is empty).  Per column and
// word, with Pv/Mv the vertical deltas and c the carry of the addition:
//   Xv = Eq | Mv;  Xh = (((Eq & Pv) + Pv + c) ^ Pv) | Eq
//   Ph = Mv | ~(Xh | Pv);  Mh = Pv & Xh
//   Ph, Mh shifted up one row (bit 31 of the word below comes in; 0 at S)
//   Pv = Mh | ~(Xv | Ph);  Mv = Ph & Xv
// and the distance at the last row moves by bit 31 of Ph minus that of Mh.
// UNI: every lane of the wavefront that runs the scan has the same span, so
// the column loop's trip count is uniform (kept in scalar registers).
template <int NW, int S, bool UNI>
__device__ __forceinline__ int32_t column_scan(const uint64_t *peq_t, uint32_t (&pv)[NW],
                                               uint32_t (&mv)[NW], const uint32_t *rp,
                                               uint32_t wsh, uint64_t span, int32_t L)
{
    int32_t score = L, best = L;
    if (UNI)
        span = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(span >> 32)) << 32) |
               __builtin_amdgcn_readfirstlane((uint32_t)span);
    if (span == 0)
        return best;
    // Loads run ahead of their use: the two reference words of the next
    // 16-column fetch one fetch ahead, and each pair of mask words of the
    // next column as soon as the current column is done with that pair.
    // The fetches reach at most three words past the reference's last one;
    // the reference is followed by zero words there (those bases are never
    // used), so the loads are unconditional and nothing waits on them before
    // their use.
    // nxt holds the next fetch's two words in memory order (first word in the
    // low half); they swap halves only where used, so that nothing waits on
    // the load before then
    uint32_t win = (uint32_t)(((uint64_t)rp[0] << 32 | rp[1]) >> (32 - wsh));
    uint64_t nxt;
    __builtin_memcpy(&nxt, rp + 1, 8);
    uint64_t e2[NW / 2];
    {
        const uint64_t *pq = peq_t + __builtin_amdgcn_ubfe(win, 30, 2) * (NW / 2 * 256);
#pragma unroll
        for (int q = S / 2; q < NW / 2; ++q)
            e2[q] = pq[q * 256];
    }
    for (uint64_t j = 0; j < span; ++j) {
        // the next column's base (the 16-base window moves on after column 15)
        const uint32_t col = (uint32_t)j & 15;
        if (col == 15) {
            win = (uint32_t)(((nxt << 32) | (nxt >> 32)) >> (32 - wsh));
            __builtin_memcpy(&nxt, rp + (j >> 4) + 2, 8);
        }
        const uint32_t cbn = __builtin_amdgcn_ubfe(win, 30 - 2 * ((col + 1) & 15), 2);
        const uint64_t *pqn = peq_t + cbn * (NW / 2 * 256);
        uint32_t c = 0, php = 0, mhp = 0;
#pragma unroll
        for (int k = S; k < NW; ++k) {
            const uint32_t eq = (k & 1) ? (uint32_t)(e2[k / 2] >> 32) : (uint32_t)e2[k / 2];
            const uint32_t xv = eq | mv[k];
            const uint32_t sm = __builtin_addc(eq & pv[k], pv[k], c, &c);
            const uint32_t xh = bitop3<kXorOr>(sm, pv[k], eq);
            const uint32_t ph = bitop3<kOrNor>(mv[k], xh, pv[k]);
            const uint32_t mh = pv[k] & xh;
            const uint32_t phs = k == S ? ph << 1 : __builtin_amdgcn_alignbit(ph, php, 31);
            const uint32_t mhs = k == S ? mh << 1 : __builtin_amdgcn_alignbit(mh, mhp, 31);
            php = ph;
            mhp = mh;
            pv[k] = bitop3<kOrNor>(mhs, xv, phs);
            mv[k] = phs & xv;
            if (k & 1) {   // pair k / 2 is done with: load the next column's
                e2[k / 2] = pqn[(k / 2) * 256];
                __builtin_amdgcn_sched_barrier(0);   // keep the load here
            }
        }
        // +1 when bit 31 of Ph is set, -1 when that of Mh is
        score += (int32_t)(php >> 31) + ((int32_t)mhp >> 31);
        best = min(best, score);
    }
    return best;
}

// Picks the scan for the wavefront's first word s (uniform across it).
template <int NW, int S, bool UNI>
__device__ __forceinline__ int32_t column_scan_from(int s, const uint64_t *peq_t,
                                                    uint32_t (&pv)[NW], uint32_t (&mv)[NW],
                                                    const uint32_t *rp, uint32_t wsh,
                                                    uint64_t span, int32_t L)
{
    if constexpr (S + 1 < NW) {
        if (s != S)
            return column_scan_from<NW, S + 1, UNI>(s, peq_t, pv, mv, rp, wsh, span, L);
    }
    return column_scan<NW, S, UNI>(peq_t, pv, mv, rp, wsh, span, L);
}

// Distance of survivor i from the scan of all columns (-1 for a read or bin id out
// of range), by thread t; *ok is set where it is within the read's tolerance.
// peq: room for the match masks of every thread's read, peq[(base * W + block) *
// 256 + thread], block = rows 64 block .. 64 block + 63 of the bottom-aligned
// vector (lane-interleaved, so that a wavefront's reads of one column are
// conflict-free whatever bases its lanes see).
template <int W>
__device__ __forceinline__ int32_t scan_survivor(const VerifyArgs &a, uint64_t i, uint64_t *peq,
                                                 int t, bool *ok)
{
    constexpr int NW = 2 * W;
    const uint64_t nb = a.nw * 16;
    const uint32_t r = a.surv_read[i], b = a.surv_bin[i];
    const uint32_t L = r < a.n_reads ? a.read_len[r] : 0u;
    const uint64_t off = r < a.n_reads ? a.read_off[r] : 0u;
    if (r < a.n_reads && b < a.n_bins && L <= 32u * NW && off <= nb &&
        L <= nb - off) {
        const uint32_t E =
            (uint32_t)(((uint64_t)a.read_e[r] * L + a.e_den - 1) / a.e_den);
        const int pad = 32 * NW - (int)L;   // rows above the read
        uint32_t pv[NW], mv[NW];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            // 16 rows at a time: rows 64 w + 16 g + k (k = 0..15) hold
            // read bases i0 + k, i0 = 64 w + 16 g - pad; rows with
            // i0 + k < 0 match every base
            uint32_t ma[2] = {0u, 0u}, mc[2] = {0u, 0u}, mg[2] = {0u, 0u},
                     mt[2] = {0u, 0u}, pw[2] = {~0u, ~0u};
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int i0 = 64 * w + 16 * g - pad;
                const uint32_t sh = 16 * (g & 1);
                const int half = g >> 1;
                uint32_t xa = 0xFFFFu, xc = 0xFFFFu, xg = 0xFFFFu, xt = 0xFFFFu,
                         pm = 0xFFFFu;
                if (i0 > -16) {
                    pm = i0 >= 0 ? 0u : (1u << -i0) - 1u;
                    // base k in bits 2k (high bit of its code) and 2k + 1 (low bit)
                    const uint32_t rv = __builtin_bitreverse32(
                        read_window(a.rw, a.nw, (int64_t)off + i0));
                    const uint32_t h = rv & 0x55555555u, l = (rv >> 1) & 0x55555555u;
                    xa = even_bits(~(h | l) & 0x55555555u) | pm;
                    xc = even_bits(l & ~h) | pm;
                    xg = even_bits(h & ~l) | pm;
                    xt = even_bits(h & l) | pm;
                }
                ma[half] |= xa << sh;
                mc[half] |= xc << sh;
                mg[half] |= xg << sh;
                mt[half] |= xt << sh;
                pw[half] &= ~(pm << sh);
            }
            peq[(0 * W + w) * 256 + t] = (uint64_t)ma[1] << 32 | ma[0];
            peq[(1 * W + w) * 256 + t] = (uint64_t)mc[1] << 32 | mc[0];
            peq[(2 * W + w) * 256 + t] = (uint64_t)mg[1] << 32 | mg[0];
            peq[(3 * W + w) * 256 + t] = (uint64_t)mt[1] << 32 | mt[0];
            pv[2 * w] = pw[0];
            pv[2 * w + 1] = pw[1];
            mv[2 * w] = mv[2 * w + 1] = 0u;
        }
        const uint64_t lo = (uint64_t)b * a.B;
        uint64_t hi = lo + a.B + a.O;
        if (hi > a.G)
            hi = a.G;
        // an empty read matches anywhere with no edits: no columns
        const uint64_t span = hi > lo && L > 0 ? hi - lo : 0;
        // the wavefront's first word: the most words any of its
        // scanning lanes needs, counted from the bottom
        const uint32_t n = (L + 31) >> 5;
        int nmax = 0;
#pragma unroll
        for (int v = 1; v <= NW; ++v)
            nmax += __builtin_amdgcn_ballot_w64(n >= (uint32_t)v) != 0;
        // 16 reference bases are fetched every 16 columns; their bit
        // offset inside the first packed word is the span start's,
        // the same at every fetch.
        const uint32_t *rp = a.ref + (lo >> 4);
        const uint32_t wsh = ((uint32_t)lo & 15u) << 1;
        // one span for all scanning lanes (all but the last bin's)?
        const uint32_t s_lo = __builtin_amdgcn_readfirstlane((uint32_t)span);
        const uint32_t s_hi = __builtin_amdgcn_readfirstlane((uint32_t)(span >> 32));
        const bool uni = __builtin_amdgcn_ballot_w64(
                             span != ((uint64_t)s_hi << 32 | s_lo)) == 0;
        const int32_t best =
            uni ? column_scan_from<NW, 0, true>(NW - nmax, peq + t, pv, mv, rp, wsh,
                                                span, (int32_t)L)
                : column_scan_from<NW, 0, false>(NW - nmax, peq + t, pv, mv, rp,
                                                 wsh, span, (int32_t)L);
        *ok = best <= (int32_t)E;
        return min<int32_t>(best, (int32_t)E + 1);
    }
    return -1;
}

// ------------------------------------------- location check by exact pieces
// A read of L bases aligned with at most E edits, cut into E + 1 disjoint
// pieces, has one that no edit touches: it occurs unchanged in the span, and the
// whole alignment stays within E diagonals of it (R. Baeza-Yates and C. Perleberg,
// 1992; the pigeonhole principle).  So the scan of all columns is needed only
// where it could matter:
//   A  every survivor's pieces are looked for in its span, by their first
//      kPieceBases bases (E + 1 of them against 160 span positions at a time);
//      a survivor without any is farther than E, and done;
//   B  around the diagonals that were hit, a band of 32, 64 or 128 diagonals is
//      computed row by row of the read (the bit-parallel recurrence again, the
//      vector now along the reference and sliding with the diagonal: H. Hyyro,
//      2003), which gives the distance exactly if it is at most E;
//   C  survivors whose pieces would be shorter than kPieceMin bases (chance hits
//      would be everywhere) or more than kPieces, and those hit all over their
//      span with too many edits to band it, take the scan of all columns below.
//
// The vector ALUs bound it: 2.5M survivors of 100-250 bases at 5-10 % edits take
// 3.9e8 wavefront instructions (1.06e9 with the scan of all columns for each)
// and 0.76 ms (1.64), 0.49 of it phase A; 7.4e4 survivors 0.14 ms (0.41).
constexpr int kPieces = 32;          // pieces at most (E <= 31: two bands of E fit 64 diagonals)
constexpr int kPieceMin = 8;         // bases of a piece at least
constexpr int kPieceBases = 9;       // bases looked for (8 where a lane's pieces have no more)
constexpr int kGroup = 5;            // 32-position words of the span taken together
constexpr int64_t kSpanMax = 30000;  // diagonals are kept in 22 bits with their slot

__device__ __forceinline__ uint32_t lane_max(uint32_t x)
{
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1)
        x = max(x, (uint32_t)__shfl_xor(x, s));
    return __builtin_amdgcn_readfirstlane(x);
}

// The n lowest bits (none for n <= 0, all for n >= 32).
__device__ __forceinline__ uint32_t low_bits(int32_t n)
{
    return n >= 32 ? ~0u : n <= 0 ? 0u : (1u << n) - 1u;
}

constexpr uint32_t kOrXor = (0xF0u | (0xCCu ^ 0xAAu)) & 0xFFu;   // a | (b ^ c)

// Phase A for one wave.  piece: this thread's pieces in LDS (256 threads apart,
// first base in the top bits); np, m: their number and length (np = 0: lane
// idle); p: the span's first reference word pair, sh its first base's bit;
// np_max: the wave's largest; span_max: the longest span, which a lane at the
// reference's end does not reach: p_last is the last word pair it may read.
// [lo, hi] holds the diagonals (span
// position minus read position) of every hit; lo > hi without one.
//
// Cost: the span's 160 positions are held as bit planes of the two code bits,
// shifted by 0 .. 8 positions (90 registers, built once per group of words);
// a piece then takes one v_bitop3 per base, code bit and word, and one
// v_bfe_i32 per base and code bit that broadcasts the piece's own bit: 108
// instructions per piece and 160 positions.
__device__ __forceinline__ void find_pieces(const uint32_t *piece, uint32_t np, uint32_t m,
                                            uint32_t np_max, bool nine, const uint2 *p,
                                            uint32_t p_last, uint32_t sh, int32_t span,
                                            int32_t span_max, int32_t &lo, int32_t &hi)
{
    constexpr int K = kPieceBases;
    lo = 0x3fffffff;
    hi = -0x3fffffff;
    const int bases = nine ? K : K - 1;
    for (int32_t at = 0; at + bases <= span_max; at += 32 * kGroup) {
        uint32_t th[kGroup + 1], tl[kGroup + 1];
        {
            uint2 w[kGroup + 2];
#pragma unroll
            for (int i = 0; i < kGroup + 2; ++i)
                w[i] = p[min((uint32_t)(at >> 5) + i, p_last)];
#pragma unroll
            for (int i = 0; i <= kGroup; ++i) {
                th[i] = __builtin_amdgcn_alignbit(w[i + 1].x, w[i].x, sh);
                tl[i] = __builtin_amdgcn_alignbit(w[i + 1].y, w[i].y, sh);
            }
        }
        uint32_t hs[K][kGroup], ls[K][kGroup], out[kGroup];
#pragma unroll
        for (int w = 0; w < kGroup; ++w) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                hs[j][w] = j ? __builtin_amdgcn_alignbit(th[w + 1], th[w], j) : th[w];
                ls[j][w] = j ? __builtin_amdgcn_alignbit(tl[w + 1], tl[w], j) : tl[w];
            }
            // positions too close to the span's end
            out[w] = ~low_bits(span - bases + 1 - at - 32 * w);
        }
        for (uint32_t i = 0; i < np_max; ++i) {
            const int32_t win = (int32_t)piece[i * 256];
            uint32_t miss[kGroup];
#pragma unroll
            for (int w = 0; w < kGroup; ++w)
                miss[w] = out[w];
#pragma unroll
            for (int j = 0; j < K - 1; ++j) {
                const uint32_t bh = (win << (2 * j)) >> 31, bl = (win << (2 * j + 1)) >> 31;
#pragma unroll
                for (int w = 0; w < kGroup; ++w) {
                    miss[w] = bitop3<kOrXor>(miss[w], hs[j][w], bh);
                    miss[w] = bitop3<kOrXor>(miss[w], ls[j][w], bl);
                }
            }
            if (nine) {
                const uint32_t bh = (win << (2 * K - 2)) >> 31, bl = (win << (2 * K - 1)) >> 31;
#pragma unroll
                for (int w = 0; w < kGroup; ++w) {
                    miss[w] = bitop3<kOrXor>(miss[w], hs[K - 1][w], bh);
                    miss[w] = bitop3<kOrXor>(miss[w], ls[K - 1][w], bl);
                }
            }
            uint32_t all = miss[0];
#pragma unroll
            for (int w = 1; w < kGroup; ++w)
                all &= miss[w];
            if (all != ~0u && i < np) {
                // first and last hit of the group (a word without one saturates)
                uint32_t a = ~0u, z = 0u;
#pragma unroll
                for (int w = 0; w < kGroup; ++w) {
                    const uint32_t x = ~miss[w];
                    a = min(a, __builtin_elementwise_add_sat((uint32_t)(__ffs(x) - 1), 32u * w));
                    z = max(z, __builtin_elementwise_sub_sat(
                                   32u * w + 31u, x ? (uint32_t)__builtin_clz(x) : ~0u));
                }
                const int32_t base = at - (int32_t)(i * m);
                lo = min(lo, base + (int32_t)a);
                hi = max(hi, base + (int32_t)z);
            }
        }
    }
}

// Phase B for one wave: smallest distance of the lane's read (L bases at `off`)
// to any substring of its span, over the alignments inside the NB * 32 diagonals
// from dlo on; never less than the true smallest distance.  p: first reference
// word pair of the whole array's base 0; lo: the span's first base.
//
// Row i, bit b is the cell (i, i + dlo + b); Pv/Mv hold the differences along
// the row, aligned for the next row.  Positions outside the span match nothing,
// which costs the same edits as the span's edge does.  Per row and 32 diagonals,
// with Eq the matches of the row's base:
//   D0 = (((Eq & Pv) + Pv) ^ Pv) | Eq | Mv   (equal to its diagonal neighbour)
//   Hp = Mv | ~(D0 | Pv);  Hn = Pv & D0;  X = D0 >> 1
//   Pv = Hn | ~(X | Hp);   Mv = X & Hp
// about 17 instructions (33 for 64 diagonals, 65 for 128), no memory but a word
// pair every 32 rows and a read word every 16.
template <int NB>
__device__ __forceinline__ int32_t band_scan(const uint2 *p, int64_t lo, int32_t dlo, int32_t span,
                                             const uint32_t *__restrict__ rw, uint64_t nw,
                                             uint64_t off, int32_t L)
{
    const int64_t t0 = lo + dlo;                     // reference position of row 0, bit 0
    const uint2 *q = p + (t0 >> 5);                  // floor, also for negative positions
    const uint32_t sh = (uint32_t)t0 & 31u;
    uint32_t th[NB + 1], tl[NB + 1], tv[NB + 1];     // aligned words, and which positions count
    // loads run one use ahead: the next word pair of the reference, the next word
    // of the read (the last one again past its end)
    uint2 raw = q[0], ahead = q[1];
    auto fetch = [&](int n, int slot) {
        th[slot] = __builtin_amdgcn_alignbit(ahead.x, raw.x, sh);
        tl[slot] = __builtin_amdgcn_alignbit(ahead.y, raw.y, sh);
        raw = ahead;
        ahead = q[n + 2];
        const int32_t x = dlo + 32 * n;
        tv[slot] = low_bits(span - x) & ~low_bits(-x);
    };
#pragma unroll
    for (int n = 0; n < NB; ++n)
        fetch(n, n);
    uint32_t pv[NB], mv[NB];
#pragma unroll
    for (int w = 0; w < NB; ++w)
        pv[w] = mv[w] = 0u;
    const uint32_t *r = rw + (off >> 4);
    const uint64_t r_last = nw - 1 - (off >> 4);
    const uint32_t rsh = (uint32_t)(off & 15) << 1;
    auto word = [&](uint64_t n) { return r[n < r_last ? n : r_last]; };
    uint32_t c0 = word(0), c1 = word(1), c2 = word(2);
    int32_t s = L;
    int32_t win = 0;
    for (int32_t i = 0; i < L; ++i) {
        const uint32_t k = (uint32_t)i & 31u;
        if (k == 0) {
            if (i) {
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    th[n] = th[n + 1];
                    tl[n] = tl[n + 1];
                    tv[n] = tv[n + 1];
                }
            }
            fetch((i >> 5) + NB, NB);
        }
        if ((k & 15u) == 0) {
            win = (int32_t)(rsh ? __builtin_amdgcn_alignbit(c0, c1, 32 - rsh) : c0);
            c0 = c1;
            c1 = c2;
            c2 = word((i >> 4) + 3);
        }
        const uint32_t bh = win >> 31, bl = (win << 1) >> 31;
        win <<= 2;
        uint32_t eq[NB], d0[NB], c = 0;
#pragma unroll
        for (int w = 0; w < NB; ++w) {
            const uint32_t a = __builtin_amdgcn_alignbit(th[w + 1], th[w], k);
            const uint32_t b = __builtin_amdgcn_alignbit(tl[w + 1], tl[w], k);
            const uint32_t v = __builtin_amdgcn_alignbit(tv[w + 1], tv[w], k);
            const uint32_t ne = (b ^ bl) | ~v;
            eq[w] = ~((a ^ bh) | ne);
            const uint32_t sm = __builtin_addc(eq[w] & pv[w], pv[w], c, &c);
            d0[w] = bitop3<kXorOr>(sm, pv[w], eq[w] | mv[w]);
        }
        s -= (int32_t)(d0[0] & 1u);
#pragma unroll
        for (int w = 0; w < NB; ++w) {
            const uint32_t x = w + 1 < NB ? __builtin_amdgcn_alignbit(d0[w + 1 < NB ? w + 1 : w], d0[w], 1)
                                          : d0[w] >> 1;
            const uint32_t hp = bitop3<kOrNor>(mv[w], d0[w], pv[w]);
            const uint32_t hn = pv[w] & d0[w];
            pv[w] = bitop3<kOrNor>(hn, x, hp);
            mv[w] = x & hp;
        }
    }
    // s is the last row's cell on the lowest diagonal; the others by the row's
    // differences
    int32_t best = s;
#pragma unroll
    for (int w = 0; w < NB; ++w) {
#pragma unroll
        for (int b = 0; b < 32; ++b) {
            if (w == NB - 1 && b == 31)
                break;
            s += (int32_t)((pv[w] >> b) & 1u) - (int32_t)((mv[w] >> b) & 1u);
            best = min(best, s);
        }
    }
    return best;
}

// Each workgroup owns one contiguous range of survivors: one chunk of CH, or a
// run of whole chunks once the list exceeds 64 times the workgroups the GPU
// holds at once (ranges start on multiples of 32, so that no two workgroups
// share a word of pass bits).  It takes its range CH survivors at a time and
// sorts them (counting sort in LDS): those whose pieces are looked for by their
// tolerated edits, as many pieces as that takes, then the others by the number
// of 32-row words of their read, empty slots of a short last chunk last.  Phase
// A runs over the first part, 64 sorted slots a wavefront, drawn from LDS with the
// most pieces first; phase B over the bands it leaves (narrow ones listed from
// the front, wide ones from the back, broad ones apart, so that a wavefront has
// one kind), the longest first; phase C over the second part and the few
// survivors whose bands found no room.  A survivor's smallest distance is
// collected in LDS as twice the distance, or 2 E + 1 while none within E is
// known; distances and pass bits leave together.  W is the number of 64-row
// blocks (NW = 2 W words) the batch's longest read needs.
//
// SCAN: phase C is the end of the same kernel (short lists, where a second launch
// costs more than it saves).  Else it is verify_scan_kernel's, for the survivors
// marked with kScanMark in place of a distance: beside phase A's registers and LDS
// the scan has 3 wavefronts a SIMD, by itself 8 (4 and 2 for reads of over 128 and
// 256 bases), and idle ones in chunks of which only a part comes to it (2.5e6
// survivors of 100 bases at 15 % edits 1.26 ms, 1.47 in one kernel, 1.32 with the scan
// alone for every survivor; of 64-250 bases at 8 and 15 % 1.89, 2.29 and 1.99).  A few
// survivors alone take it 110 us, so the list of broad bands has room for those of
// repeats too (2.8e5 survivors of 250 bases, seeds in repeats: 424 us, 533 with 512).
constexpr int kVerifyChunk = 1024;
constexpr int kVerifySmall = 256;
constexpr int32_t kScanMark = INT32_MIN;

template <int W, int CH, bool SCAN>
__global__ __launch_bounds__(256, W > 4 ? 2 : 3) void verify_kernel(VerifyArgs a)
{
    constexpr int NW = 2 * W;
    constexpr int kKeys = kPieces + (SCAN ? NW : 0) + 2;   // edits | words | past the chunk's end
    constexpr uint32_t kSettled = ~0u;        // written to memory already
    constexpr uint32_t kBroad = SCAN ? 512 : CH + CH / 2;   // as many as LDS has room for
    constexpr int U = CH / 256;   // slots per thread
    static_assert(kKeys <= 64, "one wavefront scans the keys");
    __shared__ uint16_t order[CH];
    __shared__ uint32_t cls[64];
    __shared__ uint32_t okw[CH / 32];
    __shared__ uint32_t best[CH];
    // bands to compute (a survivor has one narrow or wide one, or broad ones): slot in
    // the low 10 bits, first diagonal + 8192 above
    __shared__ uint32_t bands[CH], broad[kBroad];
    __shared__ uint16_t rest[CH];             // survivors of phase A for phase C
    __shared__ uint32_t n_narrow, n_wide, n_broad, n_rest;
    __shared__ uint32_t next_a, next_b;       // wavefront runs of phases A and B handed out
    // phase A: pieces[piece * 256 + thread]; phase C: match masks
    __shared__ uint64_t peq[(SCAN && W > 4 ? 4 * W : 16) * 256];
    uint32_t *pieces = reinterpret_cast<uint32_t *>(peq);
    const int t = threadIdx.x, lane = t & 63;
    auto draw = [&](uint32_t *next) -> uint32_t {
        uint32_t x = 0;
        if (lane == 0)
            x = atomicAdd(next, 1u);
        return __builtin_amdgcn_readfirstlane(x);
    };
    const uint32_t max_rows = SCAN ? 32u * NW : a.max_rows;
    const uint64_t nb = a.nw * 16;
    const uint64_t per = ((a.n_surv + gridDim.x - 1) / gridDim.x + 31) & ~31ull;
    const uint64_t g0 = (uint64_t)blockIdx.x * per;
    const uint64_t g1 = g0 + per < a.n_surv ? g0 + per : a.n_surv;
    auto span_of = [&](uint64_t lo) -> uint64_t {
        uint64_t hi = lo + a.B + a.O;
        if (hi > a.G)
            hi = a.G;
        return hi > lo ? hi - lo : 0;
    };
    // the longest span, in 32 bits: batches with longer ones have no survivor
    // in phases A and B
    const uint64_t span_all = a.B + a.O < a.G ? a.B + a.O : a.G;
    for (uint64_t base = g0; base < g1; base += CH) {
        const uint32_t cnt = (uint32_t)(g1 - base < (uint64_t)CH ? g1 - base : CH);
        if (t < 64)
            cls[t] = 0;
        if (t < CH / 32)
            okw[t] = 0;
        if (t == 0)
            n_narrow = n_wide = n_broad = n_rest = next_a = next_b = 0;
        __syncthreads();
        // class of slot u 256 + t
        int key[U];
        uint32_t rank[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t p = u * 256 + t;
            int k = kKeys - 1;
            if (p < cnt) {
                k = kPieces;
                const uint32_t r = a.surv_read[base + p], b = a.surv_bin[base + p];
                if (r < a.n_reads) {
                    const uint32_t L = a.read_len[r];
                    if (SCAN && L <= max_rows)
                        k = kPieces + (int)((L + 31) >> 5);
                    const uint64_t off = a.read_off[r];
                    const uint64_t E = ((uint64_t)a.read_e[r] * L + a.e_den - 1) / a.e_den;
                    if (b < a.n_bins && L <= max_rows && off <= nb && L <= nb - off &&
                        E < (uint64_t)kPieces && L >= (E + 1) * kPieceMin &&
                        span_all <= (uint64_t)kSpanMax) {
                        k = (int)E;
                        best[p] = 2 * (uint32_t)E + 1;   // more than E
                    }
                }
            }
            key[u] = k;
            rank[u] = atomicAdd(&cls[k], 1u);
        }
        __syncthreads();
        if (t < 64) {   // first slot of every class
            const uint32_t n = cls[t];
            uint32_t before = n;
#pragma unroll
            for (int s = 1; s < 64; s <<= 1) {
                const uint32_t y = __shfl_up(before, s);
                if (t >= s)
                    before += y;
            }
            cls[t] = before - n;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u)
            order[cls[key[u]] + rank[u]] = (uint16_t)(u * 256 + t);
        // survivors of phase A; where they are few they go to the scan as well: a
        // chunk with 141 of 1024 takes 100 us here, its wavefronts one run each and
        // the others waiting, and their scan no longer
        uint32_t n_pieces = __builtin_amdgcn_readfirstlane(cls[kPieces]);
        if (!SCAN && n_pieces * 6 < cnt)
            n_pieces = 0;
        __syncthreads();

        // ------------------------------------------------ phase A: pieces
        // the bands of a survivor whose pieces hit on diagonals h0 .. h1: one
        // where the hits lie together (nearly always), else as many of 128
        // diagonals as it takes to cover all of them
        auto settle = [&](uint32_t slot, int32_t E, int32_t h0, int32_t h1) {
            auto entry = [&](int32_t first) { return slot | (uint32_t)(first - E + 8192) << 10; };
            bool done = true;
            if (h1 - h0 < 64 - 2 * E) {
                const uint32_t at = h1 - h0 < 32 - 2 * E ? atomicAdd(&n_narrow, 1u)
                                                         : CH - 1 - atomicAdd(&n_wide, 1u);
                bands[at] = entry(h0);
            } else {
                const int32_t step = 128 - 2 * E;
                for (; done && h0 <= h1; h0 += step) {
                    const uint32_t at = atomicAdd(&n_broad, 1u);
                    done = at < kBroad;
                    if (done)
                        broad[at] = entry(h0);
                }
            }
            if (!done) {
                rest[atomicAdd(&n_rest, 1u)] = (uint16_t)slot;
                best[slot] = kSettled;
            }
        };
        for (;;) {
            const uint32_t run = draw(&next_a);
            if (run * kWave >= n_pieces)
                break;
            const uint32_t x0 = ((n_pieces - 1) / kWave - run) * kWave;   // most pieces first
            const bool on = x0 + lane < n_pieces;
            const uint32_t slot = order[on ? x0 + lane : x0];
            const uint32_t r = a.surv_read[base + slot], b = a.surv_bin[base + slot];
            const int32_t L = (int32_t)a.read_len[r];
            const uint64_t off = a.read_off[r];
            const int32_t E = (int32_t)(best[slot] >> 1);
            const uint32_t m = (uint32_t)L / (uint32_t)(E + 1);
            const uint32_t np = on ? (uint32_t)E + 1 : 0u;
            const uint32_t np_max = lane_max(np);
            const bool nine = __builtin_amdgcn_ballot_w64(m < kPieceBases) == 0;
#pragma unroll 4
            for (uint32_t i = 0; i < np_max; ++i)
                pieces[i * 256 + t] = read_window_in(a.rw, a.nw, off + (i < np ? i * m : 0u));
            const uint64_t lo = (uint64_t)b * a.B;
            const int32_t span = (int32_t)span_of(lo);
            int32_t h0, h1;
            const uint64_t p_left = (a.ref_words + 1) / 2 + kPlanePad - 1 - (lo >> 5);
            find_pieces(pieces + t, np, m, np_max, nine, a.planes + (lo >> 5),
                        (uint32_t)min<uint64_t>(p_left, ~0u), (uint32_t)lo & 31u, span,
                        (int32_t)span_all, h0, h1);
            if (on && h0 <= h1)
                settle(slot, E, h0, h1);
        }
        __syncthreads();

        // ------------------------------------------------- phase B: bands
        // runs of one kind, the longest first
        const uint32_t n1 = n_narrow, n2 = n_wide, n4 = min(n_broad, kBroad);
        const uint32_t end4 = (n4 + kWave - 1) / kWave * kWave;
        const uint32_t end2 = end4 + (n2 + kWave - 1) / kWave * kWave;
        for (;;) {
            const uint32_t x0 = draw(&next_b) * kWave;
            if (x0 >= end2 + n1)
                break;
            const int kind = x0 < end4 ? 4 : x0 < end2 ? 2 : 1;
            const uint32_t x = x0 + lane - (kind == 4 ? 0u : kind == 2 ? end4 : end2);
            if (x < (kind == 4 ? n4 : kind == 2 ? n2 : n1)) {
                const uint32_t e = kind == 4 ? broad[x] : bands[kind == 2 ? CH - 1 - x : x];
                const uint32_t slot = e & 1023u;
                const int32_t dlo = (int32_t)(e >> 10) - 8192;
                const uint32_t v = best[slot];
                if (v != kSettled) {
                    const uint32_t r = a.surv_read[base + slot], b = a.surv_bin[base + slot];
                    const int32_t L = (int32_t)a.read_len[r];
                    const uint64_t off = a.read_off[r];
                    const int64_t lo = (int64_t)((uint64_t)b * a.B);
                    const int32_t span = (int32_t)span_of((uint64_t)lo);
                    int32_t d;
                    if (kind == 1)
                        d = band_scan<1>(a.planes, lo, dlo, span, a.rw, a.nw, off, L);
                    else if (kind == 2)
                        d = band_scan<2>(a.planes, lo, dlo, span, a.rw, a.nw, off, L);
                    else
                        d = band_scan<4>(a.planes, lo, dlo, span, a.rw, a.nw, off, L);
                    atomicMin(&best[slot], 2u * (uint32_t)d);
                }
            }
        }
        __syncthreads();

        // --------------------------------------------- phase C: all columns
        const uint32_t n_all = cls[kKeys - 1] - n_pieces;   // survivors without pieces
        for (uint32_t x = t; x < n_all + n_rest; x += 256) {
            const uint32_t slot = x < n_all ? order[n_pieces + x] : rest[x - n_all];
            if constexpr (SCAN) {
                bool ok = false;
                a.dist[base + slot] = scan_survivor<W>(a, base + slot, peq, t, &ok);
                if (ok)
                    atomicOr(&okw[slot >> 5], 1u << (slot & 31));
            } else {
                a.dist[base + slot] = kScanMark;
            }
        }
        // distances of phases A and B
        for (uint32_t x = t; x < n_pieces; x += 256) {
            const uint32_t slot = order[x];
            const uint32_t v = best[slot];
            if (v != kSettled) {
                a.dist[base + slot] = (int32_t)((v + 1) >> 1);
                if (!(v & 1u))
                    atomicOr(&okw[slot >> 5], 1u << (slot & 31));
            }
        }
        __syncthreads();
        if (t < (int)((cnt + 31) / 32))
            a.ok_bits[(base >> 5) + t] = okw[t];
        __syncthreads();
    }
}

// Phase C by itself, in ranges like verify_kernel's and chunks of 256: the
// survivors that kernel marked (ALL: every survivor, of batches it is not run on),
// sorted by the number of 32-row words of their read (counting sort in LDS) so
// that a wavefront starts at one word.  Chunks of 1024 sort better but leave the
// last round of workgroups nearly empty (5e5 survivors of 100 bases at 15 % edits
// 359 us, 512 248, 256 223; 2.5e6 of 100-250 bases 2.09 ms, 1.96, 1.85).
template <int W, bool ALL>
__global__ __launch_bounds__(256, W <= 2 ? 8 : W <= 4 ? 4 : 2) void verify_scan_kernel(VerifyArgs a)
{
    constexpr int NW = 2 * W;
    constexpr uint32_t CH = kVerifySmall;
    __shared__ uint16_t order[CH];
    __shared__ uint32_t cls[NW + 1], okw[CH / 32];
    __shared__ uint64_t peq[4 * W * 256];
    const uint32_t t = threadIdx.x;
    const uint64_t per = ((a.n_surv + gridDim.x - 1) / gridDim.x + 31) & ~31ull;
    const uint64_t g0 = (uint64_t)blockIdx.x * per;
    const uint64_t g1 = g0 + per < a.n_surv ? g0 + per : a.n_surv;
    for (uint64_t base = g0; base < g1; base += CH) {
        const uint32_t cnt = (uint32_t)(g1 - base < CH ? g1 - base : CH);
        const bool mine = t < cnt && (ALL || a.dist[base + t] == kScanMark);
        if (!__syncthreads_or(mine))
            continue;
        if (t < NW + 1)
            cls[t] = 0;
        if (t < CH / 32)
            okw[t] = 0;
        __syncthreads();
        // class of survivor t: its read's word count, 0 when there is nothing to align
        uint32_t key = 0, rank = 0;
        if (mine) {
            const uint32_t r = a.surv_read[base + t];
            const uint32_t L = r < a.n_reads ? a.read_len[r] : 0u;
            key = L <= 32u * NW ? (L + 31) >> 5 : 0u;
            rank = atomicAdd(&cls[key], 1u);
        }
        __syncthreads();
        uint32_t before = 0, n = 0;
        for (uint32_t c = 0; c <= (uint32_t)NW; ++c) {
            before += c < key ? cls[c] : 0u;
            n += cls[c];
        }
        if (mine)
            order[before + rank] = (uint16_t)t;
        __syncthreads();
        if (t < n) {
            const uint32_t slot = order[t];
            bool ok = false;
            a.dist[base + slot] = scan_survivor<W>(a, base + slot, peq, t, &ok);
            if (ok)
                atomicOr(&okw[slot >> 5], 1u << (slot & 31));
        }
        __syncthreads();
        if (t < (cnt + 31) / 32) {
            uint32_t *w = &a.ok_bits[(base >> 5) + t];   // this workgroup's alone
            *w = ALL ? okw[t] : *w | okw[t];
        }
        __syncthreads();
    }
}

// Splits the packed reference into bit planes: word pair j holds the high (x) and
// low (y) code bits of bases 32 j .. 32 j + 31, the first in bit 0.
__global__ __launch_bounds__(256) void planes_kernel(const uint32_t *__restrict__ ref, uint64_t nw,
                                                     uint64_t n_pairs, uint2 *__restrict__ out)
{
    const uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= n_pairs)
        return;
    const uint32_t r0 = __builtin_bitreverse32(ref[2 * j]);   // 2 j < nw
    const uint32_t r1 = __builtin_bitreverse32(2 * j + 1 < nw ? ref[2 * j + 1] : 0u);
    out[j] = make_uint2(even_bits(r0 & 0x55555555u) | even_bits(r1 & 0x55555555u) << 16,
                        even_bits((r0 >> 1) & 0x55555555u) |
                            even_bits((r1 >> 1) & 0x55555555u) << 16);
}

hipError_t launch_planes(hipStream_t s, const uint32_t *ref, uint64_t nw, uint2 *planes)
{
    const uint64_t n_pairs = (nw + 1) / 2;
    if (n_pairs)
        hipLaunchKernelGGL(planes_kernel, dim3((uint32_t)((n_pairs + 255) / 256)), dim3(256), 0, s,
                           ref, nw, n_pairs, planes);
    return hipGetLastError();
}

// Launches kernel k over the survivors, a sorted chunk per workgroup, dispatched as
// resident ones finish; past 64 times the resident count each takes a run of whole
// chunks.  resident: workgroups a CU holds (LDS or register bound), asked once per
// kernel and process; it only sizes the grid's cap, never what is computed.
static hipError_t launch_chunks(hipStream_t s, const void *k, std::atomic<int> &resident, int cus,
                                uint64_t chunk, const VerifyArgs &a)
{
    int per_cu = resident.load(std::memory_order_relaxed);
    if (per_cu <= 0) {
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, 256, 0);
        if (e != hipSuccess)
            return e;
        if (per_cu <= 0)
            per_cu = 1;
        resident.store(per_cu, std::memory_order_relaxed);
    }
    const uint64_t chunks = (a.n_surv + chunk - 1) / chunk;
    const uint64_t cap = (uint64_t)per_cu * (uint64_t)(cus > 0 ? cus : 1) * 64;
    const uint64_t m = (chunks + cap - 1) / cap;
    const uint64_t grid = (chunks + m - 1) / m;
    if (grid == 0)
        return hipSuccess;
    VerifyArgs copy = a;
    void *args[] = {&copy};
    return hipLaunchKernel(k, dim3((uint32_t)grid), dim3(256), args, 0, s);
}

template <int W>
static hipError_t launch_verify_w(hipStream_t s, int cus, const VerifyArgs &a)
{
    static std::atomic<int> resident[4];
    const void *all = reinterpret_cast<const void *>(&verify_scan_kernel<W, true>);
    const void *marked = reinterpret_cast<const void *>(&verify_scan_kernel<W, false>);
    const void *small = reinterpret_cast<const void *>(&verify_kernel<W, kVerifySmall, true>);
    const void *large = reinterpret_cast<const void *>(&verify_kernel<1, kVerifyChunk, false>);
    const uint64_t span = a.B + a.O < a.G ? a.B + a.O : a.G;
    if (!a.planes || span > (uint64_t)kSpanMax)   // no survivor has pieces
        return launch_chunks(s, all, resident[0], cus, kVerifySmall, a);
    // chunks of 1024 sort and pack better (2.5M survivors: 512 9 % slower; 5.3e5:
    // 246 us, 256 327 us); lists that would leave CUs without one take chunks of
    // 256 (7.4e4: 0.14 ms; 64, the wavefronts sharing each survivor's pieces, took a
    // fifth longer)
    if (a.n_surv < (uint64_t)(cus > 0 ? cus : 1) * kVerifyChunk)
        return launch_chunks(s, small, resident[1], cus, kVerifySmall, a);
    const hipError_t e = launch_chunks(s, large, resident[2], cus, kVerifyChunk, a);
    if (e != hipSuccess)
        return e;
    return launch_chunks(s, marked, resident[3], cus, kVerifySmall, a);
}

hipError_t launch_verify(hipStream_t s, int W, int cus, const VerifyArgs &a)
{
    VerifyArgs b = a;
    b.max_rows = 64u * (uint32_t)W;
    switch (W) {
    case 1: return launch_verify_w<1>(s, cus, b);
    case 2: return launch_verify_w<2>(s, cus, b);
    case 4: return launch_verify_w<4>(s, cus, b);
    case 8: return launch_verify_w<8>(s, cus, b);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace grim
