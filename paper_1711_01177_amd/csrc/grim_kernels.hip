// GRIM-Filter HIP kernels for gfx950 (MI355X).
//
// The filter (Kim et al., BMC Genomics 2018, Sections "GRIM-Filter Operation"
// and "Taking Errors into Account") is an integer gather + popcount: for each
// (read, candidate bin) pair, sum over the read's token positions the bin's
// existence bit of that token, then compare with T = ntok - q * ceil(e L).
//
// Decomposition used on the GPU (exact, no approximation):
//   Let m(t) be the number of positions of the read whose token is t.  Then
//     sum_i V[tok_i] = sum_t m(t) V[t] = sum_k 2^k popcount(M_k & V)
//   where M_k is the bit plane holding bit k of m(t) for every token t.  The
//   planes of one read are built once in LDS with atomic-xor carry chains (an
//   increment of a bit-sliced counter), so the per-candidate work is a few
//   AND + popcount per 16-byte slice of the candidate's vector, independent of
//   the read length, with repeated tokens counted exactly.
//
// Memory layout: bin vectors bin-major, 4^q / 8 bytes each, so one candidate
// is one contiguous 32 B .. 2 KiB run; G lanes load it with 16-byte loads.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "grim_device.h"
#include "grim_internal.h"

namespace grim {

// ------------------------------------------------------------ device helpers
// Orders the LDS traffic of one wavefront across phases (build planes, read
// planes, reuse).  Waves of a workgroup never share LDS regions in these
// kernels, so wavefront scope is enough and no memory counters are drained.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t uniform_u32(uint32_t x)
{
    return __builtin_amdgcn_readfirstlane(x);
}

__device__ __forceinline__ uint64_t uniform_u64(uint64_t x)
{
    uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Token of Q bases starting at stream position pos of a packed sequence
// (16 bases per word, first base in the top bits): a funnel shift of two
// adjacent words.  Reads past the end of the buffer see zero words.
template <int Q>
__device__ __forceinline__ uint32_t token_at(const uint32_t *__restrict__ w, uint64_t nw,
                                             uint64_t pos)
{
    const uint64_t wi = pos >> 4;
    const uint32_t sh = (uint32_t)(pos & 15u) << 1;
    uint64_t x = (uint64_t)(wi < nw ? w[wi] : 0u) << 32;
    if (sh + 2 * Q > 32)
        x |= (wi + 1 < nw ? w[wi + 1] : 0u);
    return (uint32_t)((x << sh) >> (64 - 2 * Q));
}

__device__ __forceinline__ uint32_t popc_and(const uint4 &a, const uint4 &b)
{
    return __popc(a.x & b.x) + __popc(a.y & b.y) + __popc(a.z & b.z) + __popc(a.w & b.w);
}

// Add one read's tokens to its multiplicity bit planes in LDS (one wave); the
// npl planes of VW words each are zero on entry.  Returns the number of planes
// in use (0 for a read without tokens).  npl is chosen by the host so that
// 2^npl > ntok, hence no carry can leave the last plane.
template <int Q>
__device__ int add_planes(uint32_t *planes, int npl, const uint32_t *__restrict__ rw, uint64_t nw,
                          uint64_t off, uint32_t ntok, int lane)
{
    constexpr int VW = (1 << (2 * Q)) >> 5;
    int top = 0;
    for (uint32_t i = lane; i < ntok; i += kWave) {
        const uint32_t t = token_at<Q>(rw, nw, off + i);
        const uint32_t wd = t >> 5, bit = 1u << (t & 31u);
        int k = 0;
        uint32_t old = atomicXor(&planes[wd], bit);
        while ((old & bit) && k + 1 < npl) {
            ++k;
            old = atomicXor(&planes[k * VW + wd], bit);
        }
        top = max(top, k + 1);
    }
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1)
        top = max(top, __shfl_xor(top, s));
    wave_fence();
    return top;
}

// The same on planes with any contents: clears them first.
template <int Q>
__device__ int build_planes(uint32_t *planes, int npl, const uint32_t *__restrict__ rw, uint64_t nw,
                            uint64_t off, uint32_t ntok, int lane)
{
    constexpr int VW = (1 << (2 * Q)) >> 5;
    for (int i = lane; i < npl * VW; i += kWave)
        planes[i] = 0u;
    wave_fence();
    return add_planes<Q>(planes, npl, rw, nw, off, ntok, lane);
}

__device__ __forceinline__ void flag(uint32_t *status, uint32_t f)
{
    atomicOr(status, f);
}

// ---------------------------------------------------------------- bin build
// One wavefront per bin (grid-stride): every lane takes every 64th token start
// of the bin's span and sets the token's bit in an LDS copy of the vector,
// which is then written out whole.  Bin b spans [b*B, min(G, (b+1)*B + O)).
template <int Q>
__global__ __launch_bounds__(256) void build_bins_kernel(const uint32_t *__restrict__ ref,
                                                         uint64_t nw, uint64_t G, uint64_t B,
                                                         uint64_t O, uint64_t n_bins,
                                                         uint32_t *__restrict__ out)
{
    constexpr int VW = (1 << (2 * Q)) >> 5;
    __shared__ uint32_t vec_lds[4][VW];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t *vec = vec_lds[wv];
    for (uint64_t b = (uint64_t)blockIdx.x * 4 + wv; b < n_bins; b += (uint64_t)gridDim.x * 4) {
        for (int i = lane; i < VW; i += kWave)
            vec[i] = 0u;
        wave_fence();
        const uint64_t lo = b * B;
        uint64_t hi = (b + 1) * B + O;
        if (hi > G)
            hi = G;
        for (uint64_t p = lo + lane; p + Q <= hi; p += kWave) {
            const uint32_t t = token_at<Q>(ref, nw, p);
            atomicOr(&vec[t >> 5], 1u << (t & 31u));
        }
        wave_fence();
        uint32_t *dst = out + b * VW;
        for (int i = lane; i < VW; i += kWave)
            dst[i] = vec[i];
        wave_fence();
    }
}

// ---------------------------------------------------------------- work list
// Ticket k of the batched filter is one run of consecutive pairs: the first
// n_big tickets hold big_pairs pairs each, the rest small_pairs.
__device__ __forceinline__ uint64_t ticket_start(uint32_t k, uint32_t n_big, uint32_t big_pairs,
                                                 uint32_t small_pairs)
{
    return k < n_big ? (uint64_t)k * big_pairs
                     : (uint64_t)n_big * big_pairs + (uint64_t)(k - n_big) * small_pairs;
}

// Thread i < n_table records the read that owns the first pair of ticket i: the
// last read r with cand_off[r] <= that pair.  Thread 0 also resets the status
// word and the ticket counters of this launch: wave w of the n_waves that the
// filter runs starts with ticket w, so counter c starts at the number of waves
// w with w % kTicketCounters == c.
__global__ __launch_bounds__(256) void worklist_kernel(const uint64_t *__restrict__ cand_off,
                                                       uint64_t n_reads, uint32_t n_table,
                                                       uint32_t n_big, uint32_t big_pairs,
                                                       uint32_t small_pairs, uint32_t n_waves,
                                                       uint32_t *ticket_read, uint32_t *status,
                                                       uint32_t *counters)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) {
        *status = 0u;
        for (uint32_t c = 0; c < kTicketCounters; ++c)
            counters[c * kTicketStride] = (n_waves + kTicketCounters - 1 - c) / kTicketCounters;
    }
    if (i >= n_table || n_reads == 0)
        return;
    const uint64_t p = ticket_start((uint32_t)i, n_big, big_pairs, small_pairs);
    uint64_t lo = 0, hi = n_reads - 1;
    while (lo < hi) {
        const uint64_t mid = (lo + hi + 1) >> 1;
        if (cand_off[mid] <= p)
            lo = mid;
        else
            hi = mid - 1;
    }
    ticket_read[i] = (uint32_t)lo;
}

__global__ void zero_words_kernel(uint32_t *p, uint64_t n)
{
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

__global__ void zero_words2_kernel(uint32_t *p, uint64_t n, uint32_t *p2, uint64_t n2)
{
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n + n2;
         i += (uint64_t)gridDim.x * blockDim.x)
        (i < n ? p[i] : p2[i - n]) = 0u;
}

// ----------------------------------------------------------- batched filter
// Sums acc[0 .. U) over the G lanes of a group: lane lg ends with the group's
// total of acc[lg % U] (U <= G).  log2 U exchange steps halve the values that
// travel, the rest of the group is a butterfly on the one value left.
template <int G, int U>
__device__ __forceinline__ uint32_t group_sums(uint32_t (&acc)[U], int lane)
{
#pragma unroll
    for (int n = U / 2, m = 1; n >= 1; n /= 2, m *= 2) {
        const bool hi = (lane & m) != 0;
#pragma unroll
        for (int j = 0; j < n; ++j) {
            const uint32_t keep = hi ? acc[2 * j + 1] : acc[2 * j];
            const uint32_t send = hi ? acc[2 * j] : acc[2 * j + 1];
            acc[j] = keep + lane_xor(send, m);
        }
    }
#pragma unroll
    for (int m = U; m < G; m *= 2)
        acc[0] += lane_xor(acc[0], m);
    return acc[0];
}

// Bin id of pair u of a group, ids held one pair a lane, the group's first pair
// in lane `first`: within a quad a DPP broadcast where a group is one.
template <int G, int U>
__device__ __forceinline__ uint32_t group_id(uint32_t ids, int first, int u)
{
    if constexpr (G == 4 && U == 4) {
        switch (u) {
        case 0: return __builtin_amdgcn_mov_dpp(ids, 0x00, 0xF, 0xF, true);
        case 1: return __builtin_amdgcn_mov_dpp(ids, 0x55, 0xF, 0xF, true);
        case 2: return __builtin_amdgcn_mov_dpp(ids, 0xAA, 0xF, 0xF, true);
        default: return __builtin_amdgcn_mov_dpp(ids, 0xFF, 0xF, 0xF, true);
        }
    }
    return __shfl(ids, first + u);
}

// Adds ntok tokens of a read to its bit planes (as add_planes), from the wave's
// registers: lane l holds packed word l from the first one on, the tokens starting
// at base po of lane 0's word and ending inside lane 63's.  Four tokens per lane
// are in flight, and a carry level runs only when some lane needs it, so the
// number of planes reached comes out uniform without a reduction.
template <int Q>
__device__ __forceinline__ int add_planes_lanes(uint32_t *planes, int npl, uint32_t word,
                                                  uint32_t po, uint32_t ntok, int lane)
{
    constexpr int VW = (1 << (2 * Q)) >> 5;
    int np = 0;
    for (uint32_t base = 0; base < ntok; base += 4 * kWave) {
        uint32_t tok[4], old[4];
        constexpr uint32_t kIdle = ~0u;   // no token, or its carry has ended
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            tok[t] = kIdle;
            old[t] = 0u;
            if (base + t * kWave < ntok) {   // uniform
                const uint32_t i = base + t * kWave + lane;
                const uint32_t pos = po + i;
                const uint32_t sh = (pos & 15u) << 1;
                const uint32_t h = __shfl(word, (int)(pos >> 4)), l = __shfl(word, (int)(pos >> 4) + 1);
                if (i < ntok)
                    tok[t] = (uint32_t)(((((uint64_t)h << 32) | l) << sh) >> (64 - 2 * Q));
            }
        }
        for (int k = 0; k < npl; ++k) {
            bool any = false;
#pragma unroll
            for (int t = 0; t < 4; ++t)
                any |= tok[t] != kIdle;
            if (!__ballot(any))
                break;
            np = max(np, k + 1);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (tok[t] != kIdle)
                    old[t] = atomicXor(&planes[k * VW + (tok[t] >> 5)], 1u << (tok[t] & 31u));
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (!((old[t] >> (tok[t] & 31u)) & 1u))
                    tok[t] = kIdle;
        }
    }
    return np;
}

// x / d, rounded down, for x < 2^52: the product with the rounded reciprocal is
// off by less than one either way.  (A 64-bit integer division would need more
// registers than the rest of the reads' setup.)
__device__ __forceinline__ uint64_t div_by(uint64_t x, uint32_t d, double inv)
{
    uint64_t q = (uint64_t)((double)x * inv);
    const int64_t r = (int64_t)(x - q * d);
    if (r < 0)
        --q;
    else if (r >= (int64_t)d)
        ++q;
    return q;
}

// Persistent kernel.  A wavefront takes tickets (runs of consecutive pairs; the
// first one by its own number, later ones from a counter, drawn while the ticket
// before is worked on) and goes through a ticket's pairs in blocks of 64 and
// steps of 64 / G x U pairs, G lanes a pair.
//
// What bounds it is the gather of bin vectors (random lines of a multi-GB index,
// or of the caches), so the loads are kept apart from everything else: a step's
// vectors are requested one step ahead, by bin id alone, whatever reads the pairs
// belong to, and the ids two blocks ahead.  The metadata of 64 reads at a time
// sits in the lanes (CSR range, length, offset, threshold), and the next read's
// packed bases are requested while the current one's candidates are counted, so
// a short candidate list costs the building of its planes and no round trips.
// A step that several reads share is counted once per read, each with its own
// planes.  Group g of a step owns U consecutive pairs, and the lane sums are
// exchanged so that lane g * G + u ends with pair g * U + u: a block's 64 counts
// leave in one coalesced store and its pass bits are one ballot (no LDS, no
// atomics; tickets start on multiples of 64 pairs, so no two waves share a
// word).
//
// Measured, against the kernel before it (one round trip after another per read,
// every tile of 1024 pairs drawn from one counter at 11.4 ns a draw): 64 reads x
// 64 pairs 10.6 us (47.5), of which the work list 1.9 (4.5), 100k reads / 2.1e7 pairs on
// a 64 MB index 436 us (521; a gather of as many vectors alone takes 372), 8.3e8
// pairs on the 2 GB index 20.0 ms (20.5; gather alone 19.9), q = 6, 2.0e8 pairs
// 16.5 ms (17.2), q = 7, 5.1e6 pairs of reads up to 2000 bases 1.40 ms (2.66).
//
// Registers: two steps of vectors and planes 0 and 1, 8 C (U + 1) of them, beside
// about 80 others; waves per SIMD as many as that leaves room for.
constexpr int batched_waves(int c, int u)
{
    return 8 * c * (u + 1) <= 48 ? 4 : 8 * c * (u + 1) <= 80 ? 3 : 2;
}

template <int Q, int G, int U>
__global__ __launch_bounds__(256, batched_waves((1 << (2 * Q)) / 128 / G, U)) void filter_batched_kernel(
    FilterArgs a)
{
    constexpr int VW = (1 << (2 * Q)) >> 5;  // 32-bit words per vector
    constexpr int CH = VW / 4;               // 16-byte slices per vector
    constexpr int C = CH / G;                // slices per lane
    constexpr int NG = kWave / G;            // candidates per load
    constexpr int SZ = NG * U;               // pairs per step
    constexpr int SPB = kWave / SZ;          // steps per block
    static_assert(C >= 1 && CH % G == 0, "lane group wider than the vector");
    static_assert(U <= G && (SPB == 1 || SPB % 2 == 0), "a step is at most one block");
    constexpr int32_t kNone = 0x7fffffff;    // threshold of a pair without a valid read

    extern __shared__ uint32_t lds[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int npl = a.npl;
    uint32_t *planes = lds + (size_t)wv * npl * VW;
    uint4 *planes4 = reinterpret_cast<uint4 *>(planes);
    const int g = lane / G, lg = lane % G;
    // lane (within a block) -> the lane of its step that holds its pair's sum
    const int src_lane = (lane % SZ) / U * G + (lane % SZ) % U;

    const uint32_t wave = uniform_u32(blockIdx.x * (blockDim.x >> 6) + wv);
    const uint32_t shard = wave % kTicketCounters;
    uint32_t ticket = wave;
    for (int i = lane; i < npl * (VW / 4); i += kWave)
        planes4[i] = make_uint4(0, 0, 0, 0);
    int np = 0;                              // planes in use (the others are zero)

    while (ticket < a.n_tickets) {
        uint32_t drawn = 0;
        if (lane == 0)
            drawn = atomicAdd(a.counters + shard * kTicketStride, 1u);
        const uint64_t t0 = ticket_start(ticket, a.n_big, a.big_pairs, a.small_pairs);
        const uint64_t room = a.n_pairs - t0;
        const uint32_t span = ticket < a.n_big ? a.big_pairs : a.small_pairs;
        const uint32_t len = room < span ? (uint32_t)room : span;   // pairs of this ticket
        const uint32_t *ids_at = a.cand_bin + t0;

        // ------------------------------------------------ bin ids and vectors
        auto load_ids = [&](uint32_t b) -> uint32_t {
            const uint32_t x = b + lane;
            return x < len ? ids_at[x] : 0u;
        };
        auto gather = [&](uint4 (&v)[U][C], uint32_t ids, int s) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t id = group_id<G, U>(ids, s * SZ + g * U, u);
                // an id out of range reads vector 0; its count is replaced below
                const uint4 *src = a.vec + (uint64_t)(id < a.n_bins ? id : 0u) * CH + lg;
#pragma unroll
                for (int c = 0; c < C; ++c)
                    v[u][c] = src[c * G];
            }
        };
        uint32_t ids_cur = load_ids(0), ids_nxt = load_ids(kWave);

        // ---------------------------------------------- the ticket's reads
        // lane l holds read r0 + l: its CSR range within the ticket, offset,
        // tokens and threshold (kNone: the read is invalid)
        uint64_t r0, m_off = 0;
        uint32_t m_beg = 0, m_end = 0, m_tok = 0;
        int32_t m_thr = kNone;
        auto load_reads = [&]() {
            const uint64_t r = r0 + lane;
            m_beg = m_end = m_tok = 0;
            m_thr = kNone;
            if (r < a.n_reads) {
                const uint64_t cb = a.cand_off[r], ce = a.cand_off[r + 1];
                const uint32_t L = a.read_len[r], e_num = a.read_e[r];
                m_off = a.read_off[r];
                const uint64_t nbases = a.nw * 16;
                m_beg = cb <= t0 ? 0u : (cb - t0 >= len ? len : (uint32_t)(cb - t0));
                m_end = ce <= t0 ? 0u : (ce - t0 >= len ? len : (uint32_t)(ce - t0));
                if (!(L > a.max_len || m_off > nbases || L > nbases - m_off)) {
                    m_tok = L >= (uint32_t)Q ? L - Q + 1 : 0u;
                    const uint64_t E = div_by((uint64_t)e_num * L + a.e_den - 1, a.e_den, a.inv_den);
                    const int64_t T = (int64_t)m_tok - (int64_t)Q * (int64_t)E;
                    m_thr = T > 0 ? (int32_t)T : 0;   // counts are never negative
                }
            }
        };
        // packed words of the read in lane j from its first one on, one a lane
        auto load_words = [&](int j) -> uint32_t {
            const uint64_t w = (((uint64_t)(uint32_t)__shfl((uint32_t)(m_off >> 32), j) << 32 |
                                 (uint32_t)__shfl((uint32_t)m_off, j)) >> 4) + lane;
            return w < a.nw ? a.rw[w] : 0u;
        };
        uint32_t first_read = a.ticket_read ? a.ticket_read[ticket] : 0u;
        uint4 v0[U][C], v1[U][C];
        gather(v0, ids_cur, 0);
        if (!a.ticket_read)
            first_read = (uint32_t)wave_read_of(a.cand_off, a.n_reads, t0, lane);
        r0 = uniform_u32(first_read);
        load_reads();

        uint32_t seg_end = 0;       // pairs [.., seg_end) belong to the current segment
        int32_t thr = kNone;        // its threshold; kNone when it has no valid read
        int j_next = 0;             // first lane not yet looked at
        int j_words = -1;           // lane whose read's words are in `words`
        uint32_t words = 0;
        uint4 p0[C], p1[C];

        // the segment that holds pair pos
        auto advance = [&](uint32_t pos) {
            thr = kNone;
            uint64_t m;
            for (;;) {
                m = j_next < kWave ? __ballot(m_end > pos) >> j_next << j_next : 0ull;
                if (m)
                    break;
                r0 += kWave;
                j_next = 0;
                j_words = -1;
                if (r0 >= a.n_reads) {   // pairs beyond the last read's range
                    if (lane == 0)
                        flag(a.status, GRIM_FLAG_CAND_OFF);
                    seg_end = len;
                    return;
                }
                load_reads();
            }
            const int j = (int)uniform_u32((uint32_t)__builtin_ctzll(m));
            const uint32_t beg = __builtin_amdgcn_readlane(m_beg, j);
            if (beg > pos) {   // a gap owned by no read: cand_off is not a CSR array
                if (lane == 0)
                    flag(a.status, GRIM_FLAG_CAND_OFF);
                seg_end = beg;
                j_next = j;
                return;
            }
            seg_end = __builtin_amdgcn_readlane(m_end, j);
            j_next = j + 1;
            thr = (int32_t)__builtin_amdgcn_readlane((uint32_t)m_thr, j);
            if (thr == kNone) {
                if (lane == 0)
                    flag(a.status, GRIM_FLAG_READ);
                return;
            }
            const uint32_t ntok = __builtin_amdgcn_readlane(m_tok, j);
            const uint32_t po = __builtin_amdgcn_readlane((uint32_t)m_off, j) & 15u;
            wave_fence();
            for (int i = lane; i < np * (VW / 4); i += kWave)
                planes4[i] = make_uint4(0, 0, 0, 0);
            wave_fence();
            if (po + ntok + Q <= 16u * kWave) {
                if (j_words != j)
                    words = load_words(j);
                np = add_planes_lanes<Q>(planes, npl, words, po, ntok, lane);
            } else {
                // longer reads in stretches that the lanes hold, the next one's
                // words ahead (q = 6, reads of 8000 bases with 1-512 candidates: 503
                // us, 650 with one token a lane at a time from memory)
                constexpr uint32_t kStretch = 12 * kWave;
                const uint64_t first = ((uint64_t)__builtin_amdgcn_readlane((uint32_t)(m_off >> 32), j)
                                            << 32 | __builtin_amdgcn_readlane((uint32_t)m_off, j)) >> 4;
                auto stretch = [&](uint32_t t) -> uint32_t {
                    const uint64_t w = first + (t >> 4) + lane;
                    return t < ntok && w < a.nw ? a.rw[w] : 0u;
                };
                uint32_t cur = stretch(0);
                np = 0;
                for (uint32_t t = 0; t < ntok; t += kStretch) {
                    const uint32_t nxt = stretch(t + kStretch);
                    np = max(np, add_planes_lanes<Q>(planes, npl, cur, po, min(ntok - t, kStretch),
                                                     lane));
                    cur = nxt;
                }
            }
            wave_fence();
            // planes 0 and 1 stay in registers for the whole segment
#pragma unroll
            for (int c = 0; c < C; ++c) {
                p0[c] = planes4[c * G + lg];
                p1[c] = npl > 1 ? planes4[VW / 4 + c * G + lg] : make_uint4(0, 0, 0, 0);
            }
            // the words of the next read of this ticket
            const uint64_t after =
                j_next < kWave && seg_end < len ? __ballot(m_end > seg_end) >> j_next << j_next : 0ull;
            if (after) {
                j_words = (int)uniform_u32((uint32_t)__builtin_ctzll(after));
                words = load_words(j_words);
            }
        };

        int32_t res;    // count of pair b + lane, -1 until one is known
        int32_t my_thr; // and its read's threshold
        // counts of step s of block b (vectors in v)
        auto count = [&](const uint4 (&v)[U][C], uint32_t b, int s) {
            uint32_t pos = b + s * SZ;
            const uint32_t pe = min(pos + SZ, len);
            while (pos < pe) {
                if (pos >= seg_end)
                    advance(pos);
                const uint32_t e = min(seg_end, pe);
                if (thr != kNone) {
                    uint32_t acc[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        uint32_t a0 = 0, a1 = 0;
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            a0 += popc_and(p0[c], v[u][c]);
                            a1 += popc_and(p1[c], v[u][c]);
                        }
                        acc[u] = a0 + (a1 << 1);
                    }
                    for (int k = 2; k < np; ++k) {
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            const uint4 pk = planes4[k * (VW / 4) + c * G + lg];
#pragma unroll
                            for (int u = 0; u < U; ++u)
                                acc[u] += popc_and(pk, v[u][c]) << k;
                        }
                    }
                    uint32_t sum = group_sums<G, U>(acc, lane);
                    if constexpr (!(SPB == 1 && U == G))
                        sum = __shfl(sum, src_lane);
                    const uint32_t x = b + lane;
                    if (x >= pos && x < e) {
                        res = (int32_t)sum;
                        my_thr = thr;
                    }
                }
                pos = e;
            }
        };
        auto finish = [&](uint32_t b) {
            const uint32_t x = b + lane;
            if (my_thr != kNone && ids_cur >= a.n_bins) {   // lanes past len hold id 0
                res = -1;
                flag(a.status, GRIM_FLAG_BIN_RANGE);
            }
            if (x < len)
                a.counts[t0 + x] = res;
            const uint64_t bits = __ballot(res >= my_thr);
            const uint32_t n_words = (min(len - b, (uint32_t)kWave) + 31) >> 5;
            if ((uint32_t)lane < n_words)
                a.pass_bits[((t0 + b) >> 5) + lane] = (uint32_t)(lane ? bits >> 32 : bits);
        };
        // one block: x0 holds its first step's vectors; leaves the next block's
        // first step in x0 (several steps a block) or x1 (one)
        auto block = [&](uint32_t b, uint4 (&x0)[U][C], uint4 (&x1)[U][C]) {
            const uint32_t ids_new = load_ids(b + 2 * kWave);
            res = -1;
            my_thr = kNone;
            if constexpr (SPB == 1) {
                if (b + kWave < len)
                    gather(x1, ids_nxt, 0);
                count(x0, b, 0);
            } else {
#pragma unroll 1
                for (int s = 0; s < SPB; s += 2) {
                    if (b + (s + 1) * SZ < len)
                        gather(x1, ids_cur, s + 1);
                    count(x0, b, s);
                    if (s + 2 < SPB) {
                        if (b + (s + 2) * SZ < len)
                            gather(x0, ids_cur, s + 2);
                    } else if (b + kWave < len) {
                        gather(x0, ids_nxt, 0);
                    }
                    count(x1, b, s + 1);
                }
            }
            finish(b);
            ids_cur = ids_nxt;
            ids_nxt = ids_new;
        };
        if constexpr (SPB == 1) {
            for (uint32_t b = 0; b < len; b += 2 * kWave) {
                block(b, v0, v1);
                if (b + kWave < len)
                    block(b + kWave, v1, v0);
            }
        } else {
            for (uint32_t b = 0; b < len; b += kWave)
                block(b, v0, v1);
        }
        ticket = uniform_u32(__shfl(drawn, 0)) * kTicketCounters + shard;
    }
}

// ------------------------------------------------------------- plain filter
// One workgroup (one wavefront) per read: build the read's planes, then walk
// its candidates NG at a time, reading every plane from LDS for every
// candidate; pass bits are set with global atomics into a pre-zeroed mask.
template <int Q>
__global__ __launch_bounds__(64) void filter_plain_kernel(FilterArgs a)
{
    constexpr int VW = (1 << (2 * Q)) >> 5;
    constexpr int CH = VW / 4;
    constexpr int G = CH < kWave ? CH : kWave;
    constexpr int C = CH / G;
    constexpr int NG = kWave / G;
    extern __shared__ uint32_t lds[];
    uint32_t *planes = lds;
    const int lane = threadIdx.x & 63;
    const int g = lane / G, lg = lane % G;
    for (uint64_t r = blockIdx.x; r < a.n_reads; r += gridDim.x) {
        const uint64_t cb = a.cand_off[r], ce = a.cand_off[r + 1];
        if (ce <= cb) {
            if (ce < cb && lane == 0)
                flag(a.status, GRIM_FLAG_CAND_OFF);
            continue;
        }
        if (ce > a.n_pairs) {
            if (lane == 0)
                flag(a.status, GRIM_FLAG_CAND_OFF);
            continue;
        }
        const uint32_t L = a.read_len[r];
        const uint64_t off = a.read_off[r];
        const uint64_t nbases = a.nw * 16;
        if (L > a.max_len || off > nbases || L > nbases - off) {
            if (lane == 0)
                flag(a.status, GRIM_FLAG_READ);
            for (uint64_t k = cb + lane; k < ce; k += kWave)
                a.counts[k] = -1;
            continue;
        }
        const uint32_t ntok = L >= (uint32_t)Q ? L - Q + 1 : 0u;
        const int np = build_planes<Q>(planes, a.npl, a.rw, a.nw, off, ntok, lane);
        const uint64_t E = ((uint64_t)a.read_e[r] * L + a.e_den - 1) / a.e_den;
        const int64_t T = (int64_t)ntok - (int64_t)Q * (int64_t)E;
        for (uint64_t c0 = cb; c0 < ce; c0 += NG) {
            const uint64_t kk = c0 + g;
            const bool ok = kk < ce;
            const uint32_t bin = ok ? a.cand_bin[kk] : 0u;
            const bool inr = ok && bin < a.n_bins;
            uint32_t acc = 0;
            if (inr) {
                const uint4 *src = a.vec + (uint64_t)bin * CH + lg;
                for (int c = 0; c < C; ++c) {
                    const uint4 v = src[c * G];
                    for (int k = 0; k < np; ++k) {
                        const uint4 pk =
                            *reinterpret_cast<const uint4 *>(planes + k * VW + (c * G + lg) * 4);
                        acc += popc_and(pk, v) << k;
                    }
                }
            }
            for (int s = G / 2; s >= 1; s >>= 1)
                acc += __shfl_xor(acc, s);
            if (lg == 0 && ok) {
                const int32_t cnt = inr ? (int32_t)acc : -1;
                a.counts[kk] = cnt;
                if (!inr)
                    flag(a.status, GRIM_FLAG_BIN_RANGE);
                else if ((int64_t)cnt >= T)
                    atomicOr(&a.pass_bits[kk >> 5], 1u << (kk & 31u));
            }
        }
        wave_fence();
    }
}

// ---------------------------------------------------------------- dispatch
// (lanes per candidate, unroll) as the tuning names them, and the kernel that
// runs them.  A wave step holds 64 / G x U pairs and cannot pass the block of 64
// whose outputs leave together, so an unroll above G runs the G-unrolled kernel
// (which keeps the next step's loads in flight anyway).
#define GRIM_V(Q, G, U)                                                                          \
    {Q, G, U, reinterpret_cast<const void *>(&filter_batched_kernel<Q, G, (U < G ? U : G)>)}
static const BatchedVariant kBatched[] = {
    GRIM_V(4, 2, 2),  GRIM_V(4, 2, 4),  GRIM_V(4, 2, 8),  GRIM_V(4, 1, 8),
    GRIM_V(5, 8, 1),  GRIM_V(5, 8, 2),  GRIM_V(5, 8, 4),  GRIM_V(5, 8, 8),
    GRIM_V(5, 4, 2),  GRIM_V(5, 4, 4),  GRIM_V(5, 4, 8),  GRIM_V(5, 2, 4),
    GRIM_V(6, 32, 1), GRIM_V(6, 32, 2), GRIM_V(6, 32, 4), GRIM_V(6, 32, 8),
    GRIM_V(6, 16, 2), GRIM_V(6, 16, 4), GRIM_V(6, 8, 1),  GRIM_V(6, 8, 2),
    GRIM_V(7, 64, 1), GRIM_V(7, 64, 2), GRIM_V(7, 64, 4), GRIM_V(7, 32, 1),
    GRIM_V(7, 32, 2),
};
#undef GRIM_V

const BatchedVariant *batched_variants(int *n)
{
    *n = (int)(sizeof(kBatched) / sizeof(kBatched[0]));
    return kBatched;
}

const void *plain_kernel(int q)
{
    switch (q) {
    case 4: return reinterpret_cast<const void *>(&filter_plain_kernel<4>);
    case 5: return reinterpret_cast<const void *>(&filter_plain_kernel<5>);
    case 6: return reinterpret_cast<const void *>(&filter_plain_kernel<6>);
    case 7: return reinterpret_cast<const void *>(&filter_plain_kernel<7>);
    default: return nullptr;
    }
}

hipError_t launch_build(int q, dim3 grid, hipStream_t s, const uint32_t *ref, uint64_t nw,
                        uint64_t G, uint64_t B, uint64_t O, uint64_t n_bins, uint32_t *out)
{
    switch (q) {
    case 4: hipLaunchKernelGGL(build_bins_kernel<4>, grid, dim3(256), 0, s, ref, nw, G, B, O, n_bins, out); break;
    case 5: hipLaunchKernelGGL(build_bins_kernel<5>, grid, dim3(256), 0, s, ref, nw, G, B, O, n_bins, out); break;
    case 6: hipLaunchKernelGGL(build_bins_kernel<6>, grid, dim3(256), 0, s, ref, nw, G, B, O, n_bins, out); break;
    case 7: hipLaunchKernelGGL(build_bins_kernel<7>, grid, dim3(256), 0, s, ref, nw, G, B, O, n_bins, out); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_worklist(hipStream_t s, const FilterArgs &a, uint32_t n_waves)
{
    const uint32_t n_table = a.ticket_read ? a.n_tickets : 0u;
    const uint32_t blocks = n_table ? (n_table + 255) / 256 : 1;
    hipLaunchKernelGGL(worklist_kernel, dim3(blocks), dim3(256), 0, s, a.cand_off, a.n_reads,
                       n_table, a.n_big, a.big_pairs, a.small_pairs, n_waves,
                       const_cast<uint32_t *>(a.ticket_read), a.status, a.counters);
    return hipGetLastError();
}

hipError_t launch_zero(hipStream_t s, uint32_t *p, uint64_t n)
{
    uint64_t blocks = (n + 255) / 256;
    if (blocks < 1)
        blocks = 1;
    if (blocks > 65536)
        blocks = 65536;
    hipLaunchKernelGGL(zero_words_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_zero2(hipStream_t s, uint32_t *p, uint64_t n, uint32_t *p2, uint64_t n2)
{
    const uint64_t blocks = std::min<uint64_t>((n + n2 + 255) / 256, 65536);
    hipLaunchKernelGGL(zero_words2_kernel, dim3((uint32_t)(blocks ? blocks : 1)), dim3(256), 0, s,
                       p, n, p2, n2);
    return hipGetLastError();
}

hipError_t launch_filter(const void *kernel, dim3 grid, dim3 block, size_t lds_bytes,
                         hipStream_t s, const FilterArgs &a)
{
    FilterArgs copy = a;
    void *args[] = {&copy};
    return hipLaunchKernel(kernel, grid, block, args, lds_bytes, s);
}

}  // namespace grim
