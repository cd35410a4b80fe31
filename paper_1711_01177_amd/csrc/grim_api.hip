// C ABI of the GRIM-Filter library: index build and storage, the batched and
// plain filter launches, status, autotuning and HIP-graph capture.  Kernels
// live in grim_kernels.hip; the serving runtime in grim_serve.cpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>
#include <tuple>
#include <vector>

#include "grim_internal.h"

using namespace grim;

namespace {

thread_local char g_hip_msg[256] = "";

int hip_fail(hipError_t e, const char *what)
{
    std::snprintf(g_hip_msg, sizeof(g_hip_msg), "%s: %s", what, hipGetErrorString(e));
    return GRIM_E_HIP;
}

#define HIP_TRY(x)                                  \
    do {                                            \
        hipError_t e_ = (x);                        \
        if (e_ != hipSuccess)                       \
            return hip_fail(e_, #x);                \
    } while (0)

int current_device(int *dev)
{
    hipError_t e = hipGetDevice(dev);
    return e == hipSuccess ? GRIM_OK : hip_fail(e, "hipGetDevice");
}

int cu_count(int dev)
{
    static std::mutex mu;
    static std::map<int, int> cache;
    std::lock_guard<std::mutex> lk(mu);
    auto it = cache.find(dev);
    if (it != cache.end())
        return it->second;
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
        n = 256;
    cache[dev] = n;
    return n;
}

uint64_t vector_words(uint32_t q) { return (1ull << (2 * q)) >> 5; }

// Multiplicity planes needed so that no token count of a read of up to max_len
// bases overflows: bit length of the largest token count.
int planes_for(uint32_t q, uint32_t max_len)
{
    uint32_t ntok = max_len >= q ? max_len - q + 1 : 1;
    int n = 0;
    while (ntok) {
        ++n;
        ntok >>= 1;
    }
    return n;
}

const BatchedVariant *find_variant(uint32_t q, uint32_t g, uint32_t u)
{
    int n = 0;
    const BatchedVariant *v = batched_variants(&n);
    for (int i = 0; i < n; ++i)
        if ((uint32_t)v[i].q == q && (uint32_t)v[i].g == g && (uint32_t)v[i].u == u)
            return &v[i];
    return nullptr;
}

std::mutex g_tune_mu;
std::map<std::tuple<int, uint32_t, uint32_t>, grim_tuning_t> g_tune_cache;

// The launch shape a call asks for.  *fixed: the caller chose its tile, else that
// is only what the workspace is checked against and the library cuts the pairs by
// their number (with grim_tune's shape too: its sample says nothing of the size of
// later batches).
int resolve_tuning(const grim_index_t *idx, uint32_t max_len, const grim_tuning_t *tune,
                   grim_tuning_t *out, bool *fixed)
{
    grim_tuning_t t;
    *fixed = tune && tune->tile_pairs;
    grim_default_tuning(idx->q, &t);
    if (!tune) {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tune_cache.find({idx->device, idx->q, max_len});
        if (it != g_tune_cache.end())
            t = it->second;
    } else {
        if (tune->lanes_per_cand)
            t.lanes_per_cand = tune->lanes_per_cand;
        if (tune->unroll)
            t.unroll = tune->unroll;
        if (tune->tile_pairs)
            t.tile_pairs = tune->tile_pairs;
        if (tune->wg_per_cu)
            t.wg_per_cu = tune->wg_per_cu;
    }
    // lanes or an unroll given alone, with a default that no kernel has beside it:
    // 2 lanes of q = 5 go with an unroll of 4, an unroll of 4 of q = 7 with 64 lanes
    if (tune && !find_variant(idx->q, t.lanes_per_cand, t.unroll)) {
        if (idx->q == 5 && !tune->unroll)
            t.unroll = 4;
        if (idx->q == 7 && !tune->lanes_per_cand)
            t.lanes_per_cand = 64;
    }
    if (t.tile_pairs < 64 || t.tile_pairs > 4096 || t.tile_pairs % 64 != 0)
        return GRIM_E_INVALID;
    if (t.wg_per_cu < 1 || t.wg_per_cu > 32)
        return GRIM_E_INVALID;
    if (!find_variant(idx->q, t.lanes_per_cand, t.unroll))
        return GRIM_E_UNSUPPORTED;
    *out = t;
    return GRIM_OK;
}

int check_batch(const grim_index_t *idx, const grim_batch_t *b)
{
    if (!idx || !b)
        return GRIM_E_INVALID;
    if (b->e_den == 0 || b->max_len == 0 || b->max_len > kMaxLen)
        return GRIM_E_INVALID;
    if (b->n_reads >= 0xffffffffull)
        return GRIM_E_INVALID;
    if (b->n_reads == 0 && b->n_pairs != 0)
        return GRIM_E_INVALID;
    if (b->n_reads && (!b->read_off || !b->read_len || !b->read_e || !b->cand_off))
        return GRIM_E_INVALID;
    if (b->n_reads && (!b->reads_2bit || b->n_read_words == 0))
        return GRIM_E_INVALID;
    if (b->n_pairs && !b->cand_bin)
        return GRIM_E_INVALID;
    if (b->n_pairs > (0xffffffffull - 1) * 4096ull)
        return GRIM_E_INVALID;
    int dev = -1;
    int rc = current_device(&dev);
    if (rc)
        return rc;
    if (dev != idx->device)
        return GRIM_E_INVALID;
    return GRIM_OK;
}

FilterArgs make_args(const grim_index_t *idx, const grim_batch_t *b, int32_t *counts,
                     uint32_t *pass_bits, void *ws)
{
    FilterArgs a;
    std::memset(&a, 0, sizeof(a));
    a.vec = reinterpret_cast<const uint4 *>(idx->d_vec);
    a.n_bins = idx->n_bins;
    a.rw = b->reads_2bit;
    a.nw = b->n_read_words;
    a.read_off = b->read_off;
    a.read_len = b->read_len;
    a.read_e = b->read_e;
    a.e_den = b->e_den;
    a.inv_den = 1.0 / b->e_den;
    a.max_len = b->max_len;
    a.cand_off = b->cand_off;
    a.cand_bin = b->cand_bin;
    a.n_reads = b->n_reads;
    a.n_pairs = b->n_pairs;
    a.counts = counts;
    a.pass_bits = pass_bits;
    a.status = reinterpret_cast<uint32_t *>(ws);
    a.counters = reinterpret_cast<uint32_t *>(ws) + 1;
    a.npl = planes_for(idx->q, b->max_len);
    return a;
}

uint64_t ws_bytes_for(uint64_t n_pairs, uint32_t tile_pairs)
{
    const uint64_t n_tiles = (n_pairs + tile_pairs - 1) / tile_pairs;
    return (kWsHeader + 4 * n_tiles + 255) & ~255ull;
}

// Workgroups of a batched launch that one CU holds at once.  The kernel's waves
// stay until the tickets are gone and start on tickets of their own, so a grid
// beyond what is resident leaves work to waves that start last (q = 4, 6.3e6
// pairs: 298 us at 8 workgroups per CU, 133 us at the 4 that fit).
hipError_t batched_resident(const BatchedVariant *v, int threads, size_t lds, int *out)
{
    static std::mutex mu;
    static std::map<std::tuple<const void *, int, size_t>, int> cache;
    std::lock_guard<std::mutex> lk(mu);
    const auto key = std::make_tuple(v->kernel, threads, lds);
    auto it = cache.find(key);
    if (it == cache.end()) {
        int n = 0;
        const hipError_t e =
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, v->kernel, threads, lds);
        if (e != hipSuccess)
            return e;
        it = cache.emplace(key, std::max(1, n)).first;
    }
    *out = it->second;
    return hipSuccess;
}

// Wavefronts and LDS of a workgroup of a batched launch, and its workgroups that
// one CU holds at once.
struct BatchedShape {
    int waves, resident;
    size_t lds;
};

int batched_shape(const grim_index_t *idx, int npl, const BatchedVariant *v, BatchedShape *out)
{
    const size_t per_wave = (size_t)npl * vector_words(idx->q) * 4;
    if (per_wave > 65536)
        return GRIM_E_UNSUPPORTED;
    int waves = 4;
    while (waves > 1 && per_wave * waves > 65536)
        --waves;
    out->waves = waves;
    out->lds = per_wave * waves;
    HIP_TRY(batched_resident(v, 64 * waves, out->lds, &out->resident));
    return GRIM_OK;
}

// How the pairs of a launch are cut into tickets (FilterArgs).
struct Tickets {
    uint32_t big_pairs, small_pairs, n_big, n_tickets;
};

uint64_t div_up(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

// Fewest pairs of a ticket with wide vectors, 64 to 512: those whose vectors cost four
// times the planes of a read of max_len bases (which take as long as max_len / 48
// vectors of 512 bytes), but no more than a read or a wave has.  q = 6, 5000 reads
// of 8000 bases, 1-512 candidates each: 432 us, 503 with 64-pair tickets at the end
// (one tile of 1024 pairs after another, planes from one token a lane at a time: 464);
// 2000 bases 169, 173 (196).  Reads of up to 1500 bases, 6000 with q = 7, keep 64.
uint32_t build_pairs(const grim_batch_t *b, uint64_t n_waves, uint64_t vector_bytes)
{
    const uint64_t want = std::min({(uint64_t)b->max_len * 512 / vector_bytes / 12,
                                    b->n_pairs / std::max<uint64_t>(1, b->n_reads),
                                    b->n_pairs / n_waves});
    uint32_t p = 64;
    while (p < 512 && 2 * p <= want)
        p *= 2;
    return p;
}

// Tickets of a launch that leaves the cut to the library, n_waves waves and
// room for a table of `room` first reads.  A ticket costs its wave a first round
// trip (reads, ids, vectors), the planes of one more read and a draw from a
// counter (2.1e8 a second for the whole GPU), so it holds 512 pairs where each
// wave gets one of those, and fewer, down to the 64 whose pass bits one wave
// stores, where waves would idle (q = 5, 4.2e5 pairs: 256 pairs a ticket 48 us,
// 128 52 us, 64 57 us; 1.1e5 pairs: 64 29 us, 256 35 us, 1024 63 us; q = 4,
// 6.3e6 pairs: 512 135 us, 256 169 us, bound by the draws).  Vectors of 512
// bytes and more pay for smaller ones: four tickets a wave at any size, and a
// tail of 64-pair tickets (one large one's pairs per wave) so that the waves end
// together.  Where a read's candidates are cut that finely its planes are built
// once more for every ticket, which for long reads takes as long as the vectors of
// many pairs: `floor` pairs are the fewest then (build_pairs).  512-pair
// tickets are also what the workspace's table is sized for; with the tail it holds
// 1024-pair ones, and finer cuts than that search.
Tickets auto_tickets(uint64_t n_pairs, uint64_t n_waves, uint64_t vector_bytes, uint32_t floor,
                     uint64_t room)
{
    const bool wide = vector_bytes >= 512;
    auto cut = [&](uint32_t big) {
        Tickets t = {big, wide ? floor : big, 0, 0};
        const uint64_t tail = n_waves * big;
        t.n_big = (uint32_t)(n_pairs > tail ? (n_pairs - tail) / big : 0);
        t.n_tickets = t.n_big + (uint32_t)div_up(n_pairs - (uint64_t)t.n_big * big, t.small_pairs);
        return t;
    };
    uint32_t big = 512;
    while (big > (wide ? floor : 64u) && n_pairs * 2 < n_waves * big * (wide ? 8 : 1))
        big /= 2;
    const Tickets t = cut(big);
    if (t.n_tickets <= room || !wide || big < 512)
        return t;
    const Tickets t2 = cut(1024);
    return t2.n_tickets <= room ? t2 : t;
}

// Queue the work-list and batched filter kernels on `s`.  fixed: the caller
// chose the tile (every ticket has t.tile_pairs pairs).  status (may be null)
// replaces the workspace's status word as the word the kernels reset and flag.
int enqueue_batched(const grim_index_t *idx, const grim_batch_t *b, int32_t *counts,
                    uint32_t *pass_bits, void *ws, uint64_t ws_bytes, const grim_tuning_t &t,
                    bool fixed, hipStream_t s, uint32_t *status = nullptr)
{
    const uint64_t need = ws_bytes_for(b->n_pairs, t.tile_pairs);
    if (!ws || ws_bytes < need || (reinterpret_cast<uintptr_t>(ws) & 255))
        return GRIM_E_INVALID;
    if (b->n_pairs && (!counts || !pass_bits))
        return GRIM_E_INVALID;
    FilterArgs a = make_args(idx, b, counts, pass_bits, ws);
    if (status)
        a.status = status;
    const uint64_t n_tiles = div_up(b->n_pairs, t.tile_pairs);
    if (n_tiles >= (1ull << 32) - (1ull << 24))  // the 32-bit ticket counters must not wrap
        return GRIM_E_UNSUPPORTED;
    const BatchedVariant *v = find_variant(idx->q, t.lanes_per_cand, t.unroll);
    BatchedShape shape;
    const int rc = batched_shape(idx, a.npl, v, &shape);
    if (rc)
        return rc;
    const int waves = shape.waves;
    uint64_t grid = (uint64_t)cu_count(idx->device) * std::min<uint32_t>(t.wg_per_cu, shape.resident);
    const uint64_t room = (ws_bytes - kWsHeader) / 4;
    Tickets k = {t.tile_pairs, t.tile_pairs, (uint32_t)n_tiles, (uint32_t)n_tiles};
    if (!fixed)
        k = auto_tickets(b->n_pairs, grid * waves, idx->vector_bytes,
                         build_pairs(b, grid * waves, idx->vector_bytes), room);
    a.big_pairs = k.big_pairs;
    a.small_pairs = k.small_pairs;
    a.n_big = k.n_big;
    a.n_tickets = k.n_tickets;
    // the table of first reads where the workspace holds one; batches cut finer
    // than it is sized for look the read up themselves
    a.ticket_read = nullptr;
    if (k.n_tickets <= room)
        a.ticket_read = reinterpret_cast<const uint32_t *>(static_cast<char *>(ws) + kWsHeader);
    const uint64_t useful = div_up(k.n_tickets, waves);
    if (grid > useful)
        grid = useful;
    HIP_TRY(launch_worklist(s, a, (uint32_t)(grid * waves)));
    if (k.n_tickets == 0)
        return GRIM_OK;
    HIP_TRY(launch_filter(v->kernel, dim3((uint32_t)grid), dim3(64 * waves), shape.lds, s, a));
    return GRIM_OK;
}

}  // namespace

// --------------------------------------------------------------- basics
extern "C" const char *grim_strerror(int code)
{
    switch (code) {
    case GRIM_OK: return "ok";
    case GRIM_PENDING: return "pending";
    case GRIM_E_INVALID: return "invalid argument";
    case GRIM_E_BASE: return "base outside A/C/G/T";
    case GRIM_E_BIN_RANGE: return "candidate bin id out of range";
    case GRIM_E_NOMEM: return "out of memory";
    case GRIM_E_BUDGET: return "request exceeds the device memory budget";
    case GRIM_E_HIP: return g_hip_msg[0] ? g_hip_msg : "HIP runtime error";
    case GRIM_E_CANCELLED: return "cancelled";
    case GRIM_E_UNSUPPORTED: return "unsupported parameters";
    case GRIM_E_IO: return "index file error";
    case GRIM_E_TIMEOUT: return "timed out";
    case GRIM_E_READ: return "invalid read or candidate offsets";
    case GRIM_E_SCRATCH:
        return "batch needs more than the static scratch holds (use grim_filter_batch with a "
               "workspace)";
    default: return "unknown error";
    }
}

extern "C" int grim_version(void) { return 10000; }

// ---------------------------------------------------------------- index
extern "C" int grim_build_bins(const uint32_t *ref_2bit, uint64_t ref_len, const grim_params_t *p,
                               grim_index_t **out, void *stream)
{
    if (!ref_2bit || !p || !out || ref_len == 0 || p->bin_stride == 0 || p->build > GRIM_BUILD_BLOCKS)
        return GRIM_E_INVALID;
    if (p->q < 4 || p->q > 7)
        return GRIM_E_UNSUPPORTED;
    const uint64_t n_bins = (ref_len + p->bin_stride - 1) / p->bin_stride;
    if (n_bins > 0xffffffffull)
        return GRIM_E_INVALID;
    int dev = 0;
    int rc = current_device(&dev);
    if (rc)
        return rc;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const uint64_t vb = vector_words(p->q) * 4;
    const uint64_t nw = grim_packed_words(ref_len);
    grim_index *idx = new (std::nothrow) grim_index();
    if (!idx)
        return GRIM_E_NOMEM;
    idx->d_ref = nullptr;
    idx->d_planes = nullptr;
    idx->ref_words = 0;
    idx->d_rows = nullptr;
    idx->row_words = 0;
    idx->q = p->q;
    idx->device = dev;
    idx->B = p->bin_stride;
    idx->O = p->overlap;
    idx->G = ref_len;
    idx->n_bins = n_bins;
    idx->vector_bytes = vb;
    idx->bytes = n_bins * vb;
    if (hipMalloc(&idx->d_vec, idx->bytes) != hipSuccess) {
        delete idx;
        return GRIM_E_NOMEM;
    }
    uint32_t *d_ref = nullptr;
    if (hipMalloc(&d_ref, nw * 4) != hipSuccess) {
        (void)hipFree(idx->d_vec);
        delete idx;
        return GRIM_E_NOMEM;
    }
    hipError_t e = hipMemcpyAsync(d_ref, ref_2bit, nw * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) {
        // the first kernel that fits the geometry, or the one asked for
        uint32_t *vec = reinterpret_cast<uint32_t *>(idx->d_vec);
        const uint32_t cus = (uint32_t)cu_count(dev);
        const uint32_t want = p->build;
        e = hipErrorNotSupported;
        if (want == GRIM_BUILD_AUTO || want == GRIM_BUILD_BLOCKS)
            e = launch_build_chunked(p->q, cus, s, d_ref, nw, ref_len, p->bin_stride, p->overlap,
                                     n_bins, vec);
        if (e == hipErrorNotSupported && (want == GRIM_BUILD_AUTO || want == GRIM_BUILD_PER_BIN)) {
            uint64_t grid = (n_bins + 3) / 4;
            const uint64_t cap = (uint64_t)cus * 32;
            if (grid > cap)
                grid = cap;
            e = launch_build(p->q, dim3((uint32_t)grid), s, d_ref, nw, ref_len, p->bin_stride,
                             p->overlap, n_bins, vec);
        }
        if (e == hipErrorNotSupported) {  // only a forced kernel gets here
            (void)hipFree(d_ref);
            (void)hipFree(idx->d_vec);
            delete idx;
            return GRIM_E_UNSUPPORTED;
        }
    }
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    (void)hipFree(d_ref);
    if (e != hipSuccess) {
        (void)hipFree(idx->d_vec);
        delete idx;
        return hip_fail(e, "grim_build_bins");
    }
    *out = idx;
    return GRIM_OK;
}

extern "C" int grim_index_info(const grim_index_t *idx, grim_index_info_t *out)
{
    if (!idx || !out)
        return GRIM_E_INVALID;
    out->q = idx->q;
    out->device = idx->device;
    out->bin_stride = idx->B;
    out->overlap = idx->O;
    out->genome_len = idx->G;
    out->n_bins = idx->n_bins;
    out->vector_bytes = idx->vector_bytes;
    out->bytes = idx->bytes;
    out->vectors = idx->d_vec;
    return GRIM_OK;
}

extern "C" int grim_index_copy_to_host(const grim_index_t *idx, void *host, uint64_t bytes)
{
    if (!idx || !host || bytes < idx->bytes)
        return GRIM_E_INVALID;
    HIP_TRY(hipMemcpy(host, idx->d_vec, idx->bytes, hipMemcpyDeviceToHost));
    return GRIM_OK;
}

namespace {
struct IndexFileHeader {
    char magic[8];
    uint32_t version, q;
    uint64_t B, O, G, n_bins, checksum;
    uint64_t reserved;
};
static_assert(sizeof(IndexFileHeader) == 64, "header must be 64 bytes");

uint64_t fnv1a(const uint8_t *p, uint64_t n, uint64_t h = 1469598103934665603ull)
{
    for (uint64_t i = 0; i < n; ++i) {
        h ^= p[i];
        h *= 1099511628211ull;
    }
    return h;
}
}  // namespace

extern "C" int grim_index_save(const grim_index_t *idx, const char *path)
{
    if (!idx || !path)
        return GRIM_E_INVALID;
    std::vector<uint8_t> host;
    try {
        host.resize(idx->bytes);
    } catch (...) {
        return GRIM_E_NOMEM;
    }
    int rc = grim_index_copy_to_host(idx, host.data(), host.size());
    if (rc)
        return rc;
    IndexFileHeader h;
    std::memset(&h, 0, sizeof(h));
    std::memcpy(h.magic, "GRIMIDX1", 8);
    h.version = 1;
    h.q = idx->q;
    h.B = idx->B;
    h.O = idx->O;
    h.G = idx->G;
    h.n_bins = idx->n_bins;
    h.checksum = fnv1a(host.data(), host.size());
    FILE *f = std::fopen(path, "wb");
    if (!f)
        return GRIM_E_IO;
    bool ok = std::fwrite(&h, sizeof(h), 1, f) == 1 &&
              std::fwrite(host.data(), 1, host.size(), f) == host.size();
    ok = (std::fclose(f) == 0) && ok;
    return ok ? GRIM_OK : GRIM_E_IO;
}

extern "C" int grim_index_load(const char *path, grim_index_t **out, void *stream)
{
    if (!path || !out)
        return GRIM_E_INVALID;
    FILE *f = std::fopen(path, "rb");
    if (!f)
        return GRIM_E_IO;
    IndexFileHeader h;
    if (std::fread(&h, sizeof(h), 1, f) != 1 || std::memcmp(h.magic, "GRIMIDX1", 8) != 0 ||
        h.version != 1 || h.q < 4 || h.q > 7 || h.B == 0 ||
        h.n_bins != (h.G + h.B - 1) / h.B) {
        std::fclose(f);
        return GRIM_E_IO;
    }
    const uint64_t vb = vector_words(h.q) * 4;
    std::vector<uint8_t> host;
    try {
        host.resize(h.n_bins * vb);
    } catch (...) {
        std::fclose(f);
        return GRIM_E_NOMEM;
    }
    const bool ok = std::fread(host.data(), 1, host.size(), f) == host.size();
    std::fclose(f);
    if (!ok || fnv1a(host.data(), host.size()) != h.checksum)
        return GRIM_E_IO;
    int dev = 0;
    int rc = current_device(&dev);
    if (rc)
        return rc;
    grim_index *idx = new (std::nothrow) grim_index();
    if (!idx)
        return GRIM_E_NOMEM;
    idx->d_ref = nullptr;
    idx->d_planes = nullptr;
    idx->ref_words = 0;
    idx->d_rows = nullptr;
    idx->row_words = 0;
    idx->q = h.q;
    idx->device = dev;
    idx->B = h.B;
    idx->O = h.O;
    idx->G = h.G;
    idx->n_bins = h.n_bins;
    idx->vector_bytes = vb;
    idx->bytes = host.size();
    if (hipMalloc(&idx->d_vec, idx->bytes) != hipSuccess) {
        delete idx;
        return GRIM_E_NOMEM;
    }
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipError_t e = hipMemcpyAsync(idx->d_vec, host.data(), idx->bytes, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        (void)hipFree(idx->d_vec);
        delete idx;
        return hip_fail(e, "grim_index_load");
    }
    *out = idx;
    return GRIM_OK;
}

extern "C" void grim_index_free(grim_index_t *idx)
{
    if (!idx)
        return;
    if (idx->d_ref)
        (void)hipFree(idx->d_ref);
    if (idx->d_planes)
        (void)hipFree(idx->d_planes);
    if (idx->d_rows)
        (void)hipFree(idx->d_rows);
    (void)hipFree(idx->d_vec);
    delete idx;
}

// ------------------------------------------------------------ filtering
extern "C" int grim_default_tuning(uint32_t q, grim_tuning_t *out)
{
    if (!out)
        return GRIM_E_INVALID;
    // the shapes the autotuner picks on the 3.1 Gbp workloads (q = 5: 8.3e8
    // pairs, q = 6: 2.0e9 pairs); q = 4 and 7 from the parity sweeps
    grim_tuning_t t = {0, 0, 1024, 8};
    switch (q) {
    case 4: t = {2, 8, 1024, 8}; break;
    case 5: t = {4, 2, 1024, 4}; break;
    case 6: t = {8, 2, 512, 4}; break;
    case 7: t = {32, 2, 1024, 4}; break;
    default: return GRIM_E_UNSUPPORTED;
    }
    *out = t;
    return GRIM_OK;
}

extern "C" int grim_tuning_candidates(uint32_t q, grim_tuning_t *out, uint32_t cap, uint32_t *n)
{
    if (!n || (cap && !out))
        return GRIM_E_INVALID;
    grim_tuning_t d;
    if (grim_default_tuning(q, &d))
        return GRIM_E_UNSUPPORTED;
    int nv = 0;
    const BatchedVariant *v = batched_variants(&nv);
    uint32_t k = 0;
    for (int i = 0; i < nv; ++i) {
        if ((uint32_t)v[i].q != q)
            continue;
        if (k < cap)
            out[k] = grim_tuning_t{(uint32_t)v[i].g, (uint32_t)v[i].u, d.tile_pairs, d.wg_per_cu};
        ++k;
    }
    *n = k;
    return GRIM_OK;
}

extern "C" int grim_workspace_size(const grim_index_t *idx, uint64_t n_pairs,
                                   const grim_tuning_t *tune, uint64_t *bytes)
{
    if (!idx || !bytes)
        return GRIM_E_INVALID;
    grim_tuning_t t;
    bool fixed = false;
    int rc = resolve_tuning(idx, kMaxLen, tune, &t, &fixed);
    if (rc)
        return rc;
    // the cached tuning may use a smaller tile: size for the smallest tile
    *bytes = ws_bytes_for(n_pairs, std::min<uint32_t>(t.tile_pairs, 512));
    return GRIM_OK;
}

extern "C" int grim_filter_batch(const grim_index_t *idx, const grim_batch_t *b, int32_t *counts,
                                 uint32_t *pass_bits, void *workspace, uint64_t workspace_bytes,
                                 const grim_tuning_t *tune, void *stream)
{
    int rc = check_batch(idx, b);
    if (rc)
        return rc;
    grim_tuning_t t;
    bool fixed = false;
    rc = resolve_tuning(idx, b->max_len, tune, &t, &fixed);
    if (rc)
        return rc;
    return enqueue_batched(idx, b, counts, pass_bits, workspace, workspace_bytes, t, fixed,
                           reinterpret_cast<hipStream_t>(stream));
}

// ------------------------------------------------- filter without allocation
// The scratch of grim_filter_batch_noalloc: one file-scope device array per GPU
// (tile counter, padded header, first read of each tile).  Host code never uses
// the array's name as an address: the device address comes from
// hipGetSymbolAddress, once per device, and is kept in g_scratch_ptr.
static __device__ __align__(256) uint8_t scratch[GRIM_NOALLOC_SCRATCH_BYTES];

namespace {
std::mutex g_scratch_mu;
std::map<int, void *> g_scratch_ptr;

int scratch_address(int dev, void **out)
{
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    auto it = g_scratch_ptr.find(dev);
    if (it != g_scratch_ptr.end()) {
        *out = it->second;
        return GRIM_OK;
    }
    void *p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p || (reinterpret_cast<uintptr_t>(p) & 255))
        return hip_fail(hipErrorInvalidSymbol, "hipGetSymbolAddress(scratch)");
    g_scratch_ptr[dev] = p;
    *out = p;
    return GRIM_OK;
}
}  // namespace

extern "C" int grim_filter_batch_noalloc(const grim_index_t *idx, const grim_batch_t *b,
                                         int32_t *counts, uint32_t *pass_bits, uint32_t *status,
                                         const grim_tuning_t *tune, void *stream)
{
    int rc = check_batch(idx, b);
    if (rc)
        return rc;
    if (!status)
        return GRIM_E_INVALID;
    grim_tuning_t t;
    bool fixed = false;
    rc = resolve_tuning(idx, b->max_len, tune, &t, &fixed);
    if (rc)
        return rc;
    if (ws_bytes_for(b->n_pairs, t.tile_pairs) > GRIM_NOALLOC_SCRATCH_BYTES)
        return GRIM_E_SCRATCH;
    void *ws = nullptr;
    rc = scratch_address(idx->device, &ws);  // check_batch made idx->device current
    if (rc)
        return rc;
    return enqueue_batched(idx, b, counts, pass_bits, ws, GRIM_NOALLOC_SCRATCH_BYTES, t,
                           fixed, reinterpret_cast<hipStream_t>(stream), status);
}

extern "C" int grim_filter_plain(const grim_index_t *idx, const grim_batch_t *b, int32_t *counts,
                                 uint32_t *pass_bits, void *workspace, uint64_t workspace_bytes,
                                 void *stream)
{
    int rc = check_batch(idx, b);
    if (rc)
        return rc;
    if (!workspace || workspace_bytes < kWsHeader || (reinterpret_cast<uintptr_t>(workspace) & 255))
        return GRIM_E_INVALID;
    if (b->n_pairs && (!counts || !pass_bits))
        return GRIM_E_INVALID;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    FilterArgs a = make_args(idx, b, counts, pass_bits, workspace);
    HIP_TRY(launch_zero(s, a.status, 2));
    const uint64_t n_words = (b->n_pairs + 31) / 32;
    if (n_words)
        HIP_TRY(launch_zero(s, pass_bits, n_words));
    if (b->n_reads == 0)
        return GRIM_OK;
    const size_t lds = (size_t)a.npl * vector_words(idx->q) * 4;
    if (lds > 65536)
        return GRIM_E_UNSUPPORTED;
    const uint64_t grid = std::min<uint64_t>(b->n_reads, 1u << 22);
    HIP_TRY(launch_filter(plain_kernel(idx->q), dim3((uint32_t)grid), dim3(64), lds, s, a));
    return GRIM_OK;
}

extern "C" int grim_filter_status(const void *workspace, void *stream, uint32_t *flags)
{
    if (!workspace)
        return GRIM_E_INVALID;
    HIP_TRY(hipStreamSynchronize(reinterpret_cast<hipStream_t>(stream)));
    uint32_t f = 0;
    HIP_TRY(hipMemcpy(&f, workspace, 4, hipMemcpyDeviceToHost));
    if (flags)
        *flags = f;
    if (f & GRIM_FLAG_BIN_RANGE)
        return GRIM_E_BIN_RANGE;
    if (f & (GRIM_FLAG_READ | GRIM_FLAG_CAND_OFF))
        return GRIM_E_READ;
    return GRIM_OK;
}

extern "C" int grim_tune(const grim_index_t *idx, const grim_batch_t *sample, int32_t *counts,
                         uint32_t *pass_bits, void *workspace, uint64_t workspace_bytes,
                         void *stream, grim_tuning_t *out)
{
    int rc = check_batch(idx, sample);
    if (rc)
        return rc;
    if (!out)
        return GRIM_E_INVALID;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    // time on a prefix of the pair space (the kernel handles any prefix of a
    // valid CSR batch): keeps a sweep over every shape to a few seconds
    grim_batch_t sub = *sample;
    if (sub.n_pairs > (1ull << 26))
        sub.n_pairs = 1ull << 26;
    sample = &sub;
    int nv = 0;
    const BatchedVariant *vars = batched_variants(&nv);
    // tile 0: the library's own cut of the pairs.  The others are for callers that
    // pass the result on with batches like the sample; calls with tune = NULL
    // take the best shape with the library's cut, whatever their size.
    const uint32_t tiles[] = {0, 512, 1024, 2048};
    const uint32_t occ[] = {4, 8};
    hipEvent_t e0, e1;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    float best = 1e30f, best_own = 1e30f;
    grim_tuning_t best_t, own_t;
    grim_default_tuning(idx->q, &best_t);
    own_t = best_t;
    const uint32_t default_tile = best_t.tile_pairs;
    for (int i = 0; i < nv; ++i) {
        if ((uint32_t)vars[i].q != idx->q)
            continue;
        // an unroll above the lanes runs another name's kernel
        if (std::any_of(vars, vars + i, [&](const BatchedVariant &v) {
                return v.kernel == vars[i].kernel;
            }))
            continue;
        BatchedShape shape;
        if (batched_shape(idx, planes_for(idx->q, sample->max_len), &vars[i], &shape))
            continue;
        for (uint32_t wg : occ) {
            if (wg > occ[0] && shape.resident <= (int)occ[0])   // the same grid again
                continue;
            for (uint32_t tp : tiles) {
                grim_tuning_t t = {(uint32_t)vars[i].g, (uint32_t)vars[i].u, tp ? tp : default_tile,
                                   wg};
                if (workspace_bytes < ws_bytes_for(sample->n_pairs, t.tile_pairs))
                    continue;
                if (enqueue_batched(idx, sample, counts, pass_bits, workspace, workspace_bytes, t,
                                    tp != 0, s))
                    continue;
                float ms[3];
                bool fine = true;
                for (int rep = 0; rep < 3 && fine; ++rep) {
                    fine = hipEventRecord(e0, s) == hipSuccess &&
                           enqueue_batched(idx, sample, counts, pass_bits, workspace,
                                           workspace_bytes, t, tp != 0, s) == GRIM_OK &&
                           hipEventRecord(e1, s) == hipSuccess &&
                           hipEventSynchronize(e1) == hipSuccess &&
                           hipEventElapsedTime(&ms[rep], e0, e1) == hipSuccess;
                }
                if (!fine)
                    continue;
                std::sort(ms, ms + 3);
                if (ms[1] < best) {
                    best = ms[1];
                    best_t = t;
                    best_t.tile_pairs = tp;
                }
                if (!tp && ms[1] < best_own) {
                    best_own = ms[1];
                    own_t = t;
                }
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    HIP_TRY(hipStreamSynchronize(s));
    // a workspace sized for the result is large enough with tune = NULL as well
    if (best_t.tile_pairs)
        own_t.tile_pairs = best_t.tile_pairs;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_tune_cache[{idx->device, idx->q, sample->max_len}] = own_t;
    }
    *out = best_t;
    return GRIM_OK;
}

// ------------------------------------------------- seed location checker
extern "C" int grim_survivors_workspace_size(uint64_t n_pairs, uint64_t *bytes)
{
    if (!bytes)
        return GRIM_E_INVALID;
    *bytes = (8 * std::max<uint64_t>(1, compact_blocks(n_pairs)) + 255) & ~255ull;
    return GRIM_OK;
}

extern "C" int grim_compact_survivors(const grim_batch_t *b, const uint32_t *pass_bits,
                                      uint64_t capacity, uint64_t *surv_pair, uint32_t *surv_read,
                                      uint32_t *surv_bin, uint64_t *n_survivors, void *workspace,
                                      uint64_t workspace_bytes, void *stream)
{
    if (!b || !n_survivors || !workspace)
        return GRIM_E_INVALID;
    if (b->n_reads == 0 && b->n_pairs != 0)
        return GRIM_E_INVALID;
    if (b->n_pairs && (!pass_bits || !b->cand_off || !b->cand_bin))
        return GRIM_E_INVALID;
    if (capacity && (!surv_pair || !surv_read || !surv_bin))
        return GRIM_E_INVALID;
    uint64_t need = 0;
    grim_survivors_workspace_size(b->n_pairs, &need);
    if (workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 7))
        return GRIM_E_INVALID;
    HIP_TRY(launch_compact(reinterpret_cast<hipStream_t>(stream), pass_bits, b->n_pairs,
                           b->cand_off, b->n_reads, b->cand_bin, capacity, surv_pair, surv_read,
                           surv_bin, n_survivors, reinterpret_cast<uint64_t *>(workspace)));
    return GRIM_OK;
}

extern "C" int grim_index_attach_reference(grim_index_t *idx, const uint32_t *ref_2bit,
                                           uint64_t ref_len, void *stream)
{
    if (!idx || !ref_2bit || ref_len != idx->G)
        return GRIM_E_INVALID;
    const uint64_t nw = grim_packed_words(ref_len);
    const uint64_t n_planes = (nw + 1) / 2 + 2 * kPlanePad;
    uint32_t *d = nullptr;
    uint2 *planes = nullptr;
    if (hipMalloc(&d, (nw + kRefPadWords) * 4) != hipSuccess)
        return GRIM_E_NOMEM;
    if (hipMalloc(&planes, n_planes * 8) != hipSuccess) {
        planes = nullptr;   // the scan of all columns does without
        (void)hipGetLastError();
    }
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipError_t e = hipMemcpyAsync(d, ref_2bit, nw * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = launch_zero(s, d + nw, kRefPadWords);
    if (e == hipSuccess && planes)
        e = launch_zero(s, reinterpret_cast<uint32_t *>(planes), 2 * kPlanePad);
    if (e == hipSuccess && planes)
        e = launch_zero(s, reinterpret_cast<uint32_t *>(planes + n_planes - kPlanePad),
                        2 * kPlanePad);
    if (e == hipSuccess && planes)
        e = launch_planes(s, d, nw, planes + kPlanePad);
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        (void)hipFree(d);
        (void)hipFree(planes);
        return hip_fail(e, "grim_index_attach_reference");
    }
    if (idx->d_ref)
        (void)hipFree(idx->d_ref);
    if (idx->d_planes)
        (void)hipFree(idx->d_planes);
    idx->d_ref = d;
    idx->d_planes = planes;
    idx->ref_words = nw;
    return GRIM_OK;
}

extern "C" int grim_verify_survivors(const grim_index_t *idx, const grim_batch_t *b,
                                     const uint32_t *surv_read, const uint32_t *surv_bin,
                                     uint64_t n_survivors, int32_t *dist, uint32_t *ok_bits,
                                     void *stream)
{
    int rc = check_batch(idx, b);
    if (rc)
        return rc;
    if (!idx->d_ref)
        return GRIM_E_INVALID;
    if (n_survivors && (!surv_read || !surv_bin || !dist || !ok_bits))
        return GRIM_E_INVALID;
    const int W = b->max_len <= 64 ? 1 : b->max_len <= 128 ? 2 : b->max_len <= 256 ? 4
                : b->max_len <= 512 ? 8 : 0;
    if (!W)
        return GRIM_E_UNSUPPORTED;
    if (n_survivors == 0)
        return GRIM_OK;
    VerifyArgs a;
    std::memset(&a, 0, sizeof(a));
    a.ref = idx->d_ref;
    a.ref_words = idx->ref_words;
    a.planes = idx->d_planes ? idx->d_planes + kPlanePad : nullptr;
    a.G = idx->G;
    a.B = idx->B;
    a.O = idx->O;
    a.n_bins = idx->n_bins;
    a.rw = b->reads_2bit;
    a.nw = b->n_read_words;
    a.read_off = b->read_off;
    a.read_len = b->read_len;
    a.read_e = b->read_e;
    a.e_den = b->e_den;
    a.n_reads = b->n_reads;
    a.surv_read = surv_read;
    a.surv_bin = surv_bin;
    a.n_surv = n_survivors;
    a.dist = dist;
    a.ok_bits = ok_bits;
    HIP_TRY(launch_verify(reinterpret_cast<hipStream_t>(stream), W, cu_count(idx->device), a));
    return GRIM_OK;
}

// ---------------------------------------------------------------- bin windows
extern "C" int grim_index_transpose(grim_index_t *idx, void *stream)
{
    if (!idx)
        return GRIM_E_INVALID;
    // one 32-word (1024-bin) segment of every row per transpose tile
    const uint64_t row_words = ((idx->n_bins + 1023) / 1024) * 32;
    const uint64_t n_rows = 1ull << (2 * idx->q);
    uint32_t *rows = nullptr;
    // one pad word past the last row: the window kernel reads two adjacent
    // words of a row with one load
    if (hipMalloc(&rows, n_rows * row_words * 4 + 256) != hipSuccess)
        return GRIM_E_NOMEM;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    uint64_t grid = row_words / 32;
    const uint64_t cap = (uint64_t)cu_count(idx->device) * 2;
    if (grid > cap)
        grid = cap;
    hipError_t e = launch_transpose(s, idx->q, reinterpret_cast<const uint32_t *>(idx->d_vec),
                                    idx->n_bins, row_words, rows, (uint32_t)grid);
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        (void)hipFree(rows);
        return hip_fail(e, "grim_index_transpose");
    }
    if (idx->d_rows)
        (void)hipFree(idx->d_rows);
    idx->d_rows = rows;
    idx->row_words = row_words;
    return GRIM_OK;
}

extern "C" int grim_filter_windows(const grim_index_t *idx, const grim_batch_t *b,
                                   const uint32_t *win_lo, const uint32_t *order, int32_t *counts,
                                   uint32_t *pass_bits, void *workspace, uint64_t workspace_bytes,
                                   void *stream)
{
    if (!idx || !b)
        return GRIM_E_INVALID;
    if (b->e_den == 0 || b->max_len == 0 || (b->n_reads == 0 && b->n_pairs != 0))
        return GRIM_E_INVALID;
    if (b->max_len > 4096)
        return GRIM_E_UNSUPPORTED;
    if (b->n_reads && (!b->read_off || !b->read_len || !b->read_e || !b->cand_off || !win_lo ||
                       !b->reads_2bit || b->n_read_words == 0))
        return GRIM_E_INVALID;
    if (b->n_pairs && (!counts || !pass_bits))
        return GRIM_E_INVALID;
    if (!idx->d_rows)
        return GRIM_E_INVALID;
    if (!workspace || workspace_bytes < kWsHeader || (reinterpret_cast<uintptr_t>(workspace) & 255))
        return GRIM_E_INVALID;
    int dev = -1;
    int rc = current_device(&dev);
    if (rc)
        return rc;
    if (dev != idx->device)
        return GRIM_E_INVALID;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    WindowArgs a;
    std::memset(&a, 0, sizeof(a));
    a.rows = idx->d_rows;
    a.row_words = idx->row_words;
    a.rows_bytes = (1ull << (2 * idx->q)) * idx->row_words * 4 + 256;
    a.n_bins = idx->n_bins;
    a.rw = b->reads_2bit;
    a.nw = b->n_read_words;
    a.read_off = b->read_off;
    a.read_len = b->read_len;
    a.read_e = b->read_e;
    a.e_den = b->e_den;
    a.max_len = b->max_len;
    a.cand_off = b->cand_off;
    a.win_lo = win_lo;
    a.order = order;
    a.n_reads = b->n_reads;
    a.n_pairs = b->n_pairs;
    a.counts = counts;
    a.pass_bits = pass_bits;
    a.status = reinterpret_cast<uint32_t *>(workspace);
    a.counters = reinterpret_cast<uint64_t *>(a.status + kWindowFirst);
    a.npl = planes_for(idx->q, b->max_len);
    HIP_TRY(launch_zero2(s, a.status, kWsHeader / 4, pass_bits, (b->n_pairs + 31) / 32));
    if (b->n_reads == 0)
        return GRIM_OK;
    HIP_TRY(launch_window(s, idx->q, (uint32_t)cu_count(idx->device), (size_t)b->max_len * 4, a));
    return GRIM_OK;
}

extern "C" int grim_window_order_workspace_size(const grim_index_t *idx, uint64_t n_reads,
                                                uint64_t *bytes)
{
    (void)n_reads;
    if (!idx || !bytes)
        return GRIM_E_INVALID;
    uint32_t n_buckets = 0;
    order_shift(idx->n_bins, &n_buckets);
    *bytes = std::max<uint64_t>(256, ((uint64_t)n_buckets * 4 + 255) & ~255ull);
    return GRIM_OK;
}

extern "C" int grim_window_order(const grim_index_t *idx, const uint32_t *win_lo, uint64_t n_reads,
                                 uint32_t *order, void *workspace, uint64_t workspace_bytes,
                                 void *stream)
{
    if (!idx)
        return GRIM_E_INVALID;
    if (n_reads == 0)
        return GRIM_OK;
    if (!win_lo || !order || !workspace)
        return GRIM_E_INVALID;
    if (n_reads > 0xffffffffull)
        return GRIM_E_UNSUPPORTED;
    uint32_t n_buckets = 0;
    const uint32_t shift = order_shift(idx->n_bins, &n_buckets);
    if (workspace_bytes < (uint64_t)n_buckets * 4)
        return GRIM_E_INVALID;
    int dev = -1;
    int rc = current_device(&dev);
    if (rc)
        return rc;
    if (dev != idx->device)
        return GRIM_E_INVALID;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    uint32_t *cnt = reinterpret_cast<uint32_t *>(workspace);
    HIP_TRY(launch_zero(s, cnt, n_buckets));
    HIP_TRY(launch_window_order(s, (uint32_t)cu_count(idx->device), win_lo, (uint32_t)n_reads,
                                idx->n_bins, shift, n_buckets, cnt, order));
    return GRIM_OK;
}

// ---------------------------------------------------------------- probes
extern "C" int grim_probe_gather(const grim_index_t *idx, const uint32_t *ids, uint64_t n,
                                 int32_t *out, void *stream)
{
    if (!idx || (n && (!ids || !out)))
        return GRIM_E_INVALID;
    if (n == 0)
        return GRIM_OK;
    int dev = -1;
    int rc = current_device(&dev);
    if (rc)
        return rc;
    if (dev != idx->device)
        return GRIM_E_INVALID;
    HIP_TRY(launch_probe_gather(reinterpret_cast<hipStream_t>(stream), idx->q,
                                (uint32_t)cu_count(idx->device) * 8, idx->d_vec, idx->n_bins, ids,
                                n, out));
    return GRIM_OK;
}

extern "C" int grim_probe_stream(const grim_index_t *idx, uint32_t *sink, void *stream)
{
    if (!idx || !sink)
        return GRIM_E_INVALID;
    int dev = -1;
    int rc = current_device(&dev);
    if (rc)
        return rc;
    if (dev != idx->device)
        return GRIM_E_INVALID;
    HIP_TRY(launch_probe_stream(reinterpret_cast<hipStream_t>(stream),
                                (uint32_t)cu_count(idx->device) * 8, idx->d_vec, idx->bytes / 16,
                                sink));
    return GRIM_OK;
}

// ---------------------------------------------------------------- graphs
struct grim_graph {
    hipGraph_t graph;
    hipGraphExec_t exec;
};

extern "C" int grim_graph_create(const grim_index_t *idx, const grim_batch_t *b, int32_t *counts,
                                 uint32_t *pass_bits, void *workspace, uint64_t workspace_bytes,
                                 const grim_tuning_t *tune, grim_graph_t **out)
{
    int rc = check_batch(idx, b);
    if (rc)
        return rc;
    if (!out)
        return GRIM_E_INVALID;
    grim_tuning_t t;
    bool fixed = false;
    rc = resolve_tuning(idx, b->max_len, tune, &t, &fixed);
    if (rc)
        return rc;
    hipStream_t s;
    HIP_TRY(hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
    hipGraph_t graph = nullptr;
    hipError_t e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) {
        (void)hipStreamDestroy(s);
        return hip_fail(e, "hipStreamBeginCapture");
    }
    rc = enqueue_batched(idx, b, counts, pass_bits, workspace, workspace_bytes, t, fixed, s);
    e = hipStreamEndCapture(s, &graph);
    (void)hipStreamDestroy(s);
    if (rc) {
        if (graph)
            (void)hipGraphDestroy(graph);
        return rc;
    }
    if (e != hipSuccess)
        return hip_fail(e, "hipStreamEndCapture");
    grim_graph *g = new (std::nothrow) grim_graph();
    if (!g) {
        (void)hipGraphDestroy(graph);
        return GRIM_E_NOMEM;
    }
    g->graph = graph;
    e = hipGraphInstantiate(&g->exec, graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGraphDestroy(graph);
        delete g;
        return hip_fail(e, "hipGraphInstantiate");
    }
    *out = g;
    return GRIM_OK;
}

extern "C" int grim_graph_launch(grim_graph_t *g, void *stream)
{
    if (!g)
        return GRIM_E_INVALID;
    HIP_TRY(hipGraphLaunch(g->exec, reinterpret_cast<hipStream_t>(stream)));
    return GRIM_OK;
}

extern "C" void grim_graph_destroy(grim_graph_t *g)
{
    if (!g)
        return;
    (void)hipGraphExecDestroy(g->exec);
    (void)hipGraphDestroy(g->graph);
    delete g;
}
