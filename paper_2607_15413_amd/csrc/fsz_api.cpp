// C ABI of libfsz.so: argument validation, per-(device, stream) workspace,
// kernel launches, and the outcome of blocking calls from pinned memory.
#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <utility>
#include <vector>

#include "fsz_internal.h"

using namespace fsz;

namespace fsz {
const Tuning &tuning()
{
    static const Tuning t = [] {
        Tuning v;
        if (const char *e = std::getenv("FSZ_PREZERO_CR")) v.prezero_min_cr = std::atof(e);
        if (const char *e = std::getenv("FSZ_DEC_WIDE_ABOVE")) v.dec_wide_above = std::strtoull(e, nullptr, 10);
        if (const char *e = std::getenv("FSZ_CFG_DEC_LOOKBACK_BELOW"))
            v.cfg_dec_lookback_below = std::strtoull(e, nullptr, 10);
        if (const char *e = std::getenv("FSZ_DEC_DIRECT_BELOW")) v.dec_direct_below = std::strtoull(e, nullptr, 10);
        if (const char *e = std::getenv("FSZ_GRID_FACTOR")) {
            const int f = std::atoi(e);
            if (f >= 1 && f <= 64) v.grid_factor = f;
        }
        return v;
    }();
    return t;
}
}  // namespace fsz

namespace fsz {

bool aligned(const void *p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

bool valid_bound(int mode, double value)
{
    return (mode == FSZ_ABS || mode == FSZ_REL) && std::isfinite(value) && value > 0.0;
}

fsz_status check_compress_args(const float *d_in, size_t n, int mode, double value, const void *d_out,
                               size_t cap)
{
    if (!valid_bound(mode, value) || !d_out || (n > 0 && !d_in) || !aligned(d_in, 4) || !aligned(d_out, 4))
        return FSZ_ERR_INVALID_ARG;
    if (cap < kHeaderBytes + pad16(ceil_div(n, kBlock))) return FSZ_ERR_CAPACITY;
    return FSZ_OK;
}

fsz_status check_decompress_args(const void *d_cmp, size_t cmp_size, const float *d_out, size_t n)
{
    if (!d_cmp || (n > 0 && !d_out) || !aligned(d_cmp, 4) || !aligned(d_out, 4)) return FSZ_ERR_INVALID_ARG;
    if (cmp_size < (size_t)kHeaderBytes) return FSZ_ERR_CORRUPT;
    return FSZ_OK;
}

}  // namespace fsz

namespace {

// Pinned staging + device copy of one batch's job table.  The batch's first
// kernel, which starts behind the copy, stores the batch's epoch in the pinned
// word *h_done: once it is there the staging may be written again.  (An event
// recorded behind each batch cost 3.7 us of host time a call, the store none.)
struct DescSlot {
    void *h = nullptr;
    void *d = nullptr;
    size_t cap = 0;
    uint32_t *h_done = nullptr;
    uint32_t epoch = 0;  // of the batch that last used the slot (0: none)
};

struct Workspace {
    int device = 0;
    hipStream_t stream = nullptr;
    std::mutex mu;
    unsigned long long *d_flags = nullptr;  // chunk flag words
    uint64_t flags_cap = 0;
    unsigned long long *d_ticket = nullptr;  // chunk ticket, reset by each launch's last taker
    uint32_t call = 0;                       // per-call epoch
    fsz_result *h_final = nullptr;           // outcome of blocking calls: pinned, written by the kernel
    fsz_stats *d_stats = nullptr;            // range pass output when the caller has none
    StatsPartial *d_partials = nullptr;
    // batched form
    std::array<DescSlot, 4> ring;
    unsigned ring_next = 0;
    std::vector<DescSlot> captured;  // tables of batches captured into graphs
    unsigned long long *b_flags = nullptr;
    uint64_t b_flags_cap = 0;
    StatsPartial *b_partials = nullptr;
    uint64_t b_partials_cap = 0;
    Resolved *b_bounds = nullptr;
    uint64_t b_bounds_cap = 0;
    unsigned long long *b_ticket = nullptr;
    unsigned long long *b_words = nullptr;  // decompress jobs: group totals, chunk offsets
    uint64_t b_words_cap = 0;
    // five-read baseline: evaluation tables (53 bytes per tile)
    uint8_t *d_naive = nullptr;
    uint64_t naive_cap = 0;
    // decodes: group totals and chunk offsets of the pre-pass
    unsigned long long *d_offs = nullptr;
    uint64_t offs_cap = 0;
};

std::mutex g_mu;
std::map<std::pair<int, hipStream_t>, std::unique_ptr<Workspace>> g_ws;

bool ok(hipError_t e) { return e == hipSuccess; }


Workspace *get_workspace(hipStream_t s, fsz_status *st)
{
    int dev = 0;
    if (!ok(hipGetDevice(&dev))) {
        *st = FSZ_ERR_DEVICE;
        return nullptr;
    }
    std::lock_guard<std::mutex> g(g_mu);
    auto key = std::make_pair(dev, s);
    auto it = g_ws.find(key);
    if (it != g_ws.end()) return it->second.get();
    auto ws = std::make_unique<Workspace>();
    ws->device = dev;
    ws->stream = s;
    bool good = ok(hipMalloc(&ws->d_ticket, sizeof(unsigned long long))) &&
                ok(hipHostMalloc(&ws->h_final, sizeof(fsz_result) + ws->ring.size() * sizeof(uint32_t),
                                 hipHostMallocDefault)) &&
                ok(hipMalloc(&ws->d_stats, sizeof(fsz_stats))) &&
                ok(hipMalloc(&ws->d_partials, sizeof(StatsPartial) * kStatsMaxBlocks)) &&
                ok(hipMalloc(&ws->b_ticket, sizeof(unsigned long long))) &&
                ok(hipMemset(ws->d_ticket, 0, sizeof(unsigned long long))) &&
                ok(hipMemset(ws->b_ticket, 0, sizeof(unsigned long long))) &&
                ok(hipDeviceSynchronize());
    if (!good) {
        *st = FSZ_ERR_DEVICE;
        return nullptr;
    }
    *ws->h_final = fsz_result{};
    for (size_t k = 0; k < ws->ring.size(); k++) {
        ws->ring[k].h_done = reinterpret_cast<uint32_t *>(ws->h_final + 1) + k;
        *ws->ring[k].h_done = 0;
    }
    Workspace *raw = ws.get();
    g_ws.emplace(key, std::move(ws));
    return raw;
}

// While it lives, allocations are allowed on this thread although a stream is
// being captured.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    RelaxedCapture(const RelaxedCapture &) = delete;
    RelaxedCapture &operator=(const RelaxedCapture &) = delete;
};

// Make room for nchunks flag words.  The array that a larger one replaces stays
// allocated, here and in grow: an earlier launch may still use it, and a call
// captured into a graph names it at every replay.  Sizes double, so what stays
// is less than what is in use.
bool ensure_flags(Workspace *ws, uint64_t nchunks)
{
    if (nchunks <= ws->flags_cap) return true;
    uint64_t cap = ws->flags_cap ? ws->flags_cap : 1024;
    while (cap < nchunks) cap *= 2;
    unsigned long long *d = nullptr;
    if (!ok(hipMalloc(&d, cap * kFlagStride * sizeof(unsigned long long)))) return false;
    if (!ok(hipMemsetAsync(d, 0, cap * kFlagStride * sizeof(unsigned long long), ws->stream))) {
        (void)hipFree(d);
        return false;
    }
    ws->d_flags = d;
    ws->flags_cap = cap;
    return true;
}

// Next call epoch; clears the flag array whenever the 18-bit flag epoch wraps.
bool next_epoch(Workspace *ws, uint32_t *epoch, uint32_t *flag_epoch)
{
    if (++ws->call == 0) ++ws->call;
    *epoch = ws->call;
    *flag_epoch = (ws->call - 1) % kEpochMask + 1;
    if (*flag_epoch == 1 && ws->call > 1 && ws->d_flags)
        return ok(hipMemsetAsync(ws->d_flags, 0, ws->flags_cap * kFlagStride * sizeof(unsigned long long), ws->stream));
    return true;
}

// Blocking calls: wait for the stream; the kernel has stored the outcome in
// pinned memory (a copy behind the kernel cost 3 us a call).
fsz_status finish(Workspace *ws, uint32_t epoch, size_t *size_out)
{
    if (!ok(hipStreamSynchronize(ws->stream))) return FSZ_ERR_DEVICE;
    const volatile fsz_result *h = ws->h_final;
    const fsz_result r{h->size, h->status, h->epoch};
    if (r.epoch != epoch) return FSZ_ERR_DEVICE;
    if (r.status == FSZ_OK && size_out) *size_out = (size_t)r.size;
    return (fsz_status)r.status;
}

// Enqueue (range pass if d_stats is NULL) + compression kernel.
fsz_status enqueue_compress(Workspace *ws, const float *d_in, uint64_t n, int mode, double value,
                            const fsz_stats *d_stats, void *d_out, uint64_t cap, fsz_result *d_final,
                            uint32_t *epoch_out, uint32_t features = kFeaturesAll)
{
    CompressArgs a{};
    if (!d_stats && n > 0 && n <= kSelfRangeMax && features == kFeaturesAll) {
        a.self_range = 1;
    } else if (!d_stats) {
        StatsArgs sa{d_in, n, ws->d_stats, ws->d_partials};
        if (!ok(launch_stats_partials(sa, &a.nparts, ws->stream))) return FSZ_ERR_DEVICE;
        a.partials = ws->d_partials;
    }
    a.x = d_in;
    a.n = n;
    a.ntiles = ceil_div(n, kTile);
    a.nblocks = ceil_div(n, kBlock);
    a.nchunks = a.ntiles ? ceil_div(a.ntiles, kTilesPerChunk) : 1;
    a.data0 = kHeaderBytes + pad16(a.nblocks);
    a.out = static_cast<uint8_t *>(d_out);
    a.capacity = cap;
    a.stats = d_stats;
    a.value = value;
    a.mode = mode;
    a.features = features;
    // the pipelined kernel may use chunks as small as one wave's 8 tiles
    if (!ensure_flags(ws, std::max<uint64_t>(a.nchunks, ceil_div(a.ntiles, kTilesPerWave)))) return FSZ_ERR_DEVICE;
    if (!next_epoch(ws, &a.epoch, &a.flag_epoch)) return FSZ_ERR_DEVICE;
    a.flags = ws->d_flags;
    a.ticket = ws->d_ticket;
    a.final = d_final;
    if (!ok(launch_compress(a, ws->stream))) return FSZ_ERR_DEVICE;
    *epoch_out = a.epoch;
    return FSZ_OK;
}

template <typename T>
bool grow(T **p, uint64_t *cap, uint64_t want);

// Room for the offsets pre-pass of a decode, if it has one.
bool ensure_words(Workspace *ws, const DecompressArgs &a)
{
    if (decode_by_prefix(a.tile_begin, a.tile_end)) return true;
    return grow(&ws->d_offs, &ws->offs_cap, kMaxGroupWords + ceil_div(a.tile_end, (uint64_t)kTilesPerChunk) + 1);
}

// The five-read baseline (Sec. V-C, Fig. 6): the same stream as
// enqueue_compress, from four evaluation passes and one encode pass.
fsz_status enqueue_compress_naive(Workspace *ws, const float *d_in, uint64_t n, int mode, double value,
                                  const fsz_stats *d_stats, void *d_out, uint64_t cap, fsz_result *d_final)
{
    if (!d_stats) {
        StatsArgs sa{d_in, n, ws->d_stats, ws->d_partials};
        if (!ok(launch_stats(sa, ws->stream))) return FSZ_ERR_DEVICE;
        d_stats = ws->d_stats;
    }
    CompressArgs a{};
    a.x = d_in;
    a.n = n;
    a.ntiles = ceil_div(n, kTile);
    a.nblocks = ceil_div(n, kBlock);
    a.nchunks = a.ntiles ? ceil_div(a.ntiles, kTilesPerChunk) : 1;
    a.data0 = kHeaderBytes + pad16(a.nblocks);
    a.out = static_cast<uint8_t *>(d_out);
    a.capacity = cap;
    a.stats = d_stats;
    a.value = value;
    a.mode = mode;
    a.features = kFeaturesAll;
    const uint64_t nt = std::max<uint64_t>(a.ntiles, 1);
    const uint64_t off_rates = 16 * nt, off_mu = off_rates + 32 * nt, off_ok = off_mu + 4 * nt;
    if (!grow(&ws->d_naive, &ws->naive_cap, off_ok + nt)) return FSZ_ERR_DEVICE;
    NaiveTables t;
    t.cost = reinterpret_cast<uint32_t *>(ws->d_naive);
    t.rates = ws->d_naive + off_rates;
    t.mu = reinterpret_cast<int32_t *>(ws->d_naive + off_mu);
    t.centre_ok = ws->d_naive + off_ok;
    if (!ensure_flags(ws, a.nchunks)) return FSZ_ERR_DEVICE;
    if (!next_epoch(ws, &a.epoch, &a.flag_epoch)) return FSZ_ERR_DEVICE;
    a.flags = ws->d_flags;
    a.ticket = ws->d_ticket;
    a.final = d_final;
    if (!ok(launch_compress_naive(a, t, aligned(d_in, 16), ws->stream))) return FSZ_ERR_DEVICE;
    return FSZ_OK;
}

fsz_status enqueue_decompress(Workspace *ws, const void *d_cmp, uint64_t cmp_size, float *d_out, uint64_t n,
                              fsz_result *d_final, uint32_t *epoch_out, bool prezero = false)
{
    DecompressArgs a{};
    a.cmp = static_cast<const uint8_t *>(d_cmp);
    a.cmp_size = cmp_size;
    a.out = d_out;
    a.n = n;
    a.ntiles = ceil_div(n, kTile);
    a.nblocks = ceil_div(n, kBlock);
    a.data0 = kHeaderBytes + pad16(a.nblocks);
    a.tile_begin = 0;
    a.tile_end = a.ntiles;
    a.elem_begin = 0;
    a.elem_end = n;
    if (!ensure_words(ws, a)) return FSZ_ERR_DEVICE;
    if (!next_epoch(ws, &a.epoch, &a.flag_epoch)) return FSZ_ERR_DEVICE;
    a.final = d_final;
    const hipError_t e = prezero ? launch_decompress_prezero(a, ws->d_offs, aligned(d_out, 16), ws->stream)
                                 : launch_decompress(a, ws->d_offs, aligned(d_out, 16), false, ws->stream);
    if (!ok(e)) return FSZ_ERR_DEVICE;
    *epoch_out = a.epoch;
    return FSZ_OK;
}

// Whole-field decodes pick the pre-zeroed decoder for streams whose
// compression ratio, judged from the buffer size, exceeds the threshold.
bool auto_prezero(uint64_t n, uint64_t cmp_size)
{
    const double cr = tuning().prezero_min_cr;
    return cr > 0.0 && (double)(4 * n) > cr * (double)cmp_size;
}

// Tile configurations (Sec. VI-C, Table V): the generic lane-per-segment
// kernels, compression in chunks of kCfgPipeChunkSegs 32-element segments
// (decoder: 64 x kCfgDecWaves, or 64 x kCfgDecWideWaves in the lookback form
// of fields above dec_wide_above elements).
fsz_status enqueue_compress_config(Workspace *ws, const float *d_in, uint64_t n, int mode, double value,
                                   const fsz_stats *d_stats, int block, int tile_blocks, void *d_out, uint64_t cap,
                                   fsz_result *d_final)
{
    CompressArgs a{};
    if (!d_stats) {
        StatsArgs sa{d_in, n, ws->d_stats, ws->d_partials};
        if (!ok(launch_stats_partials(sa, &a.nparts, ws->stream))) return FSZ_ERR_DEVICE;
        a.partials = ws->d_partials;
    }
    a.x = d_in;
    a.n = n;
    a.ntiles = ceil_div(n, (uint64_t)block * tile_blocks);
    a.nblocks = ceil_div(n, (uint64_t)block);
    a.nchunks = n ? ceil_div(ceil_div(n, kBlock), kCfgPipeChunkSegs) : 1;
    a.data0 = kHeaderBytes + pad16(a.nblocks);
    a.out = static_cast<uint8_t *>(d_out);
    a.capacity = cap;
    a.stats = d_stats;
    a.value = value;
    a.mode = mode;
    a.features = kFeaturesAll;
    a.cfg_flags = cfg_flag_bits(block, tile_blocks);
    if (!ensure_flags(ws, a.nchunks)) return FSZ_ERR_DEVICE;
    if (!next_epoch(ws, &a.epoch, &a.flag_epoch)) return FSZ_ERR_DEVICE;
    a.flags = ws->d_flags;
    a.ticket = ws->d_ticket;
    a.final = d_final;
    if (!ok(launch_compress_cfg(a, block, tile_blocks, ws->stream))) return FSZ_ERR_DEVICE;
    return FSZ_OK;
}

fsz_status enqueue_decompress_config(Workspace *ws, const void *d_cmp, uint64_t cmp_size, float *d_out, uint64_t n,
                                     int block, int tile_blocks, fsz_result *d_final)
{
    DecompressArgs a{};
    a.cmp = static_cast<const uint8_t *>(d_cmp);
    a.cmp_size = cmp_size;
    a.out = d_out;
    a.n = n;
    a.ntiles = ceil_div(n, (uint64_t)block * tile_blocks);
    a.nblocks = ceil_div(n, (uint64_t)block);
    const bool prescan = n >= tuning().cfg_dec_lookback_below;
    const uint64_t chunk_segs = 64ull * (uint64_t)(prescan ? kCfgDecWaves : cfg_dec_lookback_waves(n));
    a.nchunks = n ? ceil_div(ceil_div(n, kBlock), chunk_segs) : 1;
    a.data0 = kHeaderBytes + pad16(a.nblocks);
    a.tile_begin = 0;
    a.tile_end = a.ntiles;
    a.elem_begin = 0;
    a.elem_end = n;
    a.cfg_flags = cfg_flag_bits(block, tile_blocks);
    if (!ensure_flags(ws, a.nchunks)) return FSZ_ERR_DEVICE;
    if (!next_epoch(ws, &a.epoch, &a.flag_epoch)) return FSZ_ERR_DEVICE;
    a.flags = ws->d_flags;
    a.ticket = ws->d_ticket;
    a.final = d_final;
    hipError_t e;
    if (prescan) {
        // chunk offsets from the rate header first, as for the default format
        if (!grow(&ws->d_offs, &ws->offs_cap, kMaxGroupWords + a.nchunks)) return FSZ_ERR_DEVICE;
        e = launch_decompress_cfg_prescan(a, ws->d_offs, block, tile_blocks, aligned(d_out, 16), ws->stream);
    } else {
        e = launch_decompress_cfg(a, block, tile_blocks, aligned(d_out, 16), ws->stream);
    }
    if (!ok(e)) return FSZ_ERR_DEVICE;
    return FSZ_OK;
}

// Random-access decode of elements [begin, end): the tiles that hold them,
// at the offset the rate header gives for the first one.
fsz_status enqueue_decompress_range(Workspace *ws, const void *d_cmp, uint64_t cmp_size, uint64_t n,
                                    uint64_t begin, uint64_t end, float *d_out, fsz_result *d_final)
{
    DecompressArgs a{};
    a.cmp = static_cast<const uint8_t *>(d_cmp);
    a.cmp_size = cmp_size;
    a.out = d_out;
    a.n = n;
    a.ntiles = ceil_div(n, kTile);
    a.nblocks = ceil_div(n, kBlock);
    a.data0 = kHeaderBytes + pad16(a.nblocks);
    a.tile_begin = begin / kTile;
    a.tile_end = end > begin ? ceil_div(end, kTile) : a.tile_begin;
    a.elem_begin = begin;
    a.elem_end = end;
    if (!ensure_words(ws, a)) return FSZ_ERR_DEVICE;
    if (!next_epoch(ws, &a.epoch, &a.flag_epoch)) return FSZ_ERR_DEVICE;
    a.final = d_final;
    // 16-byte stores need the field's element 0 (d_out - begin) 16-byte aligned
    const bool al16 = ((reinterpret_cast<uintptr_t>(d_out) - 4 * (uintptr_t)begin) & 15u) == 0;
    if (!ok(launch_decompress(a, ws->d_offs, al16, true, ws->stream))) return FSZ_ERR_DEVICE;
    return FSZ_OK;
}


// ------------------------------------------------------------------ batched form

// Device-side layout of a batch for one launch shape: the jobs of one kind, and
// both kinds (k[FSZ_OP_COMPRESS], k[FSZ_OP_DECOMPRESS]) one after the other.
struct KindLayout {
    std::vector<BatchJob> jobs;
    std::vector<uint64_t> chunk_end, seg_end;
    uint64_t total_chunks = 0, total_segs = 0;
    size_t bytes() const { return jobs.size() * (sizeof(BatchJob) + 2 * sizeof(uint64_t)); }
    char *pack(char *p) const
    {
        const size_t nj = jobs.size();
        if (nj == 0) return p;
        std::memcpy(p, jobs.data(), nj * sizeof(BatchJob));
        p += nj * sizeof(BatchJob);
        std::memcpy(p, chunk_end.data(), nj * sizeof(uint64_t));
        p += nj * sizeof(uint64_t);
        std::memcpy(p, seg_end.data(), nj * sizeof(uint64_t));
        return p + nj * sizeof(uint64_t);
    }
};
struct BatchLayout {
    KindLayout k[2];
    bool aligned_out = true;  // every decompress output is 16-byte aligned
    int waves = 4;           // decompress: per workgroup; a chunk is 8 tiles per wave
    int compress_waves = 8;  // compress: data waves per workgroup
    size_t desc_bytes() const { return k[0].bytes() + k[1].bytes(); }
    void pack(void *dst) const { (void)k[1].pack(k[0].pack(static_cast<char *>(dst))); }
    uint64_t flag_words() const { return k[FSZ_OP_COMPRESS].total_chunks * kFlagStride; }
    // the decompress jobs' group totals and chunk offsets
    uint64_t dec_words() const { return k[FSZ_OP_DECOMPRESS].total_segs + k[FSZ_OP_DECOMPRESS].total_chunks; }
};

// Data waves per workgroup of the batched compressor, for the elements of all
// its jobs: wide workgroups once there are enough items for the chip, narrow
// ones where the spread counts (us per call: 0.1 M elements in 2 jobs with 4
// waves 26, with 8 28; 3.0 M in 8 33.5 and 33.2; 7.0 M in 32 47 and 43, with 10
// 43; 125 M in 64 with 8 266, with 10 252, with 11 222).
int compress_batch_waves(uint64_t elems) { return elems >= (1ull << 23) ? 11 : elems >= (1ull << 21) ? 8 : 4; }

// Validates every job (nothing is enqueued unless all pass) and lays out
// global chunk and segment (or tile group) ranges of each kind in job order.
fsz_status layout_batch(const fsz_job *jobs, size_t njobs, int waves, BatchLayout *L)
{
    if (njobs > 0 && !jobs) return FSZ_ERR_INVALID_ARG;
    if (njobs >= (1u << 31)) return FSZ_ERR_INVALID_ARG;
    L->waves = waves;
    uint64_t celems = 0;
    for (size_t k = 0; k < njobs; k++) celems += jobs[k].op == FSZ_OP_COMPRESS ? jobs[k].n : 0;
    L->compress_waves = compress_batch_waves(celems);
    for (size_t k = 0; k < njobs; k++) {
        const fsz_job &j = jobs[k];
        if (!j.d_result) return FSZ_ERR_INVALID_ARG;
        fsz_status st;
        if (j.op == FSZ_OP_COMPRESS)
            st = check_compress_args(static_cast<const float *>(j.d_src), j.n, j.mode, j.value, j.d_dst,
                                     j.dst_capacity);
        else if (j.op == FSZ_OP_DECOMPRESS)
            st = check_decompress_args(j.d_src, j.src_size, static_cast<const float *>(j.d_dst), j.n);
        else
            st = FSZ_ERR_INVALID_ARG;
        if (st != FSZ_OK) return st;
        BatchJob J{};
        J.op = (uint32_t)j.op;
        J.mode = j.mode;
        J.n = j.n;
        J.ntiles = ceil_div(j.n, kTile);
        J.nblocks = ceil_div(j.n, kBlock);
        const uint64_t tiles_per_chunk =
            (uint64_t)kTilesPerWave * (uint64_t)(j.op == FSZ_OP_COMPRESS ? L->compress_waves : waves);
        J.nchunks = J.ntiles ? ceil_div(J.ntiles, tiles_per_chunk) : 1;
        J.data0 = kHeaderBytes + pad16(J.nblocks);
        J.src = j.d_src;
        J.src_size = j.op == FSZ_OP_DECOMPRESS ? j.src_size : 0;
        J.dst = j.d_dst;
        J.dst_capacity = j.op == FSZ_OP_COMPRESS ? j.dst_capacity : 0;
        J.value = j.value;
        J.final = j.d_result;
        KindLayout &K = L->k[j.op];
        J.chunk_base = K.total_chunks;
        K.total_chunks += J.nchunks;
        J.seg_base = K.total_segs;
        if (j.op == FSZ_OP_COMPRESS) {
            J.nsegs = ceil_div(j.n, kSegElems);
        } else {
            J.group_passes = group_passes(J.ntiles);
            const uint64_t tiles = (uint64_t)kGroupTiles * J.group_passes;
            J.nsegs = J.ntiles ? ceil_div(J.ntiles, tiles) : 1;
            J.group_shift = (uint32_t)__builtin_ctzll(tiles / tiles_per_chunk);
            L->aligned_out = L->aligned_out && aligned(j.d_dst, 16);
        }
        K.total_segs += J.nsegs;
        K.chunk_end.push_back(K.total_chunks);
        K.seg_end.push_back(K.total_segs);
        K.jobs.push_back(J);
    }
    // one work item per workgroup: grid x times workgroup size must fit 32 bits
    if ((L->k[0].total_chunks + L->k[1].total_chunks) * (uint64_t)(waves * 64) >= (1ull << 32) ||
        L->k[FSZ_OP_COMPRESS].total_segs * kStatsThreads >= (1ull << 32))
        return FSZ_ERR_INVALID_ARG;
    return FSZ_OK;
}

// As ensure_flags for buffers whose contents a call writes itself before it reads
// them: these may grow inside a capture, too.
template <typename T>
bool grow(T **p, uint64_t *cap, uint64_t want)
{
    if (want <= *cap) return true;
    uint64_t c = *cap ? *cap : 256;
    while (c < want) c *= 2;
    T *d = nullptr;
    RelaxedCapture relaxed;
    if (!ok(hipMalloc(&d, c * sizeof(T)))) return false;
    *p = d;
    *cap = c;
    return true;
}

BatchShape to_shape(const fsz_tuning &t)
{
    BatchShape s;
    s.waves = t.waves_per_group;
    s.groups_per_cu = t.groups_per_cu;
    return s;
}

// ---- autotune cache: best shape per (architecture, batch size class)

std::mutex g_tune_mu;
std::map<std::string, fsz_tuning> g_tune;
bool g_tune_loaded = false;

// Architecture name of the current device (cached per device; the caller
// holds g_tune_mu).
std::string arch_name()
{
    static std::map<int, std::string> names;
    int dev = 0;
    if (!ok(hipGetDevice(&dev))) return "unknown";
    auto it = names.find(dev);
    if (it != names.end()) return it->second;
    hipDeviceProp_t prop{};
    if (!ok(hipGetDeviceProperties(&prop, dev))) return "unknown";
    std::string a = prop.gcnArchName;
    const size_t colon = a.find(':');
    a = colon == std::string::npos ? a : a.substr(0, colon);
    names[dev] = a;
    return a;
}

int ilog2(uint64_t v)
{
    int l = 0;
    while (v > 1) {
        v >>= 1;
        l++;
    }
    return l;
}

// Size class: log2 of the total element count, log2 of the job count and
// which operations occur.
std::string size_class(const fsz_job *jobs, size_t njobs)
{
    uint64_t elems = 0;
    bool c = false, d = false;
    for (size_t k = 0; k < njobs; k++) {
        elems += jobs[k].n;
        (jobs[k].op == FSZ_OP_COMPRESS ? c : d) = true;
    }
    char buf[96];
    std::snprintf(buf, sizeof buf, "%s/e%d/j%d/%s%s", arch_name().c_str(), ilog2(elems + 1), ilog2(njobs + 1),
                  c ? "c" : "", d ? "d" : "");
    return buf;
}

void load_tune_file_locked()
{
    if (g_tune_loaded) return;
    g_tune_loaded = true;
    const char *path = std::getenv("FSZ_TUNE_CACHE");
    if (!path) return;
    FILE *f = std::fopen(path, "r");
    if (!f) return;
    char key[128];
    int w = 0, g = 0;
    while (std::fscanf(f, "%127s %d %d", key, &w, &g) == 3) g_tune[key] = fsz_tuning{w, g};
    std::fclose(f);
}

bool cached_tuning(const fsz_job *jobs, size_t njobs, fsz_tuning *out)
{
    std::lock_guard<std::mutex> g(g_tune_mu);
    load_tune_file_locked();
    auto it = g_tune.find(size_class(jobs, njobs));
    if (it == g_tune.end()) return false;
    *out = it->second;
    return true;
}

void store_tuning(const fsz_job *jobs, size_t njobs, const fsz_tuning &t)
{
    std::lock_guard<std::mutex> g(g_tune_mu);
    load_tune_file_locked();
    const std::string key = size_class(jobs, njobs);
    g_tune[key] = t;
    if (const char *path = std::getenv("FSZ_TUNE_CACHE")) {
        if (FILE *f = std::fopen(path, "a")) {
            std::fprintf(f, "%s %d %d\n", key.c_str(), t.waves_per_group, t.groups_per_cu);
            std::fclose(f);
        }
    }
}

fsz_status resolve_tuning(const fsz_job *jobs, size_t njobs, const fsz_tuning *tuning, fsz_tuning *out)
{
    if (tuning) {
        if (!batch_shape_supported(to_shape(*tuning))) return FSZ_ERR_INVALID_ARG;
        *out = *tuning;
        return FSZ_OK;
    }
    if (!cached_tuning(jobs, njobs, out)) *out = fsz_tuning{4, 0};
    return FSZ_OK;
}

BatchArgs batch_args(const BatchLayout &L, void *d_desc, uint32_t epoch, unsigned long long *flags,
                     unsigned long long *ticket, Resolved *bounds, StatsPartial *partials, unsigned long long *words)
{
    BatchArgs b{};
    const KindLayout &C = L.k[FSZ_OP_COMPRESS], &D = L.k[FSZ_OP_DECOMPRESS];
    auto table = [](char *p, const KindLayout &K, const BatchJob **jobs, const uint64_t **chunk_end,
                    const uint64_t **seg_end) {
        const size_t nj = K.jobs.size();
        *jobs = reinterpret_cast<const BatchJob *>(p);
        *chunk_end = reinterpret_cast<const uint64_t *>(p + nj * sizeof(BatchJob));
        *seg_end = reinterpret_cast<const uint64_t *>(p + nj * (sizeof(BatchJob) + sizeof(uint64_t)));
    };
    char *p = static_cast<char *>(d_desc);
    table(p, C, &b.jobs, &b.chunk_end, &b.seg_end);
    table(p + C.bytes(), D, &b.dec.jobs, &b.dec.chunk_end, &b.dec.group_end);
    b.njobs = (uint32_t)C.jobs.size();
    b.waves = (uint32_t)L.compress_waves;
    b.epoch = epoch;
    b.total_chunks = C.total_chunks;
    b.total_segs = C.total_segs;
    b.nflags = L.flag_words();
    b.flags = flags;
    b.ticket = ticket;
    b.bounds = bounds;
    b.partials = partials;
    b.dec.njobs = (uint32_t)D.jobs.size();
    b.dec.tpc_log2 = (uint32_t)__builtin_ctz((unsigned)(kTilesPerWave * L.waves));
    b.dec.total_chunks = D.total_chunks;
    b.dec.total_groups = D.total_segs;
    b.dec.group_wgs = (uint32_t)std::min(D.total_segs, kMaxGroupWgs);
    b.dec.groups = words;
    b.dec.offsets = words + D.total_segs;
    return b;
}

// Make a job-table slot hold `bytes` (its staging is idle).  As in grow the
// buffers that larger ones replace stay: the slot's last batch may still read
// the device copy, and freeing would wait for the whole device.
bool grow_slot(DescSlot &slot, size_t bytes)
{
    if (bytes <= slot.cap) return true;
    size_t c = 4096;
    while (c < bytes) c *= 2;
    void *h = nullptr, *d = nullptr;
    if (!ok(hipHostMalloc(&h, c, hipHostMallocDefault))) return false;
    if (!ok(hipMalloc(&d, c))) {
        (void)hipHostFree(h);
        return false;
    }
    slot.h = h;
    slot.d = d;
    slot.cap = c;
    return true;
}

// Waits until the slot's last batch has read its staging, i.e. has started:
// polls the slot's word and no more, since the stream may hold other batches and
// the caller's own work behind that one.  Every few ms the stream is looked at
// too: if nothing is left on it, the batch is done or was lost with an error.
// Rounds of 16 slices one behind the other, us per round: 40.8; 45.4 with a look
// every 4096 polls, which costs the GPU time; 42.8 with a wait for the whole
// stream after 4096 polls, which stopped the host for up to 210 us (64 fields of
// 125 M elements: 1.03 ms) and left the GPU idle meanwhile.
bool wait_slot(Workspace *ws, DescSlot &slot)
{
    if (!slot.epoch) return true;
    for (uint32_t k = 1; __atomic_load_n(slot.h_done, __ATOMIC_ACQUIRE) != slot.epoch; k++) {
        if (k % (1u << 12) == 0) std::this_thread::yield();
        if (k % (1u << 22)) continue;
        const hipError_t e = hipStreamQuery(ws->stream);
        if (e != hipErrorNotReady) return ok(e);
        if (hipPeekAtLastError() == hipErrorNotReady) (void)hipGetLastError();
    }
    return true;
}

// Enqueue one batch on the workspace's stream (caller holds ws->mu).
fsz_status enqueue_batch(Workspace *ws, const fsz_job *jobs, size_t njobs, const BatchShape &shape)
{
    BatchLayout L;
    fsz_status st = layout_batch(jobs, njobs, shape.waves, &L);
    if (st != FSZ_OK || njobs == 0) return st;
    if (!grow(&ws->b_flags, &ws->b_flags_cap, L.flag_words()) ||
        !grow(&ws->b_partials, &ws->b_partials_cap, L.k[FSZ_OP_COMPRESS].total_segs) ||
        !grow(&ws->b_bounds, &ws->b_bounds_cap, njobs) ||
        !grow(&ws->b_words, &ws->b_words_cap, L.dec_words()))
        return FSZ_ERR_DEVICE;
    // A batch captured into a graph reads its table again at every replay, when
    // nobody knows how often or until when: it gets buffers of its own, which
    // stay, and leaves the ring alone.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (!ok(hipStreamIsCapturing(ws->stream, &cap))) (void)hipGetLastError();
    const bool capturing = cap != hipStreamCaptureStatusNone;
    if (capturing) ws->captured.emplace_back();
    DescSlot &slot = capturing ? ws->captured.back() : ws->ring[ws->ring_next++ % ws->ring.size()];
    if (!wait_slot(ws, slot)) return FSZ_ERR_DEVICE;
    const size_t bytes = L.desc_bytes();
    if (capturing) {
        RelaxedCapture relaxed;
        if (!grow_slot(slot, bytes)) return FSZ_ERR_DEVICE;
    } else if (!grow_slot(slot, bytes)) {
        return FSZ_ERR_DEVICE;
    }
    L.pack(slot.h);
    if (!ok(hipMemcpyAsync(slot.d, slot.h, bytes, hipMemcpyHostToDevice, ws->stream))) return FSZ_ERR_DEVICE;
    if (++ws->call == 0) ++ws->call;
    BatchArgs b = batch_args(L, slot.d, ws->call, ws->b_flags, ws->b_ticket, ws->b_bounds, ws->b_partials, ws->b_words);
    if (!capturing) {
        b.h_done = slot.h_done;
        slot.epoch = ws->call;
    }
    return ok(launch_batch(b, L.aligned_out, shape, ws->stream)) ? FSZ_OK : FSZ_ERR_DEVICE;
}

}  // namespace

namespace fsz {

bool reserve_batch(hipStream_t stream, uint64_t jobs, uint64_t chunks, uint64_t segs)
{
    fsz_status st = FSZ_OK;
    Workspace *ws = get_workspace(stream, &st);
    if (!ws) return false;
    std::lock_guard<std::mutex> g(ws->mu);
    if (!grow(&ws->b_flags, &ws->b_flags_cap, std::max<uint64_t>(chunks, 1) * kFlagStride) ||
        !grow(&ws->b_partials, &ws->b_partials_cap, std::max<uint64_t>(segs, 1)) ||
        !grow(&ws->b_bounds, &ws->b_bounds_cap, std::max<uint64_t>(jobs, 1)) ||
        !grow(&ws->b_words, &ws->b_words_cap, chunks + segs))  // a tile group holds several segments
        return false;
    const size_t bytes = jobs * (sizeof(BatchJob) + 2 * sizeof(uint64_t));
    for (auto &slot : ws->ring) {
        if (!wait_slot(ws, slot)) return false;
        if (!grow_slot(slot, bytes)) return false;
    }
    return true;
}

}  // namespace fsz

// A captured batch (see fsz_plan_create).
struct fsz_plan {
    int device = 0;
    fsz_tuning tuning{4, 0};
    size_t njobs = 0;
    void *d_desc = nullptr;
    unsigned long long *d_flags = nullptr;
    unsigned long long *d_ticket = nullptr;
    StatsPartial *d_partials = nullptr;
    Resolved *d_bounds = nullptr;
    unsigned long long *d_words = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

namespace {

void free_plan(fsz_plan *p)
{
    if (!p) return;
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    (void)hipFree(p->d_desc);
    (void)hipFree(p->d_flags);
    (void)hipFree(p->d_ticket);
    (void)hipFree(p->d_partials);
    (void)hipFree(p->d_bounds);
    (void)hipFree(p->d_words);
    delete p;
}

uint32_t g_plan_ids = 0x80000000u;
}  // namespace

extern "C" {

size_t fsz_compressed_bound(size_t n)
{
    const uint64_t nblocks = ceil_div(n, kBlock);
    const uint64_t ntiles = ceil_div(n, kTile);
    return (size_t)(kHeaderBytes + pad16(nblocks) + 4 * ntiles + (4 + 4 * 31) * nblocks);
}

size_t fsz_compressed_bound_config(size_t n, int block, int tile_blocks)
{
    if (!cfg_supported(block, tile_blocks)) return 0;
    const uint64_t nblocks = ceil_div(n, (uint64_t)block);
    const uint64_t ntiles = ceil_div(n, (uint64_t)block * tile_blocks);
    return (size_t)(kHeaderBytes + pad16(nblocks) + 4 * ntiles + (uint64_t)(block / 8) * 32 * nblocks);
}

const char *fsz_status_string(fsz_status s)
{
    switch (static_cast<int>(s)) {  // C callers may pass any int
    case FSZ_OK: return "ok";
    case FSZ_ERR_INVALID_ARG: return "invalid argument";
    case FSZ_ERR_NONFINITE: return "input holds NaN or Inf";
    case FSZ_ERR_EB_TOO_SMALL: return "error bound below 8 ulp of max|x|";
    case FSZ_ERR_CAPACITY: return "output capacity too small";
    case FSZ_ERR_CORRUPT: return "corrupt stream";
    case FSZ_ERR_SIZE_MISMATCH: return "element count differs from the stream";
    case FSZ_ERR_DEVICE: return "HIP runtime error";
    case FSZ_ERR_EB_TOO_LARGE: return "error bound too large for the field magnitude";
    case FSZ_ERR_TOO_LARGE: return "field larger than the allocation-free scratch (2^30 elements)";
    default: return "unknown status";
    }
}

fsz_status fsz_field_stats(const float *d_in, size_t n, fsz_stats *d_stats, void *stream)
{
    if ((n > 0 && !d_in) || !d_stats || !aligned(d_in, 4)) return FSZ_ERR_INVALID_ARG;
    fsz_status st = FSZ_OK;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    StatsArgs a{d_in, n, d_stats, ws->d_partials};
    return ok(launch_stats(a, ws->stream)) ? FSZ_OK : FSZ_ERR_DEVICE;
}

fsz_status fsz_compress(const float *d_in, size_t n, fsz_eb_mode mode, double value, void *d_out,
                        size_t out_capacity, size_t *out_size, void *stream)
{
    return fsz_compress_ex(d_in, n, mode, value, nullptr, d_out, out_capacity, out_size, stream);
}

fsz_status fsz_compress_ex(const float *d_in, size_t n, fsz_eb_mode mode, double value,
                           const fsz_stats *d_stats, void *d_out, size_t out_capacity, size_t *out_size,
                           void *stream)
{
    if (!out_size) return FSZ_ERR_INVALID_ARG;
    fsz_status st = check_compress_args(d_in, n, mode, value, d_out, out_capacity);
    if (st != FSZ_OK) return st;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    uint32_t epoch = 0;
    st = enqueue_compress(ws, d_in, n, mode, value, d_stats, d_out, out_capacity, ws->h_final, &epoch);
    if (st != FSZ_OK) return st;
    return finish(ws, epoch, out_size);
}

fsz_status fsz_decompress(const void *d_cmp, size_t cmp_size, float *d_out, size_t n, void *stream)
{
    fsz_status st = check_decompress_args(d_cmp, cmp_size, d_out, n);
    if (st != FSZ_OK) return st;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    uint32_t epoch = 0;
    st = enqueue_decompress(ws, d_cmp, cmp_size, d_out, n, ws->h_final, &epoch, auto_prezero(n, cmp_size));
    if (st != FSZ_OK) return st;
    return finish(ws, epoch, nullptr);
}

fsz_status fsz_compress_async(const float *d_in, size_t n, fsz_eb_mode mode, double value,
                              const fsz_stats *d_stats, void *d_out, size_t out_capacity,
                              fsz_result *d_result, void *stream)
{
    if (!d_result) return FSZ_ERR_INVALID_ARG;
    fsz_status st = check_compress_args(d_in, n, mode, value, d_out, out_capacity);
    if (st != FSZ_OK) return st;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    uint32_t epoch = 0;
    return enqueue_compress(ws, d_in, n, mode, value, d_stats, d_out, out_capacity, d_result, &epoch);
}

fsz_status fsz_compress_features_async(const float *d_in, size_t n, fsz_eb_mode mode, double value,
                                       const fsz_stats *d_stats, unsigned features, void *d_out,
                                       size_t out_capacity, fsz_result *d_result, void *stream)
{
    if (!d_result || (features & ~(unsigned)FSZ_FEATURES_ALL) != 0) return FSZ_ERR_INVALID_ARG;
    fsz_status st = check_compress_args(d_in, n, mode, value, d_out, out_capacity);
    if (st != FSZ_OK) return st;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    uint32_t epoch = 0;
    return enqueue_compress(ws, d_in, n, mode, value, d_stats, d_out, out_capacity, d_result, &epoch, features);
}

fsz_status fsz_compress_five_read_async(const float *d_in, size_t n, fsz_eb_mode mode, double value,
                                        const fsz_stats *d_stats, void *d_out, size_t out_capacity,
                                        fsz_result *d_result, void *stream)
{
    if (!d_result) return FSZ_ERR_INVALID_ARG;
    fsz_status st = check_compress_args(d_in, n, mode, value, d_out, out_capacity);
    if (st != FSZ_OK) return st;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    return enqueue_compress_naive(ws, d_in, n, mode, value, d_stats, d_out, out_capacity, d_result);
}

fsz_status fsz_decompress_range_async(const void *d_cmp, size_t cmp_size, size_t n, size_t begin, size_t end,
                                      float *d_out, fsz_result *d_result, void *stream)
{
    if (!d_result || begin > end || end > n) return FSZ_ERR_INVALID_ARG;
    fsz_status st = check_decompress_args(d_cmp, cmp_size, d_out, end - begin);
    if (st != FSZ_OK) return st;
    // The range pass reads rate bytes before the decoder checks the header:
    // the buffer must hold every rate byte of an n-element stream.
    if (cmp_size < kHeaderBytes + pad16(ceil_div((uint64_t)n, kBlock))) return FSZ_ERR_CORRUPT;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    return enqueue_decompress_range(ws, d_cmp, cmp_size, n, begin, end, d_out, d_result);
}

fsz_status fsz_compress_config_async(const float *d_in, size_t n, fsz_eb_mode mode, double value,
                                     const fsz_stats *d_stats, int block, int tile_blocks, void *d_out,
                                     size_t out_capacity, fsz_result *d_result, void *stream)
{
    if (!d_result || !cfg_supported(block, tile_blocks) || !valid_bound(mode, value) || !d_out ||
        (n > 0 && !d_in) || !aligned(d_in, 4) || !aligned(d_out, 4))
        return FSZ_ERR_INVALID_ARG;
    if (out_capacity < kHeaderBytes + pad16(ceil_div(n, (uint64_t)block))) return FSZ_ERR_CAPACITY;
    fsz_status st = FSZ_OK;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    return enqueue_compress_config(ws, d_in, n, mode, value, d_stats, block, tile_blocks, d_out, out_capacity,
                                   d_result);
}

fsz_status fsz_decompress_config_async(const void *d_cmp, size_t cmp_size, float *d_out, size_t n, int block,
                                       int tile_blocks, fsz_result *d_result, void *stream)
{
    if (!d_result || !cfg_supported(block, tile_blocks)) return FSZ_ERR_INVALID_ARG;
    fsz_status st = check_decompress_args(d_cmp, cmp_size, d_out, n);
    if (st != FSZ_OK) return st;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    return enqueue_decompress_config(ws, d_cmp, cmp_size, d_out, n, block, tile_blocks, d_result);
}

fsz_status fsz_compress_noalloc_async(const float *d_in, size_t n, fsz_eb_mode mode, double value,
                                      const fsz_stats *d_stats, void *d_out, size_t out_capacity,
                                      fsz_result *d_result, void *stream)
{
    if (!d_result) return FSZ_ERR_INVALID_ARG;
    fsz_status st = check_compress_args(d_in, n, mode, value, d_out, out_capacity);
    if (st != FSZ_OK) return st;
    return compress_noalloc(d_in, n, mode, value, d_stats, d_out, out_capacity, d_result,
                            static_cast<hipStream_t>(stream));
}

fsz_status fsz_decompress_async(const void *d_cmp, size_t cmp_size, float *d_out, size_t n,
                                fsz_result *d_result, void *stream)
{
    if (!d_result) return FSZ_ERR_INVALID_ARG;
    fsz_status st = check_decompress_args(d_cmp, cmp_size, d_out, n);
    if (st != FSZ_OK) return st;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    uint32_t epoch = 0;
    return enqueue_decompress(ws, d_cmp, cmp_size, d_out, n, d_result, &epoch, auto_prezero(n, cmp_size));
}

fsz_status fsz_decompress_prezero_async(const void *d_cmp, size_t cmp_size, float *d_out, size_t n,
                                        fsz_result *d_result, void *stream)
{
    if (!d_result) return FSZ_ERR_INVALID_ARG;
    fsz_status st = check_decompress_args(d_cmp, cmp_size, d_out, n);
    if (st != FSZ_OK) return st;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    uint32_t epoch = 0;
    return enqueue_decompress(ws, d_cmp, cmp_size, d_out, n, d_result, &epoch, true);
}

fsz_status fsz_batch_async(const fsz_job *jobs, size_t njobs, const fsz_tuning *tuning, void *stream)
{
    if (njobs > 0 && !jobs) return FSZ_ERR_INVALID_ARG;
    fsz_tuning t{};
    fsz_status st = resolve_tuning(jobs, njobs, tuning, &t);
    if (st != FSZ_OK) return st;
    {
        BatchLayout L;  // host-side validation before any device work
        st = layout_batch(jobs, njobs, t.waves_per_group, &L);
        if (st != FSZ_OK || njobs == 0) return st;
    }
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    std::lock_guard<std::mutex> g(ws->mu);
    return enqueue_batch(ws, jobs, njobs, to_shape(t));
}

fsz_status fsz_autotune(const fsz_job *jobs, size_t njobs, int reps, void *stream, fsz_tuning *best)
{
    if (!best || reps < 1 || njobs == 0 || !jobs) return FSZ_ERR_INVALID_ARG;
    BatchLayout L;
    fsz_status st = layout_batch(jobs, njobs, 4, &L);
    if (st != FSZ_OK) return st;
    Workspace *ws = get_workspace(static_cast<hipStream_t>(stream), &st);
    if (!ws) return st;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (!ok(hipEventCreate(&e0)) || !ok(hipEventCreate(&e1))) return FSZ_ERR_DEVICE;
    float best_ms = 0.0f;
    bool found = false;
    st = FSZ_OK;
    const int waves[] = {2, 4, 8};
    const int groups[] = {0, 1, 2, 3, 4, 6};
    for (int w : waves) {
        for (int gcu : groups) {
            const fsz_tuning cand{w, gcu};
            // only decompress jobs are shaped: without them every shape runs the same kernels
            if (L.k[FSZ_OP_DECOMPRESS].jobs.empty() && (w != 4 || gcu != 0)) continue;
            if (!batch_shape_supported(to_shape(cand))) continue;
            std::lock_guard<std::mutex> g(ws->mu);
            st = enqueue_batch(ws, jobs, njobs, to_shape(cand));  // warm-up
            if (st != FSZ_OK) break;
            if (!ok(hipEventRecord(e0, ws->stream))) { st = FSZ_ERR_DEVICE; break; }
            for (int r = 0; r < reps && st == FSZ_OK; r++) st = enqueue_batch(ws, jobs, njobs, to_shape(cand));
            if (st != FSZ_OK) break;
            float ms = 0.0f;
            if (!ok(hipEventRecord(e1, ws->stream)) || !ok(hipEventSynchronize(e1)) ||
                !ok(hipEventElapsedTime(&ms, e0, e1))) {
                st = FSZ_ERR_DEVICE;
                break;
            }
            if (!found || ms < best_ms) {
                best_ms = ms;
                *best = cand;
                found = true;
            }
        }
        if (st != FSZ_OK) break;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != FSZ_OK) return st;
    if (!found) return FSZ_ERR_DEVICE;
    store_tuning(jobs, njobs, *best);
    return FSZ_OK;
}

fsz_status fsz_plan_create(const fsz_job *jobs, size_t njobs, const fsz_tuning *tuning, fsz_plan **plan)
{
    if (!plan || (njobs > 0 && !jobs)) return FSZ_ERR_INVALID_ARG;
    *plan = nullptr;
    fsz_tuning t{};
    fsz_status st = resolve_tuning(jobs, njobs, tuning, &t);
    if (st != FSZ_OK) return st;
    BatchLayout L;
    st = layout_batch(jobs, njobs, t.waves_per_group, &L);
    if (st != FSZ_OK) return st;
    auto *p = new fsz_plan();
    p->tuning = t;
    p->njobs = njobs;
    bool good = ok(hipGetDevice(&p->device));
    if (good && njobs > 0) {
        std::vector<char> host(L.desc_bytes());
        L.pack(host.data());
        hipStream_t cs = nullptr;
        good = ok(hipMalloc(&p->d_desc, host.size())) &&
               ok(hipMalloc(&p->d_flags, std::max<uint64_t>(L.flag_words(), 1) * sizeof(unsigned long long))) &&
               ok(hipMalloc(&p->d_words, std::max<uint64_t>(L.dec_words(), 1) * sizeof(unsigned long long))) &&
               ok(hipMalloc(&p->d_ticket, sizeof(unsigned long long))) &&
               ok(hipMalloc(&p->d_partials,
                            std::max<uint64_t>(L.k[FSZ_OP_COMPRESS].total_segs, 1) * sizeof(StatsPartial))) &&
               ok(hipMalloc(&p->d_bounds, njobs * sizeof(Resolved))) &&
               ok(hipMemcpy(p->d_desc, host.data(), host.size(), hipMemcpyHostToDevice)) &&
               ok(hipMemset(p->d_ticket, 0, sizeof(unsigned long long))) && ok(hipDeviceSynchronize()) &&
               ok(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
        if (good) {
            const BatchArgs b = batch_args(L, p->d_desc, g_plan_ids++, p->d_flags, p->d_ticket, p->d_bounds,
                                           p->d_partials, p->d_words);
            good = ok(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
            if (good) {
                const bool launched =
                    ok(launch_batch(b, L.aligned_out, to_shape(t), cs));
                const bool ended = ok(hipStreamEndCapture(cs, &p->graph));
                good = launched && ended && ok(hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0));
            }
        }
        if (cs) (void)hipStreamDestroy(cs);
    }
    if (!good) {
        free_plan(p);
        return FSZ_ERR_DEVICE;
    }
    *plan = p;
    return FSZ_OK;
}

fsz_status fsz_plan_launch(fsz_plan *plan, void *stream)
{
    if (!plan) return FSZ_ERR_INVALID_ARG;
    if (plan->njobs == 0) return FSZ_OK;
    return ok(hipGraphLaunch(plan->exec, static_cast<hipStream_t>(stream))) ? FSZ_OK : FSZ_ERR_DEVICE;
}

fsz_status fsz_plan_get_tuning(const fsz_plan *plan, fsz_tuning *out)
{
    if (!plan || !out) return FSZ_ERR_INVALID_ARG;
    *out = plan->tuning;
    return FSZ_OK;
}

void fsz_plan_destroy(fsz_plan *plan) { free_plan(plan); }

}  // extern "C"
