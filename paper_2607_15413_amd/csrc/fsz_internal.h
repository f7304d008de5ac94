// Internal declarations shared by the kernel and host translation units of
// libfsz.so (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fsz.h"

namespace fsz {

// Format constants: block of 32 elements, tile of 8 blocks (Sec. III-A).
constexpr int kBlock = 32;
constexpr int kBlocksPerTile = 8;
constexpr int kTile = kBlock * kBlocksPerTile;
constexpr int kHeaderBytes = 32;

// Launch geometry.  One lane owns one 32-element block, so a wave64 holds 8
// tiles; a workgroup of kWaves waves owns one chunk of 8*kWaves tiles.
constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr int kTilesPerWave = 8;
constexpr int kTilesPerChunk = kTilesPerWave * kWaves;
constexpr uint64_t kWaveElems = (uint64_t)kTilesPerWave * kTile;
// Fields up to this size are one chunk of a compressor of 4 or 8 data waves and
// are compressed without a range pass, in one launch instead of two (us per
// call, one / two: 8192 elements 7.0 / 9.6, 16384 8.7 / 9.7; with 11 waves 22528
// elements would take 10.9 / 10.2).
constexpr uint64_t kSelfRangeMax = 8 * kWaveElems;
constexpr int kStatsThreads = 256;
constexpr int kStatsMaxBlocks = 1024;
constexpr int kRangeMaxBlocks = 256;  // workgroups (and partials) of the single-field range pass

// Per-lane LDS staging row: 32 floats + 4 dwords of padding (bank spread).
constexpr int kStageRowDwords = 36;
constexpr int kStageWaveDwords = 64 * kStageRowDwords;

// Chunk flag word for the decoupled lookback (Sec. IV-D): 2-bit state,
// 18-bit call epoch (stale words from earlier calls read as "not ready"),
// 1 error bit (OR-ed along the prefix), 43-bit byte count.
constexpr uint64_t kFlagAggregate = 1;
constexpr uint64_t kFlagInclusive = 2;
constexpr int kEpochBits = 18;
constexpr uint32_t kEpochMask = (1u << kEpochBits) - 1;
constexpr int kEpochShift = 44;
constexpr int kErrorBit = 43;
constexpr uint64_t kValueMask = (1ull << kErrorBit) - 1;
// Chunk c's flag word sits at index c * kFlagStride of a flag array (32 bytes
// apart, four per 128-byte line).  The words are read and written at agent
// scope from all XCDs; packed eight to a line they measurably slowed the
// compressor's data traffic, spread four to a line they did not.
constexpr uint64_t kFlagStride = 4;

// All prediction features on: cross-block state, centering, second order.
constexpr uint32_t kFeaturesAll = FSZ_FEATURES_ALL;

inline uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }
inline uint64_t pad16(uint64_t a) { return (a + 15) / 16 * 16; }

struct StatsPartial {
    float xmin, xmax, maxabs;
    uint32_t flags;
};

// A call's error bound (Sec. V-A) as the kernels use it: the step, its inverse,
// the stream header's flag bit 0 and the status.
struct Resolved {
    float E, inv;
    uint32_t flags;
    int status;
};

struct StatsArgs {
    const float *x;
    uint64_t n;
    fsz_stats *out;
    StatsPartial *partials;
};

struct CompressArgs {
    const float *x;
    uint64_t n, ntiles, nblocks, nchunks, data0;
    uint8_t *out;
    uint64_t capacity;
    const fsz_stats *stats;        // the caller's, or
    const StatsPartial *partials;  // of the call's own range pass (null: stats)
    uint32_t nparts;
    uint32_t self_range;  // no stats and no partials: the field is one chunk, which gives its range itself
    double value;
    int mode;
    uint32_t features;    // FSZ_FEAT_* switches (kFeaturesAll = the full method)
    uint32_t cfg_flags;   // header flags bits 2-4: tile configuration (0 = B 32, T 8)
    uint32_t epoch;       // 32-bit call epoch (result words)
    uint32_t flag_epoch;  // 18-bit nonzero epoch (chunk flags)
    unsigned long long *flags;
    unsigned long long *ticket;  // zero between launches (self-resetting)
    fsz_result *final;           // written by the workgroup owning the last chunk
};

struct DecompressArgs {
    const uint8_t *cmp;
    uint64_t cmp_size;
    float *out;  // element elem_begin of the field
    uint64_t n, ntiles, nblocks, nchunks, data0;
    // Decoded range: tiles [tile_begin, tile_end), elements [elem_begin,
    // elem_end) written (a whole field: all of them; the stream's total and
    // padding are then checked too).  The launch fills in the chunks that hold
    // them, [chunk_begin, nchunks).
    uint64_t tile_begin, tile_end, elem_begin, elem_end;
    uint64_t chunk_begin;
    uint32_t cfg_flags;  // tile-configuration decoders: the header flags bits 2-4 required
    // Decodes with the offsets pre-pass, which writes them: the
    // bytes of each group of 2^group_shift chunks (bit 63: a reserved rate-byte
    // bit) and each chunk's byte offset inside its group.
    const unsigned long long *groups;
    const unsigned long long *offsets;
    uint32_t group_shift;
    uint32_t groups_scanned;  // nonzero: the bytes before each group instead
    uint32_t epoch, flag_epoch;
    unsigned long long *flags;
    unsigned long long *ticket;  // zero between launches (self-resetting)
    fsz_result *final;           // written by the workgroup owning the last chunk
};

// ---- naive five-read baseline (Sec. V-C, Fig. 6): per-tile evaluation tables
// written by four evaluation passes (one per variant) and read by the encode
// pass.  Laid out [variant][tile] (cost), [variant][tile][block] (rates).
struct NaiveTables {
    uint32_t *cost;      // 4 * ntiles: tile cost C of LZ1, LZ2, LZ1c, LZ2c
    uint8_t *rates;      // 4 * ntiles * 8: block rates of each variant
    int32_t *mu;         // ntiles: quantized tile mean (written by the centred passes)
    uint8_t *centre_ok;  // ntiles: the mean is finite
};

// ---- offsets pre-pass of the decoders: geometry of its groups

constexpr int kGroupThreads = 256;
constexpr int kGroupTilesPerThread = 4;
constexpr int kGroupTiles = kGroupThreads * kGroupTilesPerThread;
constexpr uint64_t kMaxGroupWords = 512;
constexpr uint64_t kMaxGroupWgs = 65536;  // of a batch's pre-pass (256 per CU)
// Rounds of kGroupTiles tiles per group: the least power of two that leaves at
// most kMaxGroupWords groups.
inline uint32_t group_passes(uint64_t ntiles)
{
    uint32_t p = 1;
    while (ceil_div(ntiles, (uint64_t)kGroupTiles * p) > kMaxGroupWords) p *= 2;
    return p;
}

// ---- batched form: one launch over many jobs (compress or decompress)

constexpr int kSegElems = 32768;  // elements per workgroup of the batched range pass

// One job of a batch, as the kernels read it (built by the host, uploaded to
// device memory once per batch).  The compress jobs come first, then the
// decompress jobs, each in the caller's order and with counts of their own.
// Chunks of job j are items [chunk_base, chunk_base + nchunks) of its kind;
// its range-pass segments (compress) or tile groups (decompress) are
// [seg_base, seg_base + nsegs).
struct BatchJob {
    uint32_t op;  // FSZ_OP_COMPRESS or FSZ_OP_DECOMPRESS
    int32_t mode;
    uint64_t n, ntiles, nblocks, nchunks, data0;
    const void *src;
    uint64_t src_size;
    void *dst;
    uint64_t dst_capacity;
    double value;
    fsz_result *final;
    uint64_t chunk_base, seg_base, nsegs;
    uint32_t group_passes, group_shift;  // decompress: rounds of kGroupTiles per group, log2 of its chunks
};
static_assert(sizeof(BatchJob) == 128, "BatchJob layout");

struct BatchArgs {
    // compress jobs
    const BatchJob *jobs;
    const uint64_t *chunk_end;  // chunk_end[j] = chunk_base[j] + nchunks[j]
    const uint64_t *seg_end;    // seg_end[j] = seg_base[j] + nsegs[j]
    uint32_t njobs;
    uint32_t waves;             // data waves per workgroup: a chunk is 8 tiles per wave
    uint32_t epoch;             // result tag
    uint32_t *h_done;           // pinned: the first kernel stores the epoch there (null: nobody waits)
    uint64_t total_chunks, total_segs, nflags;  // nflags: flag words (kFlagStride per chunk)
    unsigned long long *flags;  // cleared by the batch's range pass
    unsigned long long *ticket; // zero between launches (self-resetting)
    Resolved *bounds;           // one per job
    StatsPartial *partials;     // one per segment
    // decompress jobs
    struct {
        const BatchJob *jobs;
        const uint64_t *chunk_end, *group_end;
        uint32_t njobs, tpc_log2;         // log2 of the tiles per chunk
        uint32_t group_wgs;               // workgroups that sum them: one each, up to kMaxGroupWgs
        uint64_t total_chunks, total_groups;
        unsigned long long *groups, *offsets;  // one word per group / per chunk
    } dec;
};

// Launch shape of the batched kernel: waves per workgroup (a chunk is 8 tiles
// per wave) and a cap on resident workgroups per CU (0 = no cap).
struct BatchShape {
    int waves = 4;
    int groups_per_cu = 0;
};

// Kernel launchers (fsz_kernels.hip).
hipError_t launch_stats(const StatsArgs &a, hipStream_t s);
// Its first part alone, for kernels that fold the partials themselves.
hipError_t launch_stats_partials(const StatsArgs &a, uint32_t *nparts, hipStream_t s);
hipError_t launch_compress(const CompressArgs &a, hipStream_t s);
// The five-read baseline: four evaluation launches, then the encode launch
// (a.nchunks counts chunks of kTilesPerChunk tiles).
hipError_t launch_compress_naive(const CompressArgs &a, const NaiveTables &t, bool in_aligned16, hipStream_t s);
// Decompression of a.tile_begin .. a.tile_end (range: of a part of the field).
// One launch whose workgroups add up the rate bytes before their chunk
// themselves while those are few (decode_by_prefix); otherwise the offsets
// pre-pass and a decoder, one chunk of 32 tiles per workgroup or, from
// dec_direct_below elements, a persistent grid over chunks of 64.  words
// (pre-pass only): kMaxGroupWords words and one per chunk of 32 tiles up to
// tile_end.
hipError_t launch_decompress(const DecompressArgs &a, unsigned long long *words, bool out_aligned16, bool range,
                             hipStream_t s);
// Pre-zeroed decompression (Sec. III-A): a fill of out[0, n) with +0.0, then the
// same launches with a decoder that skips waves whose tiles are all zero
// (persistent behind the pre-pass at every size).
hipError_t launch_decompress_prezero(const DecompressArgs &a, unsigned long long *words, bool out_aligned16,
                                     hipStream_t s);
// Tile configurations (Sec. VI-C), block in {32, 64}, tile_blocks in {4, 8, 16}:
// the pipelined compressor, whose chunks of kCfgPipeChunkSegs segments the
// launch counts itself (the flags must cover them), and a decoder with one
// chunk of kCfgDecWaves x 64 segments per workgroup (a.nchunks counts those).
hipError_t launch_compress_cfg(const CompressArgs &a, int block, int tile_blocks, hipStream_t s);
hipError_t launch_decompress_cfg(const DecompressArgs &a, int block, int tile_blocks, bool out_aligned16,
                                 hipStream_t s);
// The same decode with chunk offsets from a pre-pass over the rate header
// (a.nchunks counts chunks of kCfgDecChunkSegs segments; words has room for
// kMaxGroupWords words and one per chunk).
hipError_t launch_decompress_cfg_prescan(const DecompressArgs &a, unsigned long long *words, int block,
                                         int tile_blocks, bool out_aligned16, hipStream_t s);
constexpr int kCfgPipeChunkSegs = 8 * 64;  // the pipelined configuration compressor's chunk
// the configuration decoder: workgroups of 4 waves, one chunk of 4 x 64 segments each
// (the lookback form of fields above dec_wide_above elements: 16 waves)
constexpr int kCfgDecWaves = 4;
constexpr int kCfgDecChunkSegs = kCfgDecWaves * 64;
constexpr int kCfgDecWideWaves = 16;
// header flags bits 2-4 of a tile configuration (0 for B 32, T 8)
inline uint32_t cfg_flag_bits(int block, int tile_blocks)
{
    return (block == 64 ? 4u : 0u) | (tile_blocks == 4 ? 8u : tile_blocks == 16 ? 16u : 0u);
}
inline bool cfg_supported(int block, int tile_blocks)
{
    return (block == 32 || block == 64) && (tile_blocks == 4 || tile_blocks == 8 || tile_blocks == 16);
}
// Range pass + flag clear + offsets pre-pass, then the decompress jobs (one
// item per workgroup) with the per-job stats, then the compress jobs (a
// persistent pipelined kernel).
hipError_t launch_batch(const BatchArgs &b, bool aligned_out, const BatchShape &shape, hipStream_t s);
bool batch_shape_supported(const BatchShape &shape);

// Allocation-free compression: fsz_compress_async's work with every scratch
// word in a fixed device array (fsz_kernels.hip); n above 2^30 elements
// returns FSZ_ERR_TOO_LARGE.  Arguments already checked by the caller.
fsz_status compress_noalloc(const float *d_in, uint64_t n, int mode, double value, const fsz_stats *d_stats,
                            void *d_out, uint64_t cap, fsz_result *d_result, hipStream_t s);

// Host-side argument checks shared by every entry point (fsz_api.cpp).
bool aligned(const void *p, uintptr_t a);
bool valid_bound(int mode, double value);
fsz_status check_compress_args(const float *d_in, size_t n, int mode, double value, const void *d_out,
                               size_t cap);
fsz_status check_decompress_args(const void *d_cmp, size_t cmp_size, const float *d_out, size_t n);

// Sizes the batch workspace of `stream` for rounds of up to `jobs` jobs,
// `chunks` work items and `segs` range-pass segments, so that later batches
// within those limits allocate (and synchronize the device) never again.
bool reserve_batch(hipStream_t stream, uint64_t jobs, uint64_t chunks, uint64_t segs);

// Launch tuning knobs, process-wide, read once from the environment:
// FSZ_DEC_WIDE_ABOVE (the tile configurations'
// lookback decoder: 16-wave chunks above this many elements, else 4),
// FSZ_CFG_DEC_LOOKBACK_BELOW (decodes of
// the tile configurations below this many elements use
// the lookback decoder, larger ones the offsets pre-pass), FSZ_DEC_DIRECT_BELOW
// (pre-pass decodes below this size: one chunk per workgroup), FSZ_GRID_FACTOR
// (persistent workgroups per CU slot,
// default 1) and FSZ_PREZERO_CR (whole-field decodes of streams above this
// compression ratio, judged from the buffer size, use the pre-zeroed decoder).
struct Tuning {
    uint64_t dec_wide_above = 1ull << 21;  // tile configurations, lookback form: 16 waves above, else 4
    int grid_factor = 1;
    double prezero_min_cr = 0.0;  // whole-field decodes pre-zero above this CR (0: never)
    uint64_t cfg_dec_lookback_below = 1ull << 23;  // tile configurations: lookback below, pre-pass from here
    uint64_t dec_direct_below = 1ull << 26;    // pre-pass decodes below this size: one chunk per workgroup
};
const Tuning &tuning();

// Whether a decode of tiles [t0, t1) needs no offsets pre-pass: every workgroup
// reads the rate bytes before its chunk (8 per tile) itself.  That costs each
// of them a pass over at most kPrefixBytes and all of them together the reads
// summed here (for chunks of 64 tiles), against about 3.5 us for the pre-pass
// launch.  Whole fields, GRF at REL 1e-3, prefix / pre-pass in us per call: 2^20
// 6.4 / 8.7, 2^21 7.4 / 9.1, 2^22 9.0 / 9.9 (16.8 MB summed), 6.3 M 12.6 / 11.6
// (38 MB), 2^23 14.7 / 12.3; a range of 2^20 elements at 2^22 8.6 / 9.4 (9 MB),
// one of 1.7 M at 7.6 M 12.8 / 11.6 (27 MB).
constexpr uint64_t kPrefixBytes = 1ull << 18;
inline bool decode_by_prefix(uint64_t t0, uint64_t t1)
{
    const uint64_t chunks = ceil_div(t1 - t0, 64);
    return t1 * kBlocksPerTile <= kPrefixBytes && chunks * (t0 + t1) / 2 * kBlocksPerTile <= (18ull << 20);
}

// Waves per workgroup of the configuration decoder's lookback form for an
// n-element field (the pre-pass form always takes kCfgDecWaves).
inline int cfg_dec_lookback_waves(uint64_t n) { return n > tuning().dec_wide_above ? kCfgDecWideWaves : kCfgDecWaves; }

}  // namespace fsz
