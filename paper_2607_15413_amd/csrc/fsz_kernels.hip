// FSZ compression / decompression kernels for MI355X (gfx950, CDNA4, wave64).
//
// Data layout on the GPU (the format itself is fixed by Sec. III-A / IV-C):
//   - one lane owns one 32-element block; lanes 8t..8t+7 of a wave own the
//     8 blocks of one 256-element tile, so a wave64 holds 8 tiles;
//   - the cross-block prediction state (Sec. IV-A, Eq. (2)) moves between
//     the lanes of a tile with one DPP row shift per block;
//   - per-tile reductions (mean, costs) use DPP within 8-lane groups.
// Compression is a persistent pipeline: a workgroup of 4, 8 or 11 data waves
// and a control wave takes chunks of 8 tiles per data wave by an atomic ticket,
// so that the decoupled lookback (Sec. IV-D), which the control wave walks, only
// ever waits on chunks already running; input is read once, by asynchronous
// copies to LDS a chunk ahead, and stays in VGPRs from the rate pass to the
// encode (the paper's kernel re-reads it instead).
// Decompression knows every chunk's offset before it starts, from the rate
// header alone (a sum in each workgroup for small fields, a pre-pass otherwise),
// so its workgroups wait on nobody.  The tile configurations' decoder for small
// fields and the five-read baseline keep one chunk per workgroup with a ticket
// and a lookback.
//
// Floating point: compiled with -ffp-contract=off; the quantizer is one
// binary32 multiply and a round-half-even (v_mul_f32, v_rndne_f32), the
// dequantizer one int->float conversion and one multiply.
#include "fsz_internal.h"

#include <float.h>

#include <mutex>
#include <utility>

namespace fsz {
namespace {

// ------------------------------------------------------------------ lanes

constexpr int kQuadXor1 = 0xB1;       // quad_perm:[1,0,3,2]
constexpr int kQuadXor2 = 0x4E;       // quad_perm:[2,3,0,1]
constexpr int kRowShr1 = 0x111;
constexpr int kRowShr2 = 0x112;
constexpr int kRowShr4 = 0x114;
constexpr int kRowShr8 = 0x118;
constexpr int kRowHalfMirror = 0x141;
constexpr int kRowBcast15 = 0x142;
constexpr int kRowBcast31 = 0x143;

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ int dpp(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xF, true);
}

template <int CTRL>
__device__ __forceinline__ float dppf(float v)
{
    return __int_as_float(dpp<CTRL>(__float_as_int(v)));
}

// value of lane 8*(lane/8) (block 0 of the lane's tile), in registers: each
// quad takes its first lane, then banks 1 and 3 of every row (lanes 4-7,
// 12-15) take the quad 4 lanes below
__device__ __forceinline__ int group_head(int v)
{
    v = dpp<0x00>(v);  // quad_perm:[0,0,0,0]
    return __builtin_amdgcn_update_dpp(v, v, kRowShr4, 0xF, 0xA, false);
}

// sum over the 8 lanes of a tile, result in all 8 lanes
__device__ __forceinline__ int group_sum(int v)
{
    v += dpp<kQuadXor1>(v);
    v += dpp<kQuadXor2>(v);
    v += dpp<kRowHalfMirror>(v);
    return v;
}

// exclusive prefix over the 8 lanes of a tile (j = lane & 7)
__device__ __forceinline__ uint32_t group_excl_scan(uint32_t v, int j)
{
    uint32_t s = v;
    uint32_t t = (uint32_t)dpp<kRowShr1>((int)s);
    s += j >= 1 ? t : 0u;
    t = (uint32_t)dpp<kRowShr2>((int)s);
    s += j >= 2 ? t : 0u;
    t = (uint32_t)dpp<kRowShr4>((int)s);
    s += j >= 4 ? t : 0u;
    return s - v;
}

// inclusive prefix over the 64 lanes of the wave
__device__ __forceinline__ int wave_incl_scan(int v)
{
    v += dpp<kRowShr1>(v);
    v += dpp<kRowShr2>(v);
    v += dpp<kRowShr4>(v);
    v += dpp<kRowShr8>(v);
    v += dpp<kRowBcast15, 0xA>(v);
    v += dpp<kRowBcast31, 0xC>(v);
    return v;
}

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ unsigned long long dpp64(unsigned long long v)
{
    const uint32_t lo = (uint32_t)dpp<CTRL, ROW_MASK>((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)dpp<CTRL, ROW_MASK>((int)(uint32_t)(v >> 32));
    return (unsigned long long)hi << 32 | lo;
}

// sum over the 64 lanes of the wave (register-only prefix, total of lane
// 63); the result is wave-uniform.  Every lane must be active.
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
    v += dpp64<kRowShr1>(v);
    v += dpp64<kRowShr2>(v);
    v += dpp64<kRowShr4>(v);
    v += dpp64<kRowShr8>(v);
    v += dpp64<kRowBcast15, 0xA>(v);
    v += dpp64<kRowBcast31, 0xC>(v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, 63);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), 63);
    return (unsigned long long)hi << 32 | lo;
}

// a value that every lane holds, in scalar registers
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint64_t uniform(uint64_t v)
{
    return (uint64_t)uniform((uint32_t)(v >> 32)) << 32 | uniform((uint32_t)v);
}

// Workgroup barrier that orders LDS only: the waves of a workgroup exchange
// data through LDS alone, so outstanding global loads and stores (such as
// the asynchronous copies of a prefetched chunk, which a release fence would
// wait for) stay in flight across it.  The wave's own LDS accesses complete
// before the barrier (lgkmcnt(0)); the memory clobber keeps the compiler
// from moving memory accesses across it.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Global-memory views of the hot loads and stores.  Pointers that come out of
// a job table (the batched forms) carry no address space, and the compiler
// accesses them with FLAT instructions, whose waits also cover LDS traffic;
// accesses through these types are plain global loads and stores.
typedef __attribute__((address_space(1))) uint8_t g_u8;
typedef __attribute__((address_space(1))) uint32_t g_u32;
typedef __attribute__((address_space(1))) float g_f32;
typedef __attribute__((address_space(1))) u32x4 g_u32x4;
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));
typedef __attribute__((address_space(1))) u32x4_a4 g_u32x4_a4;  // 16 bytes at a 4-byte aligned address

// Store of nw dwords from a wave's LDS staging area to global memory at a
// 4-byte aligned address g, by the whole wave: 4-byte stores up to the first
// 16-byte boundary of g and after the last one, 16-byte stores in between (a
// quarter of the store instructions of a dword-wide copy).
__device__ __forceinline__ void wave_store_staged(uint32_t *gp, const uint32_t *st, uint32_t nw, int lane)
{
    g_u32 *g = (g_u32 *)gp;
    const uint32_t head = min(nw, ((16u - ((uint32_t)(uintptr_t)gp & 15u)) & 15u) >> 2);
    if ((uint32_t)lane < head) g[lane] = st[lane];
    const uint32_t nq = (nw - head) >> 2;
    for (uint32_t q = lane; q < nq; q += 64) {
        const uint32_t o = head + 4 * q;
        const u32x4 v = {st[o], st[o + 1], st[o + 2], st[o + 3]};
        *reinterpret_cast<g_u32x4 *>(g + o) = v;
    }
    const uint32_t t0 = head + 4 * nq;
    if ((uint32_t)lane < nw - t0) g[t0 + lane] = st[t0 + lane];
}

// As wave_store_staged, for a staging area laid out at the same 16-byte
// phase as g (st + head is 16-byte aligned): the body is read with one
// 16-byte LDS read per lane (consecutive lanes, consecutive 16 bytes), free of
// bank conflicts.
__device__ __forceinline__ void wave_store_staged_phased(uint32_t *gp, const uint32_t *st, uint32_t nw, int lane)
{
    g_u32 *g = (g_u32 *)gp;
    const uint32_t head = min(nw, ((16u - ((uint32_t)(uintptr_t)gp & 15u)) & 15u) >> 2);
    if ((uint32_t)lane < head) g[lane] = st[lane];
    const uint32_t nq = (nw - head) >> 2;
    for (uint32_t q = lane; q < nq; q += 64) {
        const uint32_t o = head + 4 * q;
        *reinterpret_cast<g_u32x4 *>(g + o) = *reinterpret_cast<const u32x4 *>(st + o);
    }
    const uint32_t t0 = head + 4 * nq;
    if ((uint32_t)lane < nw - t0) g[t0 + lane] = st[t0 + lane];
}

__device__ __forceinline__ uint32_t uabs(int v) { return v < 0 ? 0u - (uint32_t)v : (uint32_t)v; }

// number of significant bits = ceil(log2(v + 1)) (the rate of Sec. IV-A)
__device__ __forceinline__ uint32_t bitlen(uint32_t v) { return v ? 32u - (uint32_t)__builtin_clz(v) : 0u; }

// Eq. (3): zero-rate blocks cost nothing, else a sign word and r planes
__device__ __forceinline__ uint32_t block_bytes(uint32_t r) { return r ? 4u + 4u * r : 0u; }

__device__ __forceinline__ uint32_t bswap32(uint32_t v) { return __builtin_bswap32(v); }

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) f4 g_f4;  // global-memory view (see g_u32)

// ------------------------------------------------------------------ bit planes
//
// Bit-shuffle (Sec. IV-C) as an in-register transpose.  A block's residual
// codes c[i] = (|l_i| << 1) | sign_i hold the sign in bit 0 and magnitude bit
// p in bit p + 1, so the block's stored words are exactly the bit planes of
// the codes: word b = bit b of every code (word 0 = sign map, word b = plane
// b - 1).  Stored words are written most-significant byte first, so in the
// little-endian dword element i sits at bit i ^ 7.
//
// Eight planes at a time (byte g of the codes): registers R[rho] take byte g
// of codes 8k + 7 - rho in their byte k; three delta-swap stages exchange the
// register index with the bit-in-byte index, after which R[p] is the stored
// dword of plane word 8g + p.  The same stages invert the mapping on decode.

// byte g of a0..a3 packed into bytes 0..3
__device__ __forceinline__ uint32_t pack_byte_g(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t g)
{
    const uint32_t sel = g | ((4u + g) << 8) | 0x0C0C0000u;
    const uint32_t t01 = __builtin_amdgcn_perm(a1, a0, sel);
    const uint32_t t23 = __builtin_amdgcn_perm(a3, a2, sel);
    return __builtin_amdgcn_perm(t23, t01, 0x05040100u);
}

template <int D, uint32_t M>
__device__ __forceinline__ void delta_swap(uint32_t &lo, uint32_t &hi)
{
    const uint32_t nlo = (M & (hi << D)) | (~M & lo);
    const uint32_t nhi = (M & hi) | (~M & (lo >> D));
    lo = nlo;
    hi = nhi;
}

// swaps the register index (0..7) with the bit-in-byte index of every byte
__device__ __forceinline__ void transpose8(uint32_t (&R)[8])
{
    delta_swap<1, 0xAAAAAAAAu>(R[0], R[1]);
    delta_swap<1, 0xAAAAAAAAu>(R[2], R[3]);
    delta_swap<1, 0xAAAAAAAAu>(R[4], R[5]);
    delta_swap<1, 0xAAAAAAAAu>(R[6], R[7]);
    delta_swap<2, 0xCCCCCCCCu>(R[0], R[2]);
    delta_swap<2, 0xCCCCCCCCu>(R[1], R[3]);
    delta_swap<2, 0xCCCCCCCCu>(R[4], R[6]);
    delta_swap<2, 0xCCCCCCCCu>(R[5], R[7]);
    delta_swap<4, 0xF0F0F0F0u>(R[0], R[4]);
    delta_swap<4, 0xF0F0F0F0u>(R[1], R[5]);
    delta_swap<4, 0xF0F0F0F0u>(R[2], R[6]);
    delta_swap<4, 0xF0F0F0F0u>(R[3], R[7]);
}

// ------------------------------------------------------------------ results

// The call's outcome, written once per launch by the workgroup that owns the
// last chunk (it sees the inclusive prefix, hence every chunk's error bit).
__device__ __forceinline__ void write_final(fsz_result *final, uint64_t size, uint32_t status, uint32_t epoch)
{
    final->size = status == FSZ_OK ? size : 0;
    final->status = status;
    final->epoch = epoch;
}

// ------------------------------------------------------------------ bound

// binary32 spacing at magnitude m, from its exponent field
__device__ __forceinline__ double spacing32(float m)
{
    uint32_t e = (__float_as_uint(m) >> 23) & 0xFFu;
    int p = e == 0 ? -149 : (int)e - 150;
    return __longlong_as_double((long long)(p + 1023) << 52);
}

// d (> 0) to binary32, rounding toward zero
__device__ __forceinline__ float f32_toward_zero(double d)
{
    float f = (float)d;
    if ((double)f > d) f = __uint_as_float(__float_as_uint(f) - 1u);
    return f;
}

// a - b (a > b > 0) rounded toward zero in binary64: the round-to-nearest
// difference plus its exact two-sum error term; a negative error means the
// rounding went up, so the result steps one unit down.  Truncated again to
// binary32 it gives the exact difference truncated to binary32.
__device__ __forceinline__ double sub_toward_zero(double a, double b)
{
    double s = a - b;
    const double bb = s - a;
    const double e = (a - (s - bb)) + (-b - bb);
    if (e < 0.0) s = __longlong_as_double(__double_as_longlong(s) - 1);
    return s;
}

// Error-bound resolution (Sec. V-A) with the binary32 step tightening:
// E = the largest binary32 <= 2 (eb - 4 ulp(max|x|)), inv = 1/E.
__device__ Resolved resolve_bound(const fsz_stats &s, int mode, double value, uint64_t n)
{
    Resolved r{1.0f, 1.0f, 0u, FSZ_OK};
    if (n == 0) return r;
    if (s.flags & 1u) {
        r.status = FSZ_ERR_NONFINITE;
        return r;
    }
    float E;
    if (mode == FSZ_REL && s.xmax == s.xmin) {
        const float c = fabsf(s.xmin);
        if (c == 0.0f) {
            E = 1.0f;
        } else if (c < FLT_MIN) {
            r.status = FSZ_ERR_EB_TOO_SMALL;
            return r;
        } else {
            E = c;
        }
        r.flags = 1;
    } else {
        const double eb = mode == FSZ_REL ? value * ((double)s.xmax - (double)s.xmin) : value;
        const double u = spacing32(s.maxabs);
        if (!(eb >= 8.0 * u)) {
            r.status = FSZ_ERR_EB_TOO_SMALL;
            return r;
        }
        const double ebq = sub_toward_zero(eb, 4.0 * u);
        E = f32_toward_zero(2.0 * ebq);
        if (E > 0x1p126f) E = 0x1p126f;
        if (E < FLT_MIN) {
            r.status = FSZ_ERR_EB_TOO_SMALL;
            return r;
        }
        if ((double)s.maxabs + (double)E > (double)FLT_MAX) {
            r.status = FSZ_ERR_EB_TOO_LARGE;
            return r;
        }
    }
    r.E = E;
    r.inv = 1.0f / E;
    return r;
}

// ------------------------------------------------------------------ lookback

constexpr uint32_t kLookbackSpinLimit = 1u << 22;

// Chunk ids come from the launch's ticket counter, so a chunk is only ever
// owned by a running workgroup and the lookback always makes progress.
// A grid of G workgroups takes `takes` tickets in total (G for one chunk per
// workgroup; nchunks + G for a persistent grid, whose workgroups take tickets
// until one is out of range); the last take resets the counter for the next
// launch on the stream.
__device__ __forceinline__ unsigned long long take_ticket(unsigned long long *ticket, uint64_t takes)
{
    const unsigned long long t = atomicAdd(ticket, 1ull);
    if (t == takes - 1) __hip_atomic_store(ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return t;
}

__device__ __forceinline__ unsigned long long pack_flag(uint64_t state, uint32_t ep, bool err, uint64_t v)
{
    return (state << 62) | ((uint64_t)ep << kEpochShift) | ((uint64_t)err << kErrorBit) | (v & kValueMask);
}

// Decoupled lookback (Sec. IV-D, three-state flags) run by one whole wave:
// publishes this chunk's aggregate, sums predecessors' aggregates 64 at a
// time until an inclusive prefix is found, publishes the inclusive prefix
// and returns the exclusive one.  Each flag word also carries an error bit
// that is OR-ed along the prefix, so the last chunk learns whether any chunk
// failed.  Flags are plain relaxed agent-scope atomics (coherent across the
// 8 XCDs' L2s, no cache-flushing fences): the value travels inside the flag
// word, so no other memory needs ordering.  The spin is bounded so that every
// wave exits even if the protocol were broken (*err is then set).
struct Prefix {
    uint64_t excl;
    bool err;
};

// Publishes this chunk's aggregate (chunk 0 publishes its inclusive prefix).
__device__ __forceinline__ void publish_aggregate(unsigned long long *flags, uint64_t chunk, uint32_t ep,
                                                  uint64_t total, bool err)
{
    __hip_atomic_store(&flags[chunk * kFlagStride], pack_flag(chunk == 0 ? kFlagInclusive : kFlagAggregate, ep, err, total),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits for the exclusive prefix of `chunk` (whose aggregate is published)
// and publishes its inclusive prefix.  Run by one whole wave.  A probe reads
// the 64 nearest unresolved predecessors; while one of them is not ready the
// wave re-reads only that single flag word (with a short sleep), so waiting
// chunks add little memory traffic, and then probes the window again.
//
// The caller may read the nearest kProbeWindows windows ahead of time
// (window m, lane l: the flag of chunk - 1 - 64 m - l); the lookback walks
// those values before it issues a load of its own.  A flag that was ready
// when it was read stays valid (an aggregate or an inclusive prefix of this
// launch never changes value); a window read ahead that still shows a word
// not ready is read again before the wave waits on that word.  One window:
// flag words are read across the XCDs' caches at agent scope, and on the
// 512^3 field one more window read ahead per step (walked or not) cost the
// compressor more time than the walks it saved.
constexpr int kProbeWindows = 1;
struct Probe {
    unsigned long long f[kProbeWindows];
};

__device__ __forceinline__ Probe lookback_probe(unsigned long long *flags, uint64_t chunk, uint32_t ep)
{
    Probe p;
#pragma unroll
    for (int m = 0; m < kProbeWindows; m++) {
        const long long idx = (long long)chunk - 1 - 64 * m - __lane_id();
        p.f[m] = idx >= 0 ? __hip_atomic_load(&flags[idx * kFlagStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                          : pack_flag(kFlagInclusive, ep, false, 0);
    }
    return p;
}

// Makes the probe's loads complete here on every path (an empty asm that
// reads the registers).
__device__ __forceinline__ void consume_probe(const Probe &p)
{
#pragma unroll
    for (int m = 0; m < kProbeWindows; m++) asm volatile("; probe %0" ::"v"(p.f[m]));
}

__device__ Prefix lookback_wait(unsigned long long *flags, uint64_t chunk, uint32_t ep, uint64_t total, bool err,
                                bool has_probe = false, Probe probe = Probe{})
{
    const int lane = __lane_id();
    if (chunk == 0) return Prefix{0, err};
    uint64_t excl = 0;
    bool perr = false;
    long long pos = (long long)chunk - 1;
    uint32_t spins = 0;
    auto state_of = [&](unsigned long long f) -> uint32_t {
        return (uint32_t)((f >> kEpochShift) & kEpochMask) == ep ? (uint32_t)(f >> 62) : 0u;
    };
    int window = has_probe ? 0 : kProbeWindows;  // windows walked so far (read-ahead ones first)
    bool reread = false;                          // read the current window now
    for (;;) {
        const long long idx = pos - lane;
        const bool ahead = window < kProbeWindows && !reread;
        unsigned long long f;
        if (ahead) {
            f = probe.f[0];
#pragma unroll
            for (int m = 1; m < kProbeWindows; m++) f = window == m ? probe.f[m] : f;
        } else {
            f = idx >= 0 ? __hip_atomic_load(&flags[idx * kFlagStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                         : pack_flag(kFlagInclusive, ep, false, 0);
        }
        const uint32_t state = state_of(f);
        const unsigned long long not_ready = __ballot(state == 0);
        const unsigned long long incl = __ballot(state == kFlagInclusive);
        const uint64_t v = f & kValueMask;
        const bool e = (f >> kErrorBit) & 1ull;
        const unsigned long long need =
            incl ? (__builtin_ctzll(incl) >= 63 ? ~0ull : ((2ull << __builtin_ctzll(incl)) - 1ull)) : ~0ull;
        if ((not_ready & need) == 0) {
            if (incl != 0) {
                const int first = __builtin_ctzll(incl);
                excl += wave_sum_u64(lane <= first ? v : 0);
                perr = perr || (__ballot(lane <= first && e) != 0);
                break;
            }
            excl += wave_sum_u64(v);
            perr = perr || (__ballot(e) != 0);
            pos -= 64;
            window = window < kProbeWindows ? window + 1 : kProbeWindows;
            reread = false;
            continue;
        }
        reread = true;
        if (ahead) continue;  // the read-ahead values are old: read the window first
        // wait on the nearest predecessor that is not ready yet, then read
        // this window again
        const long long widx = pos - __builtin_ctzll(not_ready & need);
        for (;;) {
            if (++spins >= kLookbackSpinLimit) break;
            __builtin_amdgcn_s_sleep(2);
            const unsigned long long g =
                __hip_atomic_load(&flags[widx * kFlagStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (state_of(g) != 0) break;
        }
        if (spins >= kLookbackSpinLimit) {  // a predecessor never published: give up
            perr = true;
            break;
        }
    }
    err = err || perr;
    if (lane == 0)
        __hip_atomic_store(&flags[chunk * kFlagStride], pack_flag(kFlagInclusive, ep, err, excl + total), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    return Prefix{excl, err};
}

// ------------------------------------------------------------------ staging

// Coalesced loads of the wave's 8 tiles (2048 floats from element e0, 16 B
// per lane per instruction), handed to the lane-per-block layout through LDS
// (rows padded to 36 dwords so that neither side has bank conflicts).
// Elements at or beyond n read as +0.
template <bool ALIGNED>
__device__ __forceinline__ void load_blocks_staged(const float *__restrict__ x, uint64_t n, uint64_t e0, uint32_t *st,
                                                   int lane, float (&v)[32])
{
    const bool full = e0 + 2048 <= n;
    if (ALIGNED) {
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int p = k * 64 + lane;  // 16-byte piece of the wave's 8 KiB
            const uint64_t e = e0 + 4ull * p;
            f4 f;
            if (full || e + 4 <= n) {
                f = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(x + e));
            } else {
                f.x = e + 0 < n ? x[e + 0] : 0.0f;
                f.y = e + 1 < n ? x[e + 1] : 0.0f;
                f.z = e + 2 < n ? x[e + 2] : 0.0f;
                f.w = e + 3 < n ? x[e + 3] : 0.0f;
            }
            *reinterpret_cast<f4 *>(st + (p >> 3) * kStageRowDwords + (p & 7) * 4) = f;
        }
    } else {
#pragma unroll 8
        for (int k = 0; k < 32; k++) {
            const int p = k * 64 + lane;
            const uint64_t e = e0 + p;
            const float f = (full || e < n) ? x[e] : 0.0f;
            st[(p >> 5) * kStageRowDwords + (p & 31)] = __float_as_uint(f);
        }
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const f4 f = *reinterpret_cast<const f4 *>(st + lane * kStageRowDwords + k * 4);
        v[4 * k + 0] = f.x;
        v[4 * k + 1] = f.y;
        v[4 * k + 2] = f.z;
        v[4 * k + 3] = f.w;
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// ------------------------------------------------------------------ stats

__device__ __forceinline__ void stats_combine(float &mn, float &mx, float &ma, uint32_t &nf, const StatsPartial &p)
{
    mn = fminf(mn, p.xmin);
    mx = fmaxf(mx, p.xmax);
    ma = fmaxf(ma, p.maxabs);
    nf |= p.flags;
}

// block-wide reduction of (min, max, max|x|, non-finite); result in every thread
template <int THREADS>
__device__ StatsPartial stats_block_reduce(float mn, float mx, float ma, uint32_t nf)
{
    for (int m = 32; m >= 1; m >>= 1) {
        mn = fminf(mn, __shfl_xor(mn, m));
        mx = fmaxf(mx, __shfl_xor(mx, m));
        ma = fmaxf(ma, __shfl_xor(ma, m));
        nf |= __shfl_xor(nf, m);
    }
    __shared__ StatsPartial wsum[THREADS / 64];
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = StatsPartial{mn, mx, ma, nf};
    lds_barrier();
    StatsPartial p = wsum[0];
    for (int k = 1; k < THREADS / 64; k++) stats_combine(p.xmin, p.xmax, p.maxabs, p.flags, wsum[k]);
    return p;
}

// Running (min, max, max |x| bit pattern) of a thread.  The largest |x|
// pattern doubles as the finiteness test: it is >= 0x7F800000 exactly when
// an Inf or NaN was seen (min and max are then of no use).
struct RangeAcc {
    float mn = INFINITY, mx = -INFINITY;
    uint32_t ma = 0;
    __device__ __forceinline__ void take(float v)
    {
        mn = fminf(mn, v);
        mx = fmaxf(mx, v);
        ma = max(ma, __float_as_uint(v) & 0x7FFFFFFFu);
    }
    __device__ __forceinline__ void take4(const f4 &f)
    {
        mn = fminf(fminf(mn, f.x), fminf(fminf(f.y, f.z), f.w));
        mx = fmaxf(fmaxf(mx, f.x), fmaxf(fmaxf(f.y, f.z), f.w));
        const uint32_t m = 0x7FFFFFFFu;
        ma = max(max(ma, __float_as_uint(f.x) & m),
                 max(max(__float_as_uint(f.y) & m, __float_as_uint(f.z) & m), __float_as_uint(f.w) & m));
    }
    template <int THREADS = kStatsThreads>
    __device__ __forceinline__ StatsPartial reduce() const
    {
        const uint32_t nf = ma >= 0x7F800000u ? 1u : 0u;
        return stats_block_reduce<THREADS>(mn, mx, __uint_as_float(ma & 0x7FFFFFFFu), nf);
    }
};

// Elements from x to its first 16-byte boundary.
__device__ __forceinline__ uint32_t align_head(const void *x)
{
    return ((16u - ((uint32_t)(uintptr_t)x & 15u)) & 15u) >> 2;
}

// Value-range pass, part 1: one partial (min, max, max|x|, non-finite) per
// workgroup.  Bound by the read: in every round a workgroup takes one piece of
// kRangeUnroll x THREADS consecutive 16-byte vectors, so that its loads
// in flight lie side by side in memory, and one workgroup of 8 waves per CU is
// enough to fill HBM (512^3: 78 us, 6.9 TB/s; a grid of 4 workgroups per CU
// whose loads in flight lay a grid apart took 92 us, 5.8 TB/s) and leaves 256
// partials to fold.  The last, partial round goes to all threads one vector at
// a time, the elements before the first and after the last 16-byte boundary
// singly.  The loads are nontemporal at every size.  Without the hint a field of
// 2^23 to 2^25 elements stays in the memory-side cache for the compressor's
// read, but the lines it displaces cost as much again once a program compresses
// field after field: rotating over 805 MB of fields, us per compression with /
// without the hint, GRF 2^24 at REL 1e-2 43.3 / 43.3, at 1e-4 46.1 / 48.5, 25 M
// 54.5 / 53.5 and 58.0 / 61.9, 2^25 68.4 / 66.4 and 71.4 / 76.7, piecewise
// quadratic 25 M at 1e-4 56.0 / 55.7; one field again and again 54.1 / 55.0.
constexpr int kRangeUnroll = 4;
template <int THREADS>
__global__ __launch_bounds__(THREADS) void stats_partial_kernel(StatsArgs a)
{
    RangeAcc acc;
    const uint64_t tid = (uint64_t)blockIdx.x * THREADS + threadIdx.x;
    const uint64_t nthreads = (uint64_t)gridDim.x * THREADS;
    const uint64_t head = min((uint64_t)align_head(a.x), a.n);
    const uint64_t nvec = (a.n - head) / 4;
    const f4 *x4 = reinterpret_cast<const f4 *>(a.x + head);
    const uint64_t whole = nvec - nvec % (kRangeUnroll * nthreads);  // vectors of whole rounds
    for (uint64_t i = (uint64_t)blockIdx.x * THREADS * kRangeUnroll + threadIdx.x; i < whole;
         i += kRangeUnroll * nthreads) {
        f4 f[kRangeUnroll];
#pragma unroll
        for (int u = 0; u < kRangeUnroll; u++) f[u] = __builtin_nontemporal_load(x4 + i + u * THREADS);
#pragma unroll
        for (int u = 0; u < kRangeUnroll; u++) acc.take4(f[u]);
    }
    if (whole < nvec) {
        f4 f[kRangeUnroll];
#pragma unroll
        for (int u = 0; u < kRangeUnroll; u++) {
            const uint64_t i = whole + tid + u * nthreads;
            if (i < nvec) f[u] = __builtin_nontemporal_load(x4 + i);
        }
#pragma unroll
        for (int u = 0; u < kRangeUnroll; u++)
            if (whole + tid + u * nthreads < nvec) acc.take4(f[u]);
    }
    const uint64_t tail = head + 4 * nvec;  // at most 3 elements on either side
    if (tid < head) acc.take(a.x[tid]);
    if (tid < a.n - tail) acc.take(a.x[tail + tid]);
    const StatsPartial p = acc.reduce<THREADS>();
    if (threadIdx.x == 0) a.partials[blockIdx.x] = p;
}

// The range pass's partials folded by one workgroup.
template <int THREADS>
__device__ __forceinline__ fsz_stats fold_partials(const StatsPartial *parts, uint32_t nparts)
{
    float mn = INFINITY, mx = -INFINITY, ma = 0.0f;
    uint32_t nf = 0;
    for (uint32_t i = threadIdx.x; i < nparts; i += THREADS) stats_combine(mn, mx, ma, nf, parts[i]);
    const StatsPartial p = stats_block_reduce<THREADS>(mn, mx, ma, nf);
    return fsz_stats{p.xmin, p.xmax, p.maxabs, p.flags};
}

// Value-range pass, part 2: one workgroup folds the partials into *out.
__global__ __launch_bounds__(kStatsThreads) void stats_final_kernel(StatsArgs a, unsigned nparts)
{
    const fsz_stats s = fold_partials<kStatsThreads>(a.partials, nparts);
    if (threadIdx.x == 0) *a.out = s;
}

// ------------------------------------------------------------------ compress

// The accumulator goes first: max(max(acc, a), b) selects to one v_max3 per
// two new values, where max(acc, max(a, b)) costs a v_max and a v_max3.
__device__ __forceinline__ int max3i(int acc, int a, int b) { return max(max(acc, a), b); }
__device__ __forceinline__ int min3i(int acc, int a, int b) { return min(min(acc, a), b); }

// Quantization (Sec. IV-B, q = round(x / (2 eb)) read as rint(fl(x * inv))):
// for |t| < 2^22 the binary32 sum t + 1.5 * 2^23 rounds t to the nearest
// integer with ties to even and holds it in the low mantissa bits, so
// bits(fl(fl(x * inv) + 1.5 * 2^23)) = kQBias + rint(fl(x * inv)) exactly.
// The bias cancels in every Lorenzo difference; |q| <= 2^21 + 1 follows from
// the step tightening of the error-bound resolution.
constexpr float kQMagic = 12582912.0f;  // 1.5 * 2^23
constexpr int kQBias = 0x4B400000;       // bits of kQMagic

// Extrema of the LZ1 / LZ2 residual magnitudes of one block (Sec. IV-A,
// Eq. (2); Sec. IV-B) from biased quantized values B, which are replaced by
// the block's LZ1 residuals d[i] = q[i] - q[i-1] (0 in slots past the end of
// the field); the LZ2 residual is d[i] - d[i-1].  The predictor state
// (carry_b = biased q of the previous block's last element, carry_l1 = its
// LZ1 residual) crosses the block boundary; at a tile start q[-1] = q[-2] = 0,
// so there d[0] = q[0].  Block 0 of a tile (j == 0) leaves its first one
// (LZ1) or two (LZ2) residuals out: they are re-rated per variant.  Slots
// whose bit in vm is clear lie past the end of the field and carry residual 0.
template <bool FULL>
__device__ __forceinline__ void block_extrema(int (&B)[32], int carry_b, int carry_l1, int j, uint32_t vm,
                                              uint32_t &a1, uint32_t &a2, int &l2_1)
{
    auto live = [&](int i, int v) { return FULL ? v : (v & ((int)(vm << (31 - i)) >> 31)); };
    const int d0 = B[0] - carry_b, d1 = B[1] - B[0], d2 = B[2] - B[1];
    const int l1_0 = live(0, d0), l2_0 = live(0, d0 - carry_l1);
    const int l1_1 = live(1, d1), l2_1v = live(1, d1 - d0);
    const int l1_2 = live(2, d2), l2_2 = live(2, d2 - d1);
    l2_1 = l2_1v;
    // neutral substitutes for the excluded leading residuals of block 0
    const int e10 = j ? l1_0 : l1_1;
    const int e20 = j ? l2_0 : l2_2;
    const int e21 = j ? l2_1v : l2_2;
    int mx1 = max3i(e10, l1_1, l1_2), mn1 = min3i(e10, l1_1, l1_2);
    int mx2 = max3i(e20, e21, l2_2), mn2 = min3i(e20, e21, l2_2);
    int pl = d2, pb = B[2];
    B[0] = l1_0;
    B[1] = l1_1;
    B[2] = l1_2;
#pragma unroll
    for (int i = 3; i < 31; i += 2) {
        const int ba = B[i], bb = B[i + 1];
        const int da = ba - pb;
        const int db = bb - ba;
        const int l1a = live(i, da), l2a = live(i, da - pl);
        const int l1b = live(i + 1, db), l2b = live(i + 1, db - da);
        pl = db;
        pb = bb;
        B[i] = l1a;
        B[i + 1] = l1b;
        mx1 = max3i(mx1, l1a, l1b);
        mn1 = min3i(mn1, l1a, l1b);
        mx2 = max3i(mx2, l2a, l2b);
        mn2 = min3i(mn2, l2a, l2b);
    }
    const int d31 = B[31] - pb;
    const int l1z = live(31, d31), l2z = live(31, d31 - pl);
    B[31] = l1z;
    mx1 = max(mx1, l1z);
    mn1 = min(mn1, l1z);
    mx2 = max(mx2, l2z);
    mn2 = min(mn2, l2z);
    // max(|mx|, |mn|) = max(mx, -mn) for mx >= mn
    a1 = (uint32_t)max(mx1, -mn1);
    a2 = (uint32_t)max(mx2, -mn2);
}

// Residual codes of the selected variant, in place, from the LZ1 residuals d
// that block_extrema left: e[i] = d[i] - order2 * d[i-1] with d[-1] =
// carry_l1, and at a centred tile start (j == 0, cent) d[0] = q[0] less the
// tile mean (the later residuals are differences, so mu cancels there).
// code = (|e| << 1) | sign.  |d| <= 2^22 + 2 fits the 24-bit multiplier.
// Codes of slots past the end of the field are garbage; the encoder clears
// them in the transposed plane words.
// a * b + c with a and b taken as signed 24-bit integers (one VALU
// instruction; the compiler splits __mul24(a, b) + c into two)
__device__ __forceinline__ int mad_i24(int a, int b, int c)
{
    int r;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

__device__ __forceinline__ void block_codes(int (&D)[32], int carry_l1, int j, int order2, int cent, int mu)
{
    const int no2 = -order2;
    int pl = carry_l1;
    D[0] -= (j == 0 && cent) ? mu : 0;
#pragma unroll
    for (int i = 0; i < 32; i++) {
        const int d = D[i];
        const int e = mad_i24(pl, no2, d);
        pl = d;
        const uint32_t m = (uint32_t)max(e, -e);
        D[i] = (int)__builtin_amdgcn_alignbit(m, (uint32_t)e, 31);  // (|e| << 1) | (e >> 31)
    }
}

// Per-lane result of the rate pass of one chunk, kept until its encode.
struct ChunkState {
    uint64_t chunk;
    int first;  // the block restarts prediction (tile start; every block without cross-block state)
    int carry_l1, mu;  // LZ1 residual of the previous block (0 where prediction restarts), tile mean
    uint32_t vm, r, blk_off, tile_excl, wave_total;
    int order2, cent;
    uint32_t rbyte;  // the block's rate byte (Sec. III-A)
};

// All of it is double-buffered.  A pipeline's step may pass a single barrier (its
// last one has no rate pass), and one wave may be a step ahead of another, so a
// step never writes the slot that the step before it reads: step k uses slot
// k % 2 of base and ticket, and is separated from step k + 2 by the barrier of
// step k + 1.
template <int W>
struct CompressShared {
    uint32_t wave_total[2][W];
    unsigned long long base[2];
    unsigned long long ticket[2];
};

// Rate pass of one chunk (8 tiles per wave), Sec. III-A steps 1-3:
//   1 quantize + cross-block LZ1/LZ2 residuals
//   2 four-way evaluation (Eq. (3)-(4)): blocks 1..7 have one rate per order;
//     block 0 is re-rated per variant from q0, q1 - 2 q0 and mu
//   3 adaptive select (strict minimum in the order LZ1, LZ2, LZ1c, LZ2c),
//     rate header; the chunk's byte count is published for the lookback.
// On return x holds the blocks' LZ1 residuals (block_extrema).
// The rate byte is left in cs.rbyte for the caller to store; wave 1 publishes the
// aggregate (wave 0's memory queue is the one a lookback may wait on).
// FEAT: honour a.features (the ablation's switches, Sec. VI-B): without the
// cross-block state every block restarts prediction and is re-rated per
// variant like block 0; switched-off variants are never selected.
template <int W, bool FEAT = false>
__device__ __forceinline__ ChunkState compress_rates(const CompressArgs &a, const Resolved &R, uint64_t chunk,
                                                     int (&x)[32], int slot, CompressShared<W> &sh)
{
    const int tid = threadIdx.x;
    const int w = tid >> 6;
    const int lane = tid & 63;
    const int j = lane & 7;
    const uint64_t tile0 = chunk * (kTilesPerWave * W) + (uint64_t)w * kTilesPerWave;
    const uint64_t tile = tile0 + (lane >> 3);
    const bool tile_ok = tile < a.ntiles;
    const uint64_t eblk = tile * kTile + (uint64_t)j * kBlock;
    const int cnt = eblk >= a.n ? 0 : (a.n - eblk >= kBlock ? kBlock : (int)(a.n - eblk));
    const bool full = (tile0 + kTilesPerWave) * kTile <= a.n;  // wave-uniform
    ChunkState cs;
    cs.chunk = chunk;
    cs.vm = cnt >= 32 ? 0xFFFFFFFFu : ((1u << cnt) - 1u);  // valid slots of the block

    // ---- tile mean: index-order pairwise binary32 tree over the 256 slots
    float s16[16];
#pragma unroll
    for (int i = 0; i < 16; i++) s16[i] = __int_as_float(x[2 * i]) + __int_as_float(x[2 * i + 1]);
#pragma unroll
    for (int i = 0; i < 8; i++) s16[i] = s16[2 * i] + s16[2 * i + 1];
#pragma unroll
    for (int i = 0; i < 4; i++) s16[i] = s16[2 * i] + s16[2 * i + 1];
#pragma unroll
    for (int i = 0; i < 2; i++) s16[i] = s16[2 * i] + s16[2 * i + 1];
    float ts = s16[0] + s16[1];
    ts = ts + dppf<kQuadXor1>(ts);       // blocks (0,1) (2,3) ...
    ts = ts + dppf<kQuadXor2>(ts);       // (0-1, 2-3) ...
    ts = ts + dppf<kRowHalfMirror>(ts);  // (0-3, 4-7)
    const float mean_q = (ts * 0x1p-8f) * R.inv;
    const bool centre_ok = __builtin_isfinite(mean_q);
    const int mu = centre_ok ? (int)__builtin_rintf(mean_q) : 0;
    cs.mu = mu;

    // ---- quantize, biased: x[i] = kQBias + rint(x * inv)
#pragma unroll
    for (int i = 0; i < 32; i++) x[i] = __float_as_int(__int_as_float(x[i]) * R.inv + kQMagic);

    // ---- cross-block state from block j-1 of the same tile (none where the
    // prediction restarts)
    const int t0 = dpp<kRowShr1>(x[31]);
    const int t1 = dpp<kRowShr1>(x[31] - x[30]);
    const bool first = FEAT ? (j == 0 || !(a.features & FSZ_FEAT_CROSS_BLOCK)) : j == 0;
    const int jr = first ? 0 : 1;  // 0: the leading residuals are re-rated per variant
    cs.first = first;
    const int carry_b = first ? kQBias : t0;
    cs.carry_l1 = first ? 0 : t1;

    uint32_t a1, a2;
    int l2_1;
    if (full)
        block_extrema<true>(x, carry_b, cs.carry_l1, jr, cs.vm, a1, a2, l2_1);
    else
        block_extrema<false>(x, carry_b, cs.carry_l1, jr, cs.vm, a1, a2, l2_1);
    const uint32_t r1 = bitlen(a1), r2 = bitlen(a2);
    uint32_t Z;
    if (FEAT) {
        // every restarting block is rated per variant, the others have one
        // rate per order; tile costs by 8-lane sums (same in all 8 lanes)
        const int q0 = x[0];  // d[0] = q[0] at a tile start
        const int d1 = cnt >= 2 ? l2_1 : 0;  // q1 - 2 q0
        const int c0 = q0 - mu;
        const int c1 = cnt >= 2 ? l2_1 + mu : 0;
        uint32_t ra = r1, rb = r2, rc = r1, rd = r2;
        if (first) {
            ra = bitlen(max(uabs(q0), a1));
            rb = bitlen(max(max(uabs(q0), uabs(d1)), a2));
            rc = bitlen(max(uabs(c0), a1));
            rd = bitlen(max(max(uabs(c0), uabs(c1)), a2));
        }
        if (cnt == 0) ra = rb = rc = rd = 0;  // blocks past the end of the field do not exist
        const uint32_t Ca = (uint32_t)group_sum((int)block_bytes(ra));
        const uint32_t Cb = (uint32_t)group_sum((int)block_bytes(rb));
        const uint32_t Cc = (uint32_t)group_sum((int)block_bytes(rc)) + 4;
        const uint32_t Cd = (uint32_t)group_sum((int)block_bytes(rd)) + 4;
        const bool lz2 = (a.features & FSZ_FEAT_LZ2) != 0;
        const bool cen = centre_ok && (a.features & FSZ_FEAT_CENTERING) != 0;
        int best = 0;
        uint32_t C = Ca, r = ra;
        if (lz2 && Cb < C) {
            best = 1;
            C = Cb;
            r = rb;
        }
        if (cen && Cc < C) {
            best = 2;
            C = Cc;
            r = rc;
        }
        if (cen && lz2 && Cd < C) {
            best = 3;
            C = Cd;
            r = rd;
        }
        if (!tile_ok) {
            best = 0;
            C = 0;
            r = 0;
        }
        cs.order2 = best & 1;
        cs.cent = best >> 1;
        Z = C;
        cs.r = r;
        cs.rbyte = j == 0 ? (r | (uint32_t)cs.order2 << 7 | (uint32_t)cs.cent << 6) : r;
    } else {
    const int T1 = group_sum(j ? (int)block_bytes(r1) : 0);
    const int T2 = group_sum(j ? (int)block_bytes(r2) : 0);

    // ---- four-way evaluation of block 0 and the selection (valid in lane j == 0)
    int dec;
    {
        const int q0 = x[0];  // d[0] = q[0] at a tile start
        const int d1 = cnt >= 2 ? l2_1 : 0;  // q1 - 2 q0
        const int c0 = q0 - mu;
        const int c1 = cnt >= 2 ? l2_1 + mu : 0;
        const uint32_t ra = bitlen(max(uabs(q0), a1));
        const uint32_t rb = bitlen(max(max(uabs(q0), uabs(d1)), a2));
        const uint32_t rc = bitlen(max(uabs(c0), a1));
        const uint32_t rd = bitlen(max(max(uabs(c0), uabs(c1)), a2));
        int best = 0;
        uint32_t C = block_bytes(ra) + T1, r0 = ra;
        const uint32_t Cb = block_bytes(rb) + T2;
        if (Cb < C) {
            best = 1;
            C = Cb;
            r0 = rb;
        }
        if (centre_ok) {
            const uint32_t Cc = block_bytes(rc) + T1 + 4;
            const uint32_t Cd = block_bytes(rd) + T2 + 4;
            if (Cc < C) {
                best = 2;
                C = Cc;
                r0 = rc;
            }
            if (Cd < C) {
                best = 3;
                C = Cd;
                r0 = rd;
            }
        }
        dec = (int)((C << 8) | ((uint32_t)(best & 1) << 7) | ((uint32_t)(best >> 1) << 6) | r0);
        if (!tile_ok) dec = 0;
    }
    dec = group_head(dec);
    cs.order2 = (dec >> 7) & 1;
    cs.cent = (dec >> 6) & 1;
    Z = (uint32_t)dec >> 8;
    cs.r = j == 0 ? (uint32_t)(dec & 31) : (cs.order2 ? r2 : r1);
    cs.rbyte = j == 0 ? (uint32_t)(dec & 0xFF) : cs.r;
    }
    const uint32_t S = block_bytes(cs.r);

    // ---- offsets inside the wave / chunk, aggregate for the lookback
    const int incl = wave_incl_scan(j == 0 ? (int)Z : 0);
    cs.tile_excl = (uint32_t)incl - Z;
    cs.wave_total = (uint32_t)__builtin_amdgcn_readlane(incl, 63);
    cs.blk_off = cs.tile_excl + group_excl_scan(S, j) + 4u * cs.cent;
    if (lane == 0) sh.wave_total[slot][w] = cs.wave_total;
    lds_barrier();
    if (tid == 64) {
        uint32_t chunk_total = 0;
#pragma unroll
        for (int k = 0; k < W; k++) chunk_total += sh.wave_total[slot][k];
        publish_aggregate(a.flags, chunk, a.flag_epoch, chunk_total, false);
    }
    return cs;
}

// Run by the thread that learns the last chunk's prefix: the stream header,
// the rate header's zero padding and the call's result.
__device__ __forceinline__ void finish_stream(const CompressArgs &a, const Resolved &R, const Prefix &pre,
                                              uint32_t chunk_total)
{
    const uint64_t total = a.data0 + pre.excl + chunk_total;
    uint32_t status = pre.err ? (uint32_t)FSZ_ERR_DEVICE : (uint32_t)FSZ_OK;
    if (status == FSZ_OK && total > a.capacity) status = FSZ_ERR_CAPACITY;
    if (status == FSZ_OK) {
        uint32_t *h = reinterpret_cast<uint32_t *>(a.out);
        h[0] = 0x315A5346u;  // "FSZ1"
        // bit 1: independent blocks; bits 2-4: tile configuration (0 = B 32, T 8)
        const uint32_t hflags = R.flags | ((a.features & FSZ_FEAT_CROSS_BLOCK) ? 0u : 2u) | a.cfg_flags;
        h[1] = 1u | ((uint32_t)a.mode << 16) | (hflags << 24);
        h[2] = (uint32_t)a.n;
        h[3] = (uint32_t)(a.n >> 32);
        h[4] = __float_as_uint(R.E);
        h[5] = __float_as_uint((float)a.value);
        h[6] = (uint32_t)total;
        h[7] = (uint32_t)(total >> 32);
        for (uint64_t k = kHeaderBytes + a.nblocks; k < a.data0; k++) a.out[k] = 0;
    }
    write_final(a.final, total, status, a.epoch);
}

// Thread 0 takes the next ticket and broadcasts it.  Consecutive calls use
// alternating slots, so a slot is rewritten only after a barrier that every
// reader of its previous value has passed.
template <typename Shared>
__device__ __forceinline__ uint64_t next_ticket(unsigned long long *ticket, uint64_t takes, Shared &sh, int &slot)
{
    if (threadIdx.x == 0) sh.ticket[slot] = take_ticket(ticket, takes);
    lds_barrier();
    const uint64_t t = uniform((uint64_t)sh.ticket[slot]);
    slot ^= 1;
    return t;
}

// ------------------------------------------------------------------ naive five-read baseline

// The comparison point of Sec. V-C (Fig. 6): the four variants evaluated in
// four separate passes over the input, each writing per-tile costs and block
// rates, then an encode pass that reads the input a fifth time.  It produces
// the same stream as the single-pass kernels; only the reads differ.

// Evaluation pass of variant v (bit 0: second order, bit 1: centred) over a
// chunk of kTilesPerChunk tiles per workgroup.
template <bool ALIGNED>
__global__ __launch_bounds__(kThreads) void naive_eval_kernel(CompressArgs a, NaiveTables t, int v)
{
    __shared__ __attribute__((aligned(16))) uint32_t stage[kWaves * kStageWaveDwords];
    const int tid = threadIdx.x;
    const int w = tid >> 6;
    const int lane = tid & 63;
    const int j = lane & 7;
    const Resolved R = resolve_bound(*a.stats, a.mode, a.value, a.n);
    if (R.status != FSZ_OK) return;  // the encode pass reports the status
    const uint64_t tile0 = (uint64_t)blockIdx.x * kTilesPerChunk + (uint64_t)w * kTilesPerWave;
    if (tile0 >= a.ntiles) return;  // wave-uniform; the kernel has no workgroup barrier
    float f[32];
    load_blocks_staged<ALIGNED>(a.x, a.n, tile0 * kTile, stage + w * kStageWaveDwords, lane, f);
    const uint64_t tile = tile0 + (lane >> 3);
    const bool tile_ok = tile < a.ntiles;
    const uint64_t eblk = tile * kTile + (uint64_t)j * kBlock;
    const int cnt = eblk >= a.n ? 0 : (a.n - eblk >= kBlock ? kBlock : (int)(a.n - eblk));
    const uint32_t vm = cnt >= 32 ? 0xFFFFFFFFu : ((1u << cnt) - 1u);
    const bool full = (tile0 + kTilesPerWave) * kTile <= a.n;
    const int order2 = v & 1, cen = v >> 1;

    int mu = 0;
    bool centre_ok = true;
    if (cen) {  // tile mean, as in the single pass
        float s16[16];
#pragma unroll
        for (int i = 0; i < 16; i++) s16[i] = f[2 * i] + f[2 * i + 1];
#pragma unroll
        for (int i = 0; i < 8; i++) s16[i] = s16[2 * i] + s16[2 * i + 1];
#pragma unroll
        for (int i = 0; i < 4; i++) s16[i] = s16[2 * i] + s16[2 * i + 1];
#pragma unroll
        for (int i = 0; i < 2; i++) s16[i] = s16[2 * i] + s16[2 * i + 1];
        float ts = s16[0] + s16[1];
        ts = ts + dppf<kQuadXor1>(ts);
        ts = ts + dppf<kQuadXor2>(ts);
        ts = ts + dppf<kRowHalfMirror>(ts);
        const float mean_q = (ts * 0x1p-8f) * R.inv;
        centre_ok = __builtin_isfinite(mean_q);
        mu = centre_ok ? (int)__builtin_rintf(mean_q) : 0;
    }
    int x[32];
#pragma unroll
    for (int i = 0; i < 32; i++) x[i] = __float_as_int(f[i] * R.inv + kQMagic);
    const int t0 = dpp<kRowShr1>(x[31]);
    const int t1 = dpp<kRowShr1>(x[31] - x[30]);
    const int carry_b = j ? t0 : kQBias;
    const int carry_l1 = j ? t1 : 0;
    uint32_t a1, a2;
    int l2_1;
    if (full)
        block_extrema<true>(x, carry_b, carry_l1, j, vm, a1, a2, l2_1);
    else
        block_extrema<false>(x, carry_b, carry_l1, j, vm, a1, a2, l2_1);
    uint32_t r = bitlen(order2 ? a2 : a1);
    if (j == 0) {  // block 0: the variant's own first residuals
        const int q0 = x[0];  // d[0] = q[0] at a tile start
        const int f0 = cen ? q0 - mu : q0;
        const int d1 = cnt >= 2 ? l2_1 : 0;
        const int f1 = cnt >= 2 ? (cen ? l2_1 + mu : d1) : 0;
        r = order2 ? bitlen(max(max(uabs(f0), uabs(f1)), a2)) : bitlen(max(uabs(f0), a1));
    }
    const uint32_t C = (uint32_t)group_sum((int)block_bytes(r)) + (cen ? 4u : 0u);
    if (tile_ok) {
        t.rates[((uint64_t)v * a.ntiles + tile) * kBlocksPerTile + j] = (uint8_t)r;
        if (j == 0) {
            t.cost[(uint64_t)v * a.ntiles + tile] = C;
            if (cen) {
                t.mu[tile] = mu;
                t.centre_ok[tile] = centre_ok ? 1 : 0;
            }
        }
    }
}

// Selection and bookkeeping of the encode pass: the rate pass of the single
// pass with the evaluation replaced by reads of the tables (same choice,
// same tie order).  On return x holds the blocks' LZ1 residuals.
__device__ __forceinline__ ChunkState naive_select(const CompressArgs &a, const Resolved &R, const NaiveTables &t,
                                                   uint64_t chunk, int (&x)[32], CompressShared<kWaves> &sh)
{
    const int tid = threadIdx.x;
    const int w = tid >> 6;
    const int lane = tid & 63;
    const int j = lane & 7;
    const uint64_t tile0 = chunk * kTilesPerChunk + (uint64_t)w * kTilesPerWave;
    const uint64_t tile = tile0 + (lane >> 3);
    const bool tile_ok = tile < a.ntiles;
    const uint64_t eblk = tile * kTile + (uint64_t)j * kBlock;
    const int cnt = eblk >= a.n ? 0 : (a.n - eblk >= kBlock ? kBlock : (int)(a.n - eblk));
    ChunkState cs;
    cs.chunk = chunk;
    cs.vm = cnt >= 32 ? 0xFFFFFFFFu : ((1u << cnt) - 1u);
#pragma unroll
    for (int i = 0; i < 32; i++) x[i] = __float_as_int(__int_as_float(x[i]) * R.inv + kQMagic);
    const int t0 = dpp<kRowShr1>(x[31]);
    const int t1 = dpp<kRowShr1>(x[31] - x[30]);
    cs.first = j == 0;
    cs.carry_l1 = j ? t1 : 0;
    {  // LZ1 residuals in place, as the encoder takes them
        int pb = j ? t0 : kQBias;
#pragma unroll
        for (int i = 0; i < 32; i++) {
            const int b = x[i];
            x[i] = b - pb;
            pb = b;
        }
    }

    int best = 0;
    uint32_t Z = 0, r = 0;
    cs.mu = 0;
    if (tile_ok) {
        const uint32_t Ca = t.cost[tile], Cb = t.cost[a.ntiles + tile];
        const uint32_t Cc = t.cost[2 * a.ntiles + tile], Cd = t.cost[3 * a.ntiles + tile];
        const bool centre_ok = t.centre_ok[tile] != 0;
        uint32_t C = Ca;
        if (Cb < C) {
            best = 1;
            C = Cb;
        }
        if (centre_ok) {
            if (Cc < C) {
                best = 2;
                C = Cc;
            }
            if (Cd < C) {
                best = 3;
                C = Cd;
            }
        }
        Z = C;
        r = t.rates[((uint64_t)best * a.ntiles + tile) * kBlocksPerTile + j];
        if (best >> 1) cs.mu = t.mu[tile];
    }
    cs.order2 = best & 1;
    cs.cent = best >> 1;
    cs.r = r;
    cs.rbyte = j == 0 ? (r | (uint32_t)cs.order2 << 7 | (uint32_t)cs.cent << 6) : r;
    if (cnt > 0) ((g_u8 *)a.out)[kHeaderBytes + tile * kBlocksPerTile + j] = (uint8_t)cs.rbyte;
    const uint32_t S = block_bytes(cs.r);
    const int incl = wave_incl_scan(j == 0 ? (int)Z : 0);
    cs.tile_excl = (uint32_t)incl - Z;
    cs.wave_total = (uint32_t)__builtin_amdgcn_readlane(incl, 63);
    cs.blk_off = cs.tile_excl + group_excl_scan(S, j) + 4u * cs.cent;
    if (lane == 0) sh.wave_total[0][w] = cs.wave_total;
    lds_barrier();
    if (tid == 0) {
        uint32_t chunk_total = 0;
#pragma unroll
        for (int k = 0; k < kWaves; k++) chunk_total += sh.wave_total[0][k];
        publish_aggregate(a.flags, chunk, a.flag_epoch, chunk_total, false);
    }
    return cs;
}

// Steps 4-5 of one chunk whose rate pass is done: wait for the chunk's output
// offset (decoupled lookback, Sec. IV-D), then the sign / bit-plane encoding
// (Sec. IV-C) through the wave's LDS staging area.  B holds the LZ1 residuals.
__device__ __forceinline__ void naive_encode(const CompressArgs &a, const Resolved &R, const ChunkState &cs,
                                             int (&B)[32], CompressShared<kWaves> &sh, uint32_t *st)
{
    const int tid = threadIdx.x;
    const int w = tid >> 6;
    const int lane = tid & 63;
    const int j = lane & 7;
    uint32_t chunk_total = 0, wave_base = 0;
#pragma unroll
    for (int k = 0; k < kWaves; k++) {
        if (k < w) wave_base += sh.wave_total[0][k];
        chunk_total += sh.wave_total[0][k];
    }
    if (w == 0) {
        const Prefix pre = lookback_wait(a.flags, cs.chunk, a.flag_epoch, chunk_total, false);
        if (lane == 0) {
            sh.base[0] = pre.excl;
            if (cs.chunk == a.nchunks - 1) finish_stream(a, R, pre, chunk_total);
        }
    }
    lds_barrier();
    const uint64_t base = sh.base[0];
    const uint64_t tile0 = cs.chunk * kTilesPerChunk + (uint64_t)w * kTilesPerWave;
    if (a.data0 + base + chunk_total > a.capacity || tile0 >= a.ntiles) return;

    uint8_t *wave_out = a.out + a.data0 + base + wave_base;
    if (cs.vm != 0 && j == 0 && cs.cent) st[cs.tile_excl >> 2] = (uint32_t)cs.mu;
    block_codes(B, cs.carry_l1, j, cs.order2, cs.cent, cs.mu);
    // valid slots in stored bit order (element i at bit i ^ 7)
    const uint32_t keep = __builtin_bswap32(__builtin_bitreverse32(cs.vm));
    const uint32_t nwords = cs.r ? cs.r + 1 : 0;  // sign word + r planes
    uint32_t *words = st + (cs.blk_off >> 2);
    for (uint32_t g = 0; __ballot(8 * g < nwords) != 0; g++) {
        uint32_t Rg[8];
#pragma unroll
        for (int rho = 0; rho < 8; rho++)
            Rg[rho] = pack_byte_g((uint32_t)B[7 - rho], (uint32_t)B[15 - rho], (uint32_t)B[23 - rho],
                                  (uint32_t)B[31 - rho], g);
        transpose8(Rg);
#pragma unroll
        for (int p = 0; p < 8; p++)
            if (8 * g + p < nwords) words[8 * g + p] = Rg[p] & keep;
    }
    // coalesced copy of the wave's contiguous output
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    wave_store_staged(reinterpret_cast<uint32_t *>(wave_out), st, cs.wave_total >> 2, lane);
}

// Encode pass: one chunk per workgroup from the ticket counter (the fifth
// read of the input), the tables' choice, lookback, the single pass's encoder.
template <bool ALIGNED>
__global__ __launch_bounds__(kThreads) void naive_encode_kernel(CompressArgs a, NaiveTables t)
{
    __shared__ CompressShared<kWaves> sh;
    __shared__ __attribute__((aligned(16))) uint32_t stage[kWaves * kStageWaveDwords];
    const int tid = threadIdx.x;
    const int w = tid >> 6;
    const int lane = tid & 63;
    uint32_t *st = stage + w * kStageWaveDwords;
    int tslot = 0;
    const uint64_t chunk = next_ticket(a.ticket, a.nchunks, sh, tslot);
    if (chunk >= a.nchunks) return;
    const Resolved R = resolve_bound(*a.stats, a.mode, a.value, a.n);
    if (R.status != FSZ_OK) {
        if (tid == 0 && chunk == a.nchunks - 1) write_final(a.final, 0, R.status, a.epoch);
        return;
    }
    const uint64_t tile0 = chunk * kTilesPerChunk + (uint64_t)w * kTilesPerWave;
    int x[32];
    {
        float f[32];
        if (tile0 < a.ntiles) {
            load_blocks_staged<ALIGNED>(a.x, a.n, tile0 * kTile, st, lane, f);
        } else {
#pragma unroll
            for (int i = 0; i < 32; i++) f[i] = 0.0f;
        }
#pragma unroll
        for (int i = 0; i < 32; i++) x[i] = __float_as_int(f[i]);
    }
    const ChunkState cs = naive_select(a, R, t, chunk, x, sh);
    naive_encode(a, R, cs, x, sh, st);
}

// ------------------------------------------------------------------ pipelined compress
//
// Persistent compression kernel: each
// workgroup keeps the next chunk's input in flight while it works on the
// current ones, through asynchronous global->LDS copies that hold no
// registers.  The LDS image of a wave's 8 tiles is unpadded and rotated:
// piece m (16 B) of block b sits at 16-byte slot 8b + ((m + b) & 7), so that
// both the copies (each instruction covers 1 KiB of contiguous input) and the
// lane-per-block reads (lane b reads piece m at step m) are free of bank
// conflicts.

constexpr int kCachePolicyNT = 2;  // cache-policy operand of the LDS copies: nontemporal
// A wave's LDS: 8 tiles of input, and its output at a 16-byte phase.  With
// statistics that cover the field the output is at most 64 x 96 bytes:
// |q| <= 2^21 + 1 bounds every LZ1 residual by 2^22 + 2, i.e. 23 bits and
// 4 + 4 x 23 bytes a block, LZ1 without centring may always be selected, and a
// tile takes its cheapest variant (a 64-element block: twice that for two
// lanes).  A caller's statistics may understate max |x|: a wave whose output is
// larger stores it without staging (store_oversize).  Room for 31 planes would
// leave 8 data waves per workgroup instead of 11.
constexpr int kPipeInDwords = 2048;
constexpr uint32_t kPipeOutBytes = 64 * 96;
constexpr int kPipeOutDwords = kPipeOutBytes / 4 + 4;
typedef __attribute__((address_space(3))) void lds_void;

typedef __attribute__((address_space(3))) uint32_t lds_u32;

template <int SIZE, int STEP, int... K>
__device__ __forceinline__ void lds_copies(const float *src, lds_u32 *dst, std::integer_sequence<int, K...>)
{
    static_assert(SIZE == 16 || SIZE == 4, "the builtin takes a literal size");
    if constexpr (SIZE == 16)
        (__builtin_amdgcn_global_load_lds((const void *)src, (lds_void *)dst, 16, K * STEP, kCachePolicyNT), ...);
    else
        (__builtin_amdgcn_global_load_lds((const void *)src, (lds_void *)dst, 4, K * STEP, kCachePolicyNT), ...);
}

// N copies of SIZE bytes per lane, each STEP bytes further in both memories: the
// instruction's offset, which counts for both, does the stepping.  (An address
// for every copy of the 4-byte form took registers that compress_ctrl_kernel<11>
// and the configuration compressors did not have: they spilled up to 12, and
// the reloads waited for everything in flight.  2^27 elements at offset 1, us per
// call before / after: 64/8 280 / 252, 64/16 294 / 256, default 234 / 233.)
template <int SIZE, int STEP, int N>
__device__ __forceinline__ void copy_to_lds(const float *src, lds_u32 *dst)
{
    if constexpr (N > 0) {
        constexpr int kPerBase = 4096 / STEP < N ? 4096 / STEP : N;  // a 13-bit signed offset
        lds_copies<SIZE, STEP>(src, dst, std::make_integer_sequence<int, kPerBase>{});
        copy_to_lds<SIZE, STEP, N - kPerBase>(src + kPerBase * STEP / 4, dst + kPerBase * STEP / 4);
    }
}

// Input of the wave's 8 tiles (element e0 onward, all in bounds) -> LDS.
// The copies carry the nontemporal hint: the input is read once, and without
// the hint it displaces cached data, among it the stream just written.
__device__ __forceinline__ void chunk_copy_async(const float *__restrict__ x, uint64_t e0, uint32_t *wbuf, int lane)
{
    const int m = ((lane & 7) - (lane >> 3)) & 7;
    copy_to_lds<16, 1024, 8>(x + e0 + 32 * (lane >> 3) + 4 * m, (lds_u32 *)wbuf);
}

// Same image from an input off the 16-byte grid, 4 bytes per lane: copy
// k brings blocks 2k and 2k + 1 (a lane's dword d = 64 k + lane is element d & 3
// of the piece at slot d >> 2).  Four times the instructions, and lines that
// straddle are fetched by two of them, but the pipeline hides most of it: 2^27
// elements at offset 1 233 us per call with the range pass, 216 aligned (a kernel
// with one chunk per workgroup: 673); 3.1 M 17.1 and 16.7 (32.1).
__device__ __forceinline__ void chunk_copy_async4(const float *__restrict__ x, uint64_t e0, uint32_t *wbuf, int lane)
{
    lds_u32 *dst = (lds_u32 *)wbuf;
    // the four rotations and their LDS addresses stay out of the pipeline loop's registers
    asm volatile("; %0 %1" : "+v"(lane), "+s"(dst));
    const int half = lane >> 5;
    const float *src = x + e0 + 32 * half + (lane & 3);
#pragma unroll
    for (int k = 0; k < 4; k++) {  // the rotation is the same every four copies
        const int m = (((lane >> 2) & 7) - 2 * k - half) & 7;
        copy_to_lds<4, 1024, 8>(src + 64 * k + 4 * m, dst + 64 * k);
    }
}

// Same image, loaded synchronously; elements at or beyond n read as +0.
__device__ __forceinline__ void chunk_copy_sync(const float *__restrict__ x, uint64_t n, uint64_t e0, uint32_t *wbuf,
                                                int lane)
{
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const int b = 8 * k + (lane >> 3);
        const int m = ((lane & 7) - b) & 7;
        const uint64_t e = e0 + 32 * b + 4 * m;
        f4 f;
        f.x = e + 0 < n ? x[e + 0] : 0.0f;
        f.y = e + 1 < n ? x[e + 1] : 0.0f;
        f.z = e + 2 < n ? x[e + 2] : 0.0f;
        f.w = e + 3 < n ? x[e + 3] : 0.0f;
        *reinterpret_cast<f4 *>(wbuf + 4 * (64 * k + lane)) = f;
    }
}

// Starts bringing the wave's part of `chunk` (W waves per chunk) into wbuf.
template <int W>
__device__ __forceinline__ void chunk_fetch(const CompressArgs &a, uint64_t chunk, uint32_t *wbuf, int w, int lane)
{
    const uint64_t e0 = (chunk * (kTilesPerWave * W) + (uint64_t)w * kTilesPerWave) * kTile;
    if (e0 + kTilesPerWave * kTile <= a.n) {
        if (((uintptr_t)a.x & 15u) == 0)  // the same for every chunk of a field
            chunk_copy_async(a.x, e0, wbuf, lane);
        else
            chunk_copy_async4(a.x, e0, wbuf, lane);
    } else
        chunk_copy_sync(a.x, a.n, e0, wbuf, lane);
}

// Lane-per-block read of the wave's image (block = lane).
__device__ __forceinline__ void chunk_read(const uint32_t *wbuf, int lane, int (&v)[32])
{
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's copies have landed
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int t = 0; t < 8; t++) {
        const int slot = 8 * lane + ((t + lane) & 7);
        const f4 f = *reinterpret_cast<const f4 *>(wbuf + 4 * slot);
        v[4 * t + 0] = __float_as_int(f.x);
        v[4 * t + 1] = __float_as_int(f.y);
        v[4 * t + 2] = __float_as_int(f.z);
        v[4 * t + 3] = __float_as_int(f.w);
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// The pipeline keeps every wait away from memory operations issued just
// before it: the vector memory operations of a wave complete in issue order,
// so a wait also waits for everything issued earlier.  Per step, wave 0 takes
// the next ticket and reads the lookback's first window before the rate
// pass and uses both after it; wave 1 publishes the aggregates; rate bytes go
// out with the chunk's data; the next chunk is read from LDS after staging
// but before the stores.  One LDS buffer per wave always receives the copy in
// flight, the other stages output.

// Lookback of cs.chunk by wave 0 (W0) from the pre-read window `probe`; the
// last chunk finishes the stream.  Wave 0 also resolves the ticket `traw` it
// took at the start of the step (resetting the counter if it was the last
// take) and broadcasts it.  Returns the chunk's exclusive prefix in every
// thread and the broadcast ticket in *next.
template <bool W0, int W>
__device__ __forceinline__ uint64_t pipe2_lookback(const CompressArgs &a, const Resolved &R, const ChunkState &cs,
                                                   int slot, CompressShared<W> &sh, const Probe &probe,
                                                   bool took, unsigned long long traw, uint64_t takes,
                                                   uint64_t *next)
{
    const int lane = threadIdx.x & 63;
    if (W0) {
        uint32_t chunk_total = 0;
#pragma unroll
        for (int k = 0; k < W; k++) chunk_total += sh.wave_total[slot][k];
        // the probe is consumed on every path (also for chunk 0), so the
        // next step's reads into its registers do not wait on stale loads
        consume_probe(probe);
        const Prefix pre = lookback_wait(a.flags, cs.chunk, a.flag_epoch, chunk_total, false, true, probe);
        const unsigned long long tk =
            took ? ((unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(traw >> 32)) << 32) |
                       (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)traw)
                 : a.nchunks;
        if (lane == 0) {
            if (took && tk == takes - 1)
                __hip_atomic_store(a.ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sh.base[slot] = pre.excl;
            sh.ticket[slot] = tk;
            if (cs.chunk == a.nchunks - 1) finish_stream(a, R, pre, chunk_total);
        }
    }
    lds_barrier();
    *next = uniform((uint64_t)sh.ticket[slot]);
    return uniform((uint64_t)sh.base[slot]);
}

// Residual codes and bit planes of one wave's blocks into its staging area
// (offsets relative to the wave's first byte).
template <bool FEAT>
__device__ __forceinline__ void pipe2_stage(const ChunkState &cs, int (&B)[32], uint32_t *st)
{
    const int j = __lane_id() & 7;
    if (cs.vm != 0 && j == 0 && cs.cent) st[cs.tile_excl >> 2] = (uint32_t)cs.mu;
    block_codes(B, cs.carry_l1, FEAT ? (cs.first ? 0 : 1) : j, cs.order2, cs.cent, cs.mu);
    const uint32_t keep = __builtin_bswap32(__builtin_bitreverse32(cs.vm));
    const uint32_t nwords = cs.r ? cs.r + 1 : 0;
    uint32_t *words = st + (cs.blk_off >> 2);
    for (uint32_t g = 0; __ballot(8 * g < nwords) != 0; g++) {
        uint32_t Rg[8];
#pragma unroll
        for (int rho = 0; rho < 8; rho++)
            Rg[rho] = pack_byte_g((uint32_t)B[7 - rho], (uint32_t)B[15 - rho], (uint32_t)B[23 - rho],
                                  (uint32_t)B[31 - rho], g);
        transpose8(Rg);
#pragma unroll
        for (int p = 0; p < 8; p++)
            if (8 * g + p < nwords) words[8 * g + p] = Rg[p] & keep;
    }
}

// The words of a wave whose output does not fit its staging area, straight to
// global memory (at wave_out), each lane's block from the input (seg0: the
// wave's first 32-element segment; LANES per tile, STRIDE dwords from one word of
// a block to the next).  Only wrong statistics bring such waves about, so this is
// written for few registers and little code beside the staging it stands in for:
// staging in two halves cost 512^3 at REL 1e-3 10% (218 -> 240 us), unrolled
// stores to global memory spilled 26 registers.
template <int LANES, int STRIDE, bool FEAT>
__device__ __forceinline__ void store_oversize(const CompressArgs &a, const Resolved &R, const ChunkState &cs,
                                               uint64_t seg0, uint32_t *wave_out)
{
    int lane = __lane_id();
    asm volatile("; %0" : "+v"(lane));  // keeps what follows from it out of the registers of the pipeline's loop
    // slots past the end of the field (the second half of a 64-element block may
    // lie there as a whole) read a valid one; their bits are cleared
    const bool live = cs.vm != 0;
    const g_f32 *x = (const g_f32 *)a.x + (live ? (seg0 + lane) * kBlock : 0);
    g_u32 *out = (g_u32 *)wave_out;
    const bool tile_start = lane % LANES == 0, first = FEAT ? cs.first != 0 : tile_start;
    if (live && tile_start && cs.cent) out[cs.tile_excl >> 2] = (uint32_t)cs.mu;
    if (cs.r == 0) return;
    auto quantized = [&](int i) { return __float_as_int(x[i] * R.inv + kQMagic); };
    const int before = quantized(first || !live ? 0 : -1);
#pragma unroll 1
    for (uint32_t b = 0; b <= cs.r; b++) {
        int pb = first ? kQBias : before, pl = cs.carry_l1;
        uint32_t word = 0;
#pragma unroll 1
        for (int i = 0; i < kBlock; i++) {
            const uint32_t valid = (cs.vm >> i) & 1u;
            const int q = quantized(valid ? i : 0);
            int d = q - pb;
            if (i == 0 && first && cs.cent) d -= cs.mu;
            const int e = mad_i24(pl, -cs.order2, d);  // as block_codes
            const uint64_t code = __builtin_amdgcn_alignbit((uint32_t)max(e, -e), (uint32_t)e, 31);
            word |= ((uint32_t)(code >> b) & valid) << (i ^ 7);
            pb = q;
            pl = d;
        }
        out[(cs.blk_off >> 2) + STRIDE * b] = word;
    }
}

// The tile geometry a compression pipeline runs: its rate pass (one
// workgroup barrier), its staging of the codes, whether a wave's first tile
// exists, and where a lane's rate byte goes.  TileB32T8 is the default format
// (blocks of 32 elements, tiles of 8 blocks); the tile-configuration sweep
// has its own.
struct TileB32T8 {
    static constexpr int kLanes = 8, kWordStride = 1;  // lanes per tile, dwords from one word of a block to the next
    template <int W, bool FEAT>
    static __device__ __forceinline__ ChunkState rates(const CompressArgs &a, const Resolved &R, uint64_t chunk,
                                                       int (&x)[32], int slot, CompressShared<W> &sh)
    {
        return compress_rates<W, FEAT>(a, R, chunk, x, slot, sh);
    }
    template <bool FEAT>
    static __device__ __forceinline__ void stage(const ChunkState &cs, int (&B)[32], uint32_t *st)
    {
        pipe2_stage<FEAT>(cs, B, st);
    }
    template <int W>
    static __device__ __forceinline__ bool wave_live(const CompressArgs &a, uint64_t chunk, int w)
    {
        return chunk * (kTilesPerWave * W) + (uint64_t)w * kTilesPerWave < a.ntiles;
    }
    template <int W>
    static __device__ __forceinline__ void store_rate(const CompressArgs &a, const ChunkState &cs, int w, int lane)
    {
        const uint64_t tile0 = cs.chunk * (kTilesPerWave * W) + (uint64_t)w * kTilesPerWave;
        if (cs.vm != 0)
            ((g_u8 *)a.out)[kHeaderBytes + (tile0 + (lane >> 3)) * kBlocksPerTile + (lane & 7)] = (uint8_t)cs.rbyte;
    }
};

// The wave totals of a chunk (slot of CompressShared): the chunk's bytes, and
// those before wave w's.  Read before the step's second barrier: a wave that is
// ahead writes the same slot in the rate pass of the next step, which only that
// barrier separates from this read.
template <int W>
__device__ __forceinline__ void chunk_totals(const CompressShared<W> &sh, int slot, int w, uint32_t &wave_base,
                                             uint32_t &chunk_total)
{
    wave_base = chunk_total = 0;
#pragma unroll
    for (int k = 0; k < W; k++) {
        if (k < w) wave_base += sh.wave_total[slot][k];
        chunk_total += sh.wave_total[slot][k];
    }
    wave_base = uniform(wave_base);
    chunk_total = uniform(chunk_total);
}

// One step with chunk A rate-passed (registers xa, wave totals in slot sa),
// chunk B read (registers yb) and chunk C being copied into qb: rate pass of
// B, lookback + staging of A, read C into xa, start the copy of the ticket
// taken in this step, store A.  Returns that ticket (nchunks if none).
// W0: the calling wave is wave 0, which takes the ticket and reads the
// lookback window at the start and uses both after the rate pass.
template <bool W0, int W, bool FEAT, class M = TileB32T8>
__device__ __forceinline__ uint64_t pipe2_step(const CompressArgs &a, const Resolved &R, uint64_t takes,
                                               const ChunkState &ca, int (&xa)[32], int sa, uint64_t B,
                                               int (&yb)[32], ChunkState &cb, uint64_t C, uint32_t *qb,
                                               uint32_t *pb, CompressShared<W> &sh, int w)
{
    const int lane = threadIdx.x & 63;
    const bool take = C < a.nchunks;
    unsigned long long traw = 0;
    Probe probe{};
    if (W0) {
        if (take && lane == 0) traw = atomicAdd(a.ticket, 1ull);
        probe = lookback_probe(a.flags, ca.chunk, a.flag_epoch);
    }
    if (B < a.nchunks) cb = M::template rates<W, FEAT>(a, R, B, yb, sa ^ 1, sh);
    uint32_t wave_base, chunk_total;
    chunk_totals<W>(sh, sa, w, wave_base, chunk_total);
    uint64_t D;
    const uint64_t base = pipe2_lookback<W0, W>(a, R, ca, sa, sh, probe, take, traw, takes, &D);

    const bool ok = a.data0 + base + chunk_total <= a.capacity && M::template wave_live<W>(a, ca.chunk, w);
    uint32_t *wave_out = reinterpret_cast<uint32_t *>(a.out + a.data0 + base + wave_base);
    uint32_t *ps = pb + (((uint32_t)(uintptr_t)wave_out >> 2) & 3u);  // staging at the output's 16-byte phase
    uint32_t staged = ok ? ca.wave_total : 0;  // bytes
    if (staged > kPipeOutBytes) {
        store_oversize<M::kLanes, M::kWordStride, FEAT>(a, R, ca, (ca.chunk * W + (uint64_t)w) * 64, wave_out);
        staged = 0;
    }
    if (staged) M::template stage<FEAT>(ca, xa, ps);
    if (C < a.nchunks) chunk_read(qb, lane, xa);
    if (D < a.nchunks) {
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the read of qb is done before it is overwritten
        chunk_fetch<W>(a, D, qb, w, lane);
    }
    M::template store_rate<W>(a, ca, w, lane);
    if (staged) {
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        wave_store_staged_phased(wave_out, ps, staged >> 2, lane);
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    return D;
}

// The start of a compressing workgroup: the first ticket A, the copy of its
// chunk under way, and the call's bound R, from the caller's stats or folded by
// every workgroup from the partials of the call's own range pass (at most one
// per thread; a launch of its own for that took 4.6 us on large fields and 2 us
// on small ones).  The partials' loads go out first, so neither the ticket's
// round trip nor the chunk's copy waits on them.  A field of one chunk needs no
// range pass (SELF, a.self_range): its workgroup takes the range from the copy in
// LDS.  False: no chunk is left, or
// the bound does not resolve (the tickets are then handed out without data
// work, and the last chunk's taker reports).
template <int THREADS, int W, bool SELF = false>
__device__ __forceinline__ bool pipe_start(const CompressArgs &a, CompressShared<W> &sh, uint32_t *qb, int w,
                                           Resolved &R, uint64_t &A, int &tslot)
{
    static_assert(THREADS >= kRangeMaxBlocks, "one partial per thread");
    const uint64_t N = a.nchunks;
    const uint64_t takes = N + gridDim.x;
    StatsPartial part{INFINITY, -INFINITY, 0.0f, 0u};
    if (a.partials && threadIdx.x < a.nparts) part = a.partials[threadIdx.x];
    tslot = 0;
    A = next_ticket(a.ticket, takes, sh, tslot);
    if (A >= N) return false;
    if (w < W) chunk_fetch<W>(a, A, qb, w, threadIdx.x & 63);
    fsz_stats s;
    if (SELF && a.self_range) {
        RangeAcc acc;
        if (w < W) {
            const int lane = threadIdx.x & 63;
            int v[32];
            chunk_read(qb, lane, v);
            const uint64_t e = (uint64_t)(w * 64 + lane) * kBlock;
            const int cnt = e >= a.n ? 0 : (a.n - e >= kBlock ? kBlock : (int)(a.n - e));
#pragma unroll
            for (int i = 0; i < 32; i++)
                if (i < cnt) acc.take(__int_as_float(v[i]));
        }
        const StatsPartial p = acc.template reduce<THREADS>();
        s = fsz_stats{p.xmin, p.xmax, p.maxabs, p.flags};
    } else if (a.partials) {
        const StatsPartial p = stats_block_reduce<THREADS>(part.xmin, part.xmax, part.maxabs, part.flags);
        s = fsz_stats{p.xmin, p.xmax, p.maxabs, p.flags};
    } else {
        s = *a.stats;
    }
    R = resolve_bound(s, a.mode, a.value, a.n);
    if (R.status == FSZ_OK) return true;
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the copy into LDS has landed
    for (uint64_t t = A; t < N; t = next_ticket(a.ticket, takes, sh, tslot))
        if (threadIdx.x == 0 && t == N - 1) write_final(a.final, 0, R.status, a.epoch);
    return false;
}

// The whole pipeline of one wave (W0: wave 0's role) from pipe_start on.
template <bool W0, int W, bool FEAT, class M = TileB32T8>
__device__ __forceinline__ void pipe2_run(const CompressArgs &a, const Resolved &R, CompressShared<W> &sh,
                                          uint32_t *qb, uint32_t *pb, int w, uint64_t A, int tslot)
{
    const int lane = threadIdx.x & 63;
    const uint64_t N = a.nchunks;
    const uint64_t takes = N + gridDim.x;
    uint64_t B = next_ticket(a.ticket, takes, sh, tslot);
    int x[32], y[32];
    chunk_read(qb, lane, x);
    if (B < N) {
        __builtin_amdgcn_s_waitcnt(0xC07F);
        chunk_fetch<W>(a, B, qb, w, lane);
    }
    ChunkState ca = M::template rates<W, FEAT>(a, R, A, x, 0, sh);
    ChunkState cb = ca;
    uint64_t C = N;
    if (B < N) {
        C = next_ticket(a.ticket, takes, sh, tslot);
        chunk_read(qb, lane, y);
        if (C < N) {
            __builtin_amdgcn_s_waitcnt(0xC07F);
            chunk_fetch<W>(a, C, qb, w, lane);
        }
    }
    // loop invariant: A rate-passed in x (slot 0), B read into y, C in flight
    for (;;) {
        const uint64_t D = pipe2_step<W0, W, FEAT, M>(a, R, takes, ca, x, 0, B, y, cb, C, qb, pb, sh, w);
        if (B >= N) return;
        const uint64_t E = pipe2_step<W0, W, FEAT, M>(a, R, takes, cb, y, 1, C, x, ca, D, qb, pb, sh, w);
        if (C >= N) return;
        B = D;
        C = E;
    }
}

// The control wave of compress_ctrl_kernel: wave 0's part of the pipeline
// without its data.  Per step it takes the ticket and walks the lookback of
// the chunk rate-passed in the previous step while the data waves run the
// next rate pass, so the offset is usually known when they reach the second
// barrier; its own memory queue holds only flag reads, so they are not
// queued behind copies and stores.  It passes every barrier the data waves
// pass (pipe2_run<false, WD>): the ticket broadcasts, the rate pass's, and
// the step's second one.
template <int WD>
__device__ __forceinline__ uint64_t ctrl_step(const CompressArgs &a, const Resolved &R, uint64_t takes,
                                              uint64_t A, int sa, uint64_t B, uint64_t C, CompressShared<WD> &sh)
{
    const uint64_t N = a.nchunks;
    const int lane = __lane_id();
    const bool take = C < N;
    unsigned long long traw = 0;
    if (take && lane == 0) traw = atomicAdd(a.ticket, 1ull);
    uint32_t chunk_total = 0;
#pragma unroll
    for (int k = 0; k < WD; k++) chunk_total += sh.wave_total[sa][k];  // A's, from the previous step
    const Prefix pre = lookback_wait(a.flags, A, a.flag_epoch, chunk_total, false);
    if (B < N) lds_barrier();  // the data waves' rate pass of B
    const unsigned long long tk =
        take ? ((unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(traw >> 32)) << 32) |
                   (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)traw)
             : N;
    if (lane == 0) {
        if (take && tk == takes - 1) __hip_atomic_store(a.ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh.base[sa] = pre.excl;
        sh.ticket[sa] = tk;
        if (A == N - 1) finish_stream(a, R, pre, chunk_total);
    }
    lds_barrier();  // the offset and the ticket go out
    return tk;
}

template <int WD>
__device__ __forceinline__ void ctrl_run(const CompressArgs &a, const Resolved &R, CompressShared<WD> &sh, uint64_t A,
                                         int tslot)
{
    const uint64_t N = a.nchunks;
    const uint64_t takes = N + gridDim.x;
    // first pick of its SIMD's issue slots: the wave shares a SIMD with two
    // data waves in their rate pass, and its short lookback bursts gate the
    // step's second barrier
    __builtin_amdgcn_s_setprio(3);
    uint64_t B = next_ticket(a.ticket, takes, sh, tslot);
    lds_barrier();  // the rate pass of A
    uint64_t C = N;
    if (B < N) C = next_ticket(a.ticket, takes, sh, tslot);
    for (int sa = 0;; sa ^= 1) {
        const uint64_t D = ctrl_step<WD>(a, R, takes, A, sa, B, C, sh);
        if (B >= N) return;
        A = B;
        B = C;
        C = D;
    }
}

// The pipelined compressor with WD data waves (8 tiles each per chunk) and
// one control wave (ctrl_run).  a.nchunks must count chunks of 8 WD tiles.
// One workgroup per CU; what bounds it are the data waves' latencies (its VALU
// is busy half of the time, HBM at 60%), so the more waves the better: 11 data
// waves and the control wave are three per SIMD, which 168 VGPRs allow, and
// fill 154 of the 160 KB of LDS.  512^3 GRF, REL 1e-2 / 1e-3 / 1e-4, with a
// range pass and fold of 97 us: 11 waves 228 / 236 / 247 us, 10 232 / 240 / 251,
// 9 239 / 246 / 258, 8 242 / 250 / 259 (at REL 1e-3 the kernel moves 663 MB in
// 140 us, 4.7 TB/s; a large copy reaches 5.0).  A field too small to give every workgroup two
// chunks takes 8 (launch_compress).
template <int WD>
__global__ __launch_bounds__((WD + 1) * 64) void compress_ctrl_kernel(CompressArgs a)
{
    __shared__ CompressShared<WD> sh;
    __shared__ __attribute__((aligned(16))) uint32_t inbuf[WD * kPipeInDwords];
    __shared__ __attribute__((aligned(16))) uint32_t stbuf[WD * kPipeOutDwords];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
    Resolved R;
    uint64_t A;
    int tslot;
    if (!pipe_start<(WD + 1) * 64, WD, WD * kWaveElems <= kSelfRangeMax>(a, sh, inbuf + w * kPipeInDwords, w, R, A, tslot)) return;
    if (w < WD)
        pipe2_run<false, WD, false>(a, R, sh, inbuf + w * kPipeInDwords, stbuf + w * kPipeOutDwords, w, A, tslot);
    else
        ctrl_run<WD>(a, R, sh, A, tslot);
}

// The wave-0 form, for the feature switches (a.features).  W waves per
// workgroup; a chunk is 8 tiles per wave.  a.nchunks must count chunks of that
// size.
template <int W>
__global__ __launch_bounds__(W * 64) void compress_pipe2_kernel(CompressArgs a)
{
    __shared__ CompressShared<W> sh;
    __shared__ __attribute__((aligned(16))) uint32_t inbuf[W * kPipeInDwords];
    __shared__ __attribute__((aligned(16))) uint32_t stbuf[W * kPipeOutDwords];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
    uint32_t *qb = inbuf + w * kPipeInDwords;
    uint32_t *pb = stbuf + w * kPipeOutDwords;

    Resolved R;
    uint64_t A;
    int tslot;
    if (!pipe_start<W * 64, W>(a, sh, qb, w, R, A, tslot)) return;
    if (w == 0)
        pipe2_run<true, W, true>(a, R, sh, qb, pb, w, A, tslot);
    else
        pipe2_run<false, W, true>(a, R, sh, qb, pb, w, A, tslot);
}

// ------------------------------------------------------------------ decompress

// Four rate bytes: sum of r + (r > 0) over them, added to acc (a block of rate
// r > 0 is one sign word and r planes long).
__device__ __forceinline__ uint32_t rate_units(uint32_t w, uint32_t acc)
{
    const uint32_t x = w & 0x1F1F1F1Fu;
    const uint32_t nz = ((x + 0x1F1F1F1Fu) >> 5) & 0x01010101u;
    return (uint32_t)__builtin_popcount(nz) + __builtin_amdgcn_sad_u8(x, 0u, acc);
}

// Per-lane state of one chunk between the size pass and the decode pass.
struct DecChunk {
    uint64_t chunk;
    uint64_t base;  // the chunk's data offset after data0 (decodes with the offsets pre-pass)
    uint32_t r, blk_off, tile_excl, wave_total;
    int order2, cent;
};

// How a decoder's workgroup learns its chunk's byte offset.
enum DecOffsets {
    kByGroups,    // group totals and in-group offsets from dec_groups_kernel, chunk after chunk
    kByGroupsOnce,  // the same for a workgroup's only chunk
    kByPrefix     // its own sum over the rate bytes before the chunk
};

// Slots rotate from chunk to chunk.  The persistent decoder with the offsets
// pre-pass passes one barrier per chunk, so a wave may be one chunk ahead of
// another and three slots are in use.
template <int W>
struct DecompressShared {
    uint32_t wave_total[3][W];
    unsigned long long wave_prefix[W];  // kByPrefix, kByGroupsOnce: the waves' shares of the sum, and
    uint32_t wave_bad[W];               // whether they saw a reserved rate-byte bit
    unsigned long long group_base[3];
    unsigned long long base;       // tile configurations
    unsigned long long ticket[2];  // (their lookback form: alternating broadcast slots)
};

// Running sum over the groups of the offsets pre-pass (dec_groups_kernel), kept
// by one wave: bytes of groups [0, next) and whether one of them holds a
// reserved rate-byte bit.
constexpr unsigned long long kGroupBad = 1ull << 63;
struct GroupCursor {
    uint64_t next = 0, sum = 0;
    bool bad = false;
};

// Moves the cursor up to group g; the whole wave runs it (64 groups per load).
__device__ __forceinline__ void groups_advance(const unsigned long long *groups, uint64_t g, GroupCursor &c)
{
    for (; c.next < g; c.next += 64) {
        const uint64_t k = c.next + __lane_id();
        const unsigned long long v = k < g ? groups[k] : 0ull;
        c.sum += wave_sum_u64(v & ~kGroupBad);
        c.bad = c.bad || __ballot(v >> 63) != 0;
    }
    c.next = g;
}

// Run by one whole wave that knows of every rate byte up to the last decoded
// tile: the call's outcome.  The stream is sound if none of them has a reserved
// bit and, for a whole field, the sizes add up to the header's total and the
// rate header's padding (at most 15 bytes, one lane each) is zero; for a range,
// if its data ends inside the stream.
template <bool RANGE>
__device__ __forceinline__ void finish_decode(const DecompressArgs &a, bool bad, uint64_t end, uint64_t total)
{
    if (RANGE) {
        bad = bad || a.data0 + end > total;
    } else {
        const uint64_t k = kHeaderBytes + a.nblocks + __lane_id();
        const bool pad = __lane_id() < 16 && k < a.data0;
        bad = bad || a.data0 + end != total || __ballot(a.cmp[pad ? k : 0] != 0 && pad) != 0;
    }
    if (__lane_id() == 0)
        write_final(a.final, total, bad ? (uint32_t)FSZ_ERR_CORRUPT : (uint32_t)FSZ_OK, a.epoch);
}

// Decompression steps 1-2 (Sec. III-A): rate bytes and tile metadata ->
// block and tile sizes, and the chunk's offset.
// RANGE: decode the tiles [a.tile_begin, a.tile_end) only (random access);
// otherwise the whole field (the range fields are not read).  Chunks count
// from the field's first tile, but from tile_begin with kByPrefix.
template <int W, bool RANGE, int OFF>
__device__ __forceinline__ uint64_t dec_chunk_tile0(const DecompressArgs &a, uint64_t chunk)
{
    return (RANGE && OFF == kByPrefix ? a.tile_begin : 0) + chunk * (kTilesPerWave * W);
}

// The lane's rate byte of `chunk` (0 past the end of the field or the range).
template <int W, bool RANGE, int OFF>
__device__ __forceinline__ uint32_t dec_rate_byte(const DecompressArgs &a, uint64_t chunk)
{
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const uint64_t tile = dec_chunk_tile0<W, RANGE, OFF>(a, chunk) + (uint64_t)(tid >> 3);
    const bool tile_ok = tile < (RANGE ? a.tile_end : a.ntiles);
    const uint64_t gblock = tile * kBlocksPerTile + (lane & 7);
    const bool blk_ok = (RANGE ? tile_ok : true) && gblock < a.nblocks;
    return blk_ok ? ((const g_u8 *)a.cmp)[kHeaderBytes + gblock] : 0u;
}

// Bytes of the tiles before `tile0` that this thread's share of the rate
// header adds up to (16 bytes, i.e. two tiles, per load; all of them whole
// tiles), and whether a reserved bit is set in it.
template <int THREADS>
__device__ __forceinline__ uint32_t dec_prefix_share(const DecompressArgs &a, uint64_t tile0, uint32_t &bad)
{
    const g_u32 *p = (const g_u32 *)(a.cmp + kHeaderBytes);
    const uint32_t n16 = (uint32_t)(tile0 / 2);
    uint32_t units = 0, cents = 0;
    auto take = [&](uint32_t w, bool head) {
        bad |= w & (head ? 0xE0E0E020u : 0xE0E0E0E0u);
        units = rate_units(w, units);
        if (head) cents += (w >> 6) & 1u;
    };
    auto take4 = [&](const u32x4 &v) {
        take(v.x, true);
        take(v.y, false);
        take(v.z, true);
        take(v.w, false);
    };
    uint32_t i = threadIdx.x;
    for (; i + 3 * THREADS < n16; i += 4 * THREADS) {
        const u32x4 v0 = *(const g_u32x4_a4 *)(p + 4 * (uint64_t)i);
        const u32x4 v1 = *(const g_u32x4_a4 *)(p + 4 * (uint64_t)(i + THREADS));
        const u32x4 v2 = *(const g_u32x4_a4 *)(p + 4 * (uint64_t)(i + 2 * THREADS));
        const u32x4 v3 = *(const g_u32x4_a4 *)(p + 4 * (uint64_t)(i + 3 * THREADS));
        take4(v0);
        take4(v1);
        take4(v2);
        take4(v3);
    }
    for (; i < n16; i += THREADS) take4(u32x4(*(const g_u32x4_a4 *)(p + 4 * (uint64_t)i)));
    if ((tile0 & 1) && threadIdx.x == 0) {  // the odd tile
        take(p[4 * (uint64_t)n16], true);
        take(p[4 * (uint64_t)n16 + 1], false);
    }
    return 4u * units + 4u * cents;
}

// Bytes of the groups before the chunk's, this wave's share of them (all
// threads of the workgroup read at once), and whether one holds a reserved bit.
template <int THREADS>
__device__ __forceinline__ unsigned long long groups_share(const DecompressArgs &a, uint32_t g, bool &bad)
{
    unsigned long long v = 0, flags = 0;
    for (uint32_t k = threadIdx.x; k < g; k += THREADS) {
        const unsigned long long t = a.groups[k];
        v += t & ~kGroupBad;
        flags |= t;
    }
    bad = (flags & kGroupBad) != 0;
    // block sizes of up to 2^29 elements cannot add up to 2^32 bytes (at most
    // 132 per block and 4 per tile), and a 32-bit sum takes a sixth of the
    // instructions, which every chunk's workgroup pays
    if (a.n <= (1ull << 29)) return (uint32_t)__builtin_amdgcn_readlane(wave_incl_scan((int)(uint32_t)v), 63);
    return wave_sum_u64(v);
}

// rb: the lane's rate byte from dec_rate_byte (loaded ahead by the caller).
// kByGroups: the offsets pre-pass has summed the groups of chunks and placed
// every chunk inside its group; wave 0 brings its group cursor up to the
// chunk's group.  kByGroupsOnce: the group totals before the chunk's are read
// by all threads at once.  kByPrefix: every thread adds up its share of the rate bytes
// before the chunk.
template <int W, bool RANGE, int OFF>
__device__ __forceinline__ DecChunk dec_sizes(const DecompressArgs &a, uint64_t chunk, uint32_t rb, int slot,
                                              DecompressShared<W> &sh, GroupCursor &gc)
{
    const int tid = threadIdx.x;
    const int w = tid >> 6;
    const int lane = tid & 63;
    const int j = lane & 7;
    const uint64_t tile = dec_chunk_tile0<W, RANGE, OFF>(a, chunk) + (uint64_t)(tid >> 3);
    const bool tile_ok = tile < (RANGE ? a.tile_end : a.ntiles);
    const uint64_t gblock = tile * kBlocksPerTile + j;
    const bool blk_ok = (RANGE ? tile_ok : true) && gblock < a.nblocks;
    const bool bad = blk_ok && (j == 0 ? (rb & 0x20u) : (rb & 0xE0u)) != 0;
    const uint32_t head = (uint32_t)group_head((int)rb);
    DecChunk d;
    d.chunk = chunk;
    d.order2 = tile_ok ? (int)((head >> 7) & 1u) : 0;
    d.cent = tile_ok ? (int)((head >> 6) & 1u) : 0;
    d.r = rb & 31u;
    const uint32_t S = block_bytes(d.r);
    const uint32_t Z = (uint32_t)group_sum((int)S) + 4u * d.cent;
    const int incl = wave_incl_scan(j == 0 ? (int)Z : 0);
    d.tile_excl = (uint32_t)incl - Z;
    d.wave_total = (uint32_t)__builtin_amdgcn_readlane(incl, 63);
    d.blk_off = d.tile_excl + group_excl_scan(S, j) + 4u * d.cent;
    d.base = 0;
    if constexpr (OFF == kByGroups) {
        if (w == 0) {
            groups_advance(a.groups, chunk >> a.group_shift, gc);
            if (lane == 0) sh.group_base[slot] = gc.sum + a.offsets[chunk];
        }
        if (lane == 0) sh.wave_total[slot][w] = d.wave_total;
        lds_barrier();
        d.base = sh.group_base[slot];
    }
    if constexpr (OFF == kByPrefix || OFF == kByGroupsOnce) {
        bool seen;
        unsigned long long psum;
        if (OFF == kByPrefix) {
            uint32_t pbad = 0;
            const uint32_t share = dec_prefix_share<W * 64>(a, dec_chunk_tile0<W, RANGE, OFF>(a, chunk), pbad);
            psum = (uint32_t)__builtin_amdgcn_readlane(wave_incl_scan((int)share), 63);
            seen = bad || pbad != 0;
        } else {
            const uint32_t g = (uint32_t)(chunk >> a.group_shift);
            psum = groups_share<W * 64>(a, g, seen);
            d.base = a.offsets[chunk];
            gc.next = g;
        }
        const bool wave_bad = __ballot(seen) != 0;
        if (lane == 0) {
            sh.wave_prefix[w] = psum;
            sh.wave_total[slot][w] = d.wave_total;
            sh.wave_bad[w] = wave_bad ? 1u : 0u;
        }
        lds_barrier();
#pragma unroll
        for (int k = 0; k < W; k++) {
            d.base += sh.wave_prefix[k];
            gc.bad = gc.bad || sh.wave_bad[k] != 0;
        }
    }
    return d;
}

// Decompression step 3 (Sec. III-A): where the wave's share of the chunk's data
// starts.  The workgroup owning the last chunk reports the outcome.  live: the wave has blocks to decode, inside the stream.
// PREZERO: the output was cleared to +0.0 before the launch (Sec. III-A, for
// highly compressible streams); a wave whose blocks all have rate 0 and whose
// tiles are all uncentred decodes to q = 0, i.e. +0.0 everywhere, and is not
// live.
struct DecPlace {
    const uint8_t *wave_data;
    uint64_t tile0;
    bool live;
};

template <int W, bool RANGE, bool PREZERO, int OFF>
__device__ __forceinline__ DecPlace dec_place(const DecompressArgs &a, const DecChunk &d, int slot, uint64_t total,
                                              DecompressShared<W> &sh, const GroupCursor &gc)
{
    const int tid = threadIdx.x;
    const int w = tid >> 6;
    const int lane = tid & 63;
    const int j = lane & 7;
    uint32_t chunk_total = 0, wave_base = 0;
#pragma unroll
    for (int k = 0; k < W; k++) {
        if (k < w) wave_base += sh.wave_total[slot][k];
        chunk_total += sh.wave_total[slot][k];
    }
    if (w == 0 && d.chunk == a.nchunks - 1) {
        const bool seen = gc.bad || (OFF != kByPrefix && (a.groups[gc.next] & kGroupBad) != 0);
        finish_decode<RANGE>(a, seen, d.base + chunk_total, total);
    }
    DecPlace p;
    p.tile0 = dec_chunk_tile0<W, RANGE, OFF>(a, d.chunk) + (uint64_t)w * kTilesPerWave;
    p.wave_data = a.cmp + a.data0 + d.base + wave_base;
    p.live = a.data0 + d.base + chunk_total <= total && p.tile0 < (RANGE ? a.tile_end : a.ntiles) &&
             (!RANGE || p.tile0 + kTilesPerWave > a.tile_begin);
    if (PREZERO && p.live) {
        const uint64_t gblock = (p.tile0 + (lane >> 3)) * kBlocksPerTile + j;
        p.live = __ballot(gblock < a.nblocks && (d.r != 0 || d.cent != 0)) != 0;
    }
    return p;
}

// Decompression steps 4-5 of a live wave: bit-unshuffle, inverse cross-block
// prediction (one inclusive scan for LZ1, two for LZ2, plus the tile mean),
// x' = (float)q * E.
template <bool ALIGNED, int W, bool RANGE>
__device__ __forceinline__ void dec_decode(const DecompressArgs &a, const DecChunk &d, const DecPlace &p, float E,
                                           bool indep, uint32_t *st)
{
    const int lane = threadIdx.x & 63;
    const int j = lane & 7;
    const uint64_t tile0 = p.tile0;
    const uint64_t gblock = (tile0 + (lane >> 3)) * kBlocksPerTile + j;
    const bool blk_ok = gblock < a.nblocks;
    const uint8_t *wave_data = p.wave_data;
    int mu = 0;
    if (d.cent) mu = (int)*(const g_u32 *)(wave_data + d.tile_excl);

    // ---- bit-unshuffle: stored words -> residuals.  With ns = -sign, a
    // residual is (m ^ ns) + sign for its magnitude m, and the bit planes of
    // m ^ ns are the stored magnitude planes xor the sign map (word 0); the
    // planes at or above the block's rate are zero, so there it is the sign
    // map itself.  G groups of 8 planes give x = (m ^ ns) mod 2^(8 G), so the
    // residual is x + sign (1 - 2^(8 G)) (mod 2^32).
    uint32_t code[32];
#pragma unroll
    for (int i = 0; i < 32; i++) code[i] = 0;
    const uint32_t r = blk_ok ? d.r : 0;  // magnitude planes
    const g_u32 *words = (const g_u32 *)(wave_data + d.blk_off);
    const uint32_t sw = r ? words[0] : 0u;  // sign map: element i at bit i ^ 7
    uint32_t G = 0;                         // groups assembled (wave-uniform)
    for (uint32_t g = 0; __ballot(8 * g < r) != 0; g++) {
        uint32_t Rg[8];
#pragma unroll
        for (int k = 0; k < 8; k++) Rg[k] = (8 * g + k < r ? words[1 + 8 * g + k] : 0u) ^ sw;
        transpose8(Rg);
        // Rg[rho] byte k = byte g of x of element 8k + 7 - rho
#pragma unroll
        for (int rho = 0; rho < 8; rho++) {
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint32_t sel = (0x03020100u & ~(0xFFu << (8 * g))) | ((4u + k) << (8 * g));
                code[8 * k + 7 - rho] = __builtin_amdgcn_perm(Rg[rho], code[8 * k + 7 - rho], sel);
            }
        }
        G = g + 1;
    }

    // ---- inverse cross-block prediction + dequantization
    const uint32_t M = G < 4 ? 1u - (1u << (8 * G)) : 1u;  // 1 - 2^(8 G) mod 2^32
    uint32_t acc = 0;
#pragma unroll
    for (int i = 0; i < 32; i++) {
        const uint32_t ns = (uint32_t)((int)(sw << (31 - (i ^ 7))) >> 31);  // -sign
        acc += code[i] + (ns & M);
        code[i] = acc;  // first running sum (LZ1 reconstruction / LZ2 first differences)
    }
    // carries from the blocks before in the tile (none when every block
    // restarts prediction)
    const uint32_t start1 = indep ? 0u : group_excl_scan(acc, j);
    const bool any2 = __ballot(d.order2) != 0;  // wave-uniform: some tile of the wave is LZ2
    uint32_t acc2 = 0;
    if (any2) {
#pragma unroll
        for (int i = 0; i < 32; i++) {
            acc2 += code[i] + start1;
        }
    }
    const uint32_t start2 = indep ? 0u : group_excl_scan(acc2, j);
    float xo[32];
    // the tile mean enters the start of the running sum that is the lane's
    // result: the first (LZ1) or the second (LZ2)
    const uint32_t s1 = start1 + (d.order2 ? 0u : (uint32_t)mu);
    if (!any2) {
#pragma unroll
        for (int i = 0; i < 32; i++) xo[i] = (float)(int)(code[i] + s1) * E;
    } else {
        uint32_t run = start2 + (d.order2 ? (uint32_t)mu : 0u);
#pragma unroll
        for (int i = 0; i < 32; i++) {
            const uint32_t d1 = code[i] + s1;  // first running sum with the carry
            run += d1;                         // second running sum
            xo[i] = (float)(int)(d.order2 ? run : d1) * E;
        }
    }

    // element e of the field goes to out[e - eb], for eb <= e < ee
    g_f32 *out = (g_f32 *)a.out;
    const uint64_t eb = RANGE ? a.elem_begin : 0, ee = RANGE ? a.elem_end : a.n;
    // ---- write back through LDS with coalesced stores
#pragma unroll
    for (int k = 0; k < 8; k++)
        *reinterpret_cast<float4 *>(st + lane * kStageRowDwords + 4 * k) =
            make_float4(xo[4 * k], xo[4 * k + 1], xo[4 * k + 2], xo[4 * k + 3]);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const uint64_t e0 = tile0 * kTile;
    const bool fullw = e0 >= eb && e0 + 2048 <= ee;  // the wave's 8 tiles lie inside the range
    if (ALIGNED) {  // 16-byte aligned: a.out - eb (the field's element 0) is
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int p = k * 64 + lane;
            const uint64_t e = e0 + 4ull * p;
            const u32x4 f = *reinterpret_cast<const u32x4 *>(st + (p >> 3) * kStageRowDwords + (p & 7) * 4);
            if (fullw || (e >= eb && e + 4 <= ee)) {
                __builtin_nontemporal_store(f, (g_u32x4 *)(out + (e - eb)));
            } else {
                if (e + 0 >= eb && e + 0 < ee) out[e + 0 - eb] = __uint_as_float(f.x);
                if (e + 1 >= eb && e + 1 < ee) out[e + 1 - eb] = __uint_as_float(f.y);
                if (e + 2 >= eb && e + 2 < ee) out[e + 2 - eb] = __uint_as_float(f.z);
                if (e + 3 >= eb && e + 3 < ee) out[e + 3 - eb] = __uint_as_float(f.w);
            }
        }
    } else {
#pragma unroll 8
        for (int k = 0; k < 32; k++) {
            const int p = k * 64 + lane;
            const uint64_t e = e0 + p;
            if (fullw || (e >= eb && e < ee))
                out[e - eb] = __uint_as_float(st[(p >> 5) * kStageRowDwords + (p & 31)]);
        }
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Stream header validation (identical in every workgroup): status, step E
// and the stream's total size.
__device__ __forceinline__ int dec_header(const DecompressArgs &a, float &E, uint64_t &total, bool &indep)
{
    const uint32_t *h = reinterpret_cast<const uint32_t *>(a.cmp);
    E = 1.0f;
    total = 0;
    const uint32_t h1 = h[1];
    indep = false;
    // flags: bits 0-1 free, bits 2-4 the tile configuration (a.cfg_flags: 0 for
    // the default format), the rest zero
    if (h[0] != 0x315A5346u || (h1 & 0xFFFFu) != 1u || ((h1 >> 16) & 0xFFu) > 1u || ((h1 >> 24) & ~0x1Fu) != 0u ||
        ((h1 >> 24) & 0x1Cu) != a.cfg_flags)
        return FSZ_ERR_CORRUPT;
    indep = ((h1 >> 25) & 1u) != 0;  // flags bit 1: prediction restarts at every block
    if (((uint64_t)h[3] << 32 | h[2]) != a.n) return FSZ_ERR_SIZE_MISMATCH;
    E = __uint_as_float(h[4]);
    total = (uint64_t)h[7] << 32 | h[6];
    if (!__builtin_isfinite(E) || !(E > 0.0f) || total > a.cmp_size || total < a.data0) return FSZ_ERR_CORRUPT;
    return FSZ_OK;
}

// Persistent decompression kernel for the offsets pre-pass: the size pass of
// the next chunk runs before the decode of the current one.  W waves per
// workgroup; a chunk is 8 tiles per wave; chunks [a.chunk_begin, a.nchunks).
// With every chunk's offset known no workgroup waits on another, and a static
// schedule (chunk = workgroup + k * grid) needs no ticket.
template <bool ALIGNED, int W, bool RANGE, bool PREZERO>
__global__ __launch_bounds__(W * 64) void decompress_kernel(DecompressArgs a)
{
    __shared__ __attribute__((aligned(16))) uint32_t stage[W * kStageWaveDwords];
    __shared__ DecompressShared<W> sh;
    const int tid = threadIdx.x;
    uint32_t *st = stage + (tid >> 6) * kStageWaveDwords;

    float E;
    uint64_t total;
    bool indep;
    const int hst = dec_header(a, E, total, indep);
    if (hst != FSZ_OK) {
        if (tid == 0 && blockIdx.x == 0) write_final(a.final, 0, hst, a.epoch);
        return;
    }
    uint64_t cur = a.chunk_begin + blockIdx.x;
    if (cur >= a.nchunks) return;
    int slot = 0;
    GroupCursor gc;
    DecChunk dc = dec_sizes<W, RANGE, kByGroups>(a, cur, dec_rate_byte<W, RANGE, kByGroups>(a, cur), slot, sh, gc);
    for (;;) {
        const uint64_t nxt = cur + gridDim.x;
        const int nslot = slot == 2 ? 0 : slot + 1;
        DecChunk dn;
        if (nxt < a.nchunks)
            dn = dec_sizes<W, RANGE, kByGroups>(a, nxt, dec_rate_byte<W, RANGE, kByGroups>(a, nxt), nslot, sh, gc);
        const DecPlace pl = dec_place<W, RANGE, PREZERO, kByGroups>(a, dc, slot, total, sh, gc);
        if (pl.live) dec_decode<ALIGNED, W, RANGE>(a, dc, pl, E, indep, st);
        if (nxt >= a.nchunks) break;
        dc = dn;
        cur = nxt;
        slot = nslot;
    }
}

// ------------------------------------------------------------------ whole-field decode: offsets pre-pass
//
// A whole-field decode's chunk offsets depend on the rate header alone
// (decompression steps 1-2, Sec. III-A), so one small launch computes them
// before the decoder starts, and the decoder reads its chunk's offset instead
// of waiting on a lookback.
//
// The pre-pass has no order between workgroups either: each takes one group of
// kGroupTiles << m consecutive tiles, writes the offset of each of its chunks
// inside the group and the group's total, and ends.  The decoder adds up the
// totals of the groups before its own, 64 per load; m is the least that keeps
// them at kMaxGroupWords (8 loads for the last chunk of any field).  What bounds
// it is one round trip for the rate bytes and the launch itself: 512^3 takes
// 4.9 us, where workgroups in ticket order with a decoupled lookback
// over their totals took 9.4 us (25 M elements: 4.7 against 8.0 us).

// One group: tiles [group * passes * kGroupTiles, ...) below a.tile_end.
// 2^tpc_log2 tiles per decoder chunk (at least a thread's tiles); T blocks per
// tile of HB 32-element segments each (the default format: 8 and 1; the tile
// configurations: the stream's).  The rate header is read where it lies inside
// the buffer, before anything has looked at the stream header.
template <int T, int HB>
__device__ __forceinline__ void group_sums(const DecompressArgs &a, uint64_t group, uint32_t passes,
                                           uint32_t tpc_log2, unsigned long long *offs, unsigned long long *groups)
{
    static_assert(T == 4 || T == 8 || T == 16, "a tile's rate bytes are 1, 2 or 4 words");
    constexpr int kWavesG = kGroupThreads / 64;
    constexpr int kWords = kGroupTilesPerThread * T / 4;
    __shared__ uint32_t wsum[2][kWavesG];
    __shared__ uint32_t wbad[kWavesG];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = tid >> 6;
    if (a.data0 > a.cmp_size) return;  // the decoder reports it
    const uint64_t nb = a.tile_end < a.ntiles ? a.tile_end * T : a.nblocks;  // blocks of the tiles up to tile_end
    uint64_t run = 0;
    uint32_t bad = 0;
    for (uint32_t p = 0; p < passes; p++) {
        const uint64_t tile0 =
            ((group * passes + p) * kGroupThreads + (uint64_t)tid) * kGroupTilesPerThread;
        uint32_t units = 0, cents = 0;
        const g_u32 *rp = (const g_u32 *)(a.cmp + kHeaderBytes + tile0 * T);
        if ((tile0 + kGroupTilesPerThread) * T <= nb) {
            uint32_t rw[kWords];
#pragma unroll
            for (int q = 0; q < kWords; q++) rw[q] = rp[q];
#pragma unroll
            for (int q = 0; q < kWords; q++) {
                const bool head = q % (T / 4) == 0;
                bad |= rw[q] & (head ? 0xE0E0E020u : 0xE0E0E0E0u);
                units = rate_units(rw[q], units);
                if (head) cents += (rw[q] >> 6) & 1u;
            }
        } else if (tile0 * T < nb) {  // the last blocks, byte by byte
            const uint64_t left = nb - tile0 * T;
            for (uint32_t k = 0; k < (uint32_t)left; k++) {
                const uint32_t rb = ((const g_u8 *)rp)[k];
                const bool head = k % T == 0;
                bad |= rb & (head ? 0x20u : 0xE0u);
                units = rate_units(rb & 0xFFu, units);
                if (head) cents += (rb >> 6) & 1u;
            }
        }
        const uint32_t z = 4u * HB * units + 4u * cents;
        const uint32_t incl = (uint32_t)wave_incl_scan((int)z);
        if (lane == 63) wsum[p & 1][w] = incl;
        lds_barrier();
        uint32_t wave_base = 0, ptotal = 0;
#pragma unroll
        for (int k = 0; k < kWavesG; k++) {
            if (k < w) wave_base += wsum[p & 1][k];
            ptotal += wsum[p & 1][k];
        }
        if (tile0 < a.tile_end && (tile0 & ((1u << tpc_log2) - 1u)) == 0) offs[tile0 >> tpc_log2] = run + wave_base + incl - z;
        run += ptotal;
    }
    const bool wave_bad = __ballot(bad != 0) != 0;
    if (lane == 0) wbad[w] = wave_bad ? 1u : 0u;
    lds_barrier();
    if (tid == 0) {
        uint32_t any = 0;
#pragma unroll
        for (int k = 0; k < kWavesG; k++) any |= wbad[k];
        groups[group] = run | (any ? kGroupBad : 0ull);
        if (a.tile_end == 0) offs[0] = 0;
    }
}

// The group totals as running sums: the bytes before each group, and in bit 63
// whether it or one before it holds a reserved bit.
__global__ __launch_bounds__(512) void dec_groups_scan_kernel(unsigned long long *groups, uint32_t ngroups)
{
    static_assert(kMaxGroupWords <= 512, "one group per thread");
    __shared__ unsigned long long sum[8];
    __shared__ uint32_t first_bad[8];
    const uint32_t k = threadIdx.x;
    const int lane = k & 63, w = k >> 6;
    const unsigned long long t = k < ngroups ? groups[k] : 0ull;
    unsigned long long v = t & ~kGroupBad;
    v += dpp64<kRowShr1>(v);
    v += dpp64<kRowShr2>(v);
    v += dpp64<kRowShr4>(v);
    v += dpp64<kRowShr8>(v);
    v += dpp64<kRowBcast15, 0xA>(v);
    v += dpp64<kRowBcast31, 0xC>(v);
    const unsigned long long bad = __ballot((t & kGroupBad) != 0);
    if (lane == 63) {
        sum[w] = v;
        first_bad[w] = bad ? 64u * w + (uint32_t)__builtin_ctzll(bad) : ~0u;
    }
    lds_barrier();
    unsigned long long before = 0;
    uint32_t first = ~0u;
#pragma unroll
    for (int j = 0; j < 8; j++) {
        if (j < w) before += sum[j];
        first = min(first, first_bad[j]);
    }
    if (k < ngroups) groups[k] = (before + v - (t & ~kGroupBad)) | (first <= k ? kGroupBad : 0ull);
}

template <int T, int HB>
__global__ __launch_bounds__(kGroupThreads) void dec_groups_kernel(DecompressArgs a, unsigned long long *offs,
                                                                   unsigned long long *groups, uint32_t passes,
                                                                   uint32_t tpc_log2)
{
    group_sums<T, HB>(a, blockIdx.x, passes, tpc_log2, offs, groups);
}

// One chunk of 8*W tiles per workgroup and no order to keep: the hardware
// dispatcher keeps the CUs busy.
// kByGroupsOnce: the decoder behind the offsets pre-pass for fields too small to
// give the persistent grid several chunks per workgroup.
// kByPrefix: the only launch of a small decode.  Every workgroup adds up all
// rate bytes before its chunk itself (at most kPrefixBytes, read from the L2
// after the first workgroups; 8 VALU operations per 4 bytes), so nothing is
// passed between workgroups: two dependent round trips to memory (rate bytes,
// then the data words) where the ticket, the aggregate's two barriers and the
// lookback of the earlier form were five (2^20 sinusoid 7.5 -> 6.1 us per call,
// 2^16 6.6 -> 4.8, a range of 300 elements at 10^6 13.8 -> 6.5).
// The size pass needs nothing of the stream header but the room for the rate
// bytes, so its loads go out before the header's have come back.
template <bool ALIGNED, int W, bool RANGE, int OFF, bool PREZERO = false>
__device__ __forceinline__ void decompress_one(const DecompressArgs &a, uint64_t chunk, DecompressShared<W> &sh,
                                               uint32_t *st)
{
    GroupCursor gc;
    DecChunk dc;
    const bool room = a.data0 <= a.cmp_size;
    if (room) dc = dec_sizes<W, RANGE, OFF>(a, chunk, dec_rate_byte<W, RANGE, OFF>(a, chunk), 0, sh, gc);
    float E;
    uint64_t total;
    bool indep;
    const int hst = dec_header(a, E, total, indep);
    if (!room || hst != FSZ_OK) {
        if (threadIdx.x == 0 && chunk == a.chunk_begin) write_final(a.final, 0, hst, a.epoch);
        return;
    }
    const DecPlace pl = dec_place<W, RANGE, PREZERO, OFF>(a, dc, 0, total, sh, gc);
    if (pl.live) dec_decode<ALIGNED, W, RANGE>(a, dc, pl, E, indep, st);
}

template <bool ALIGNED, int W, bool RANGE, int OFF, bool PREZERO>
__global__ __launch_bounds__(W * 64) void decompress_direct_kernel(DecompressArgs a)
{
    __shared__ __attribute__((aligned(16))) uint32_t stage[W * kStageWaveDwords];
    __shared__ DecompressShared<W> sh;
    decompress_one<ALIGNED, W, RANGE, OFF, PREZERO>(a, a.chunk_begin + blockIdx.x, sh,
                                                    stage + (threadIdx.x >> 6) * kStageWaveDwords);
}

// ------------------------------------------------------------------ batched form

// Index of the job owning global item t, given the non-decreasing array
// end[j] = first item after job j: the number of jobs with end[j] <= t.
// Run by a whole wave (64 jobs per probe); the result is wave-uniform.
__device__ __forceinline__ uint32_t find_job(const uint64_t *end, uint32_t njobs, uint64_t t)
{
    const int lane = __lane_id();
    for (uint32_t base = 0; base < njobs; base += 64) {
        const uint32_t idx = base + lane;
        const unsigned long long m = __ballot(idx < njobs && end[idx] <= t);
        if (m != ~0ull) return base + (uint32_t)__builtin_popcountll(m);
    }
    return njobs;
}

__device__ __forceinline__ DecompressArgs batch_decompress_args(const BatchArgs &b, const BatchJob &J)
{
    DecompressArgs a;
    a.cmp = static_cast<const uint8_t *>(J.src);
    a.cmp_size = J.src_size;
    a.out = static_cast<float *>(J.dst);
    a.n = J.n;
    a.ntiles = J.ntiles;
    a.nblocks = J.nblocks;
    a.nchunks = J.nchunks;
    a.data0 = J.data0;
    a.tile_begin = 0;
    a.tile_end = J.ntiles;
    a.elem_begin = 0;
    a.elem_end = J.n;
    a.chunk_begin = 0;
    a.cfg_flags = 0;
    a.groups = b.dec.groups + J.seg_base;
    a.offsets = b.dec.offsets + J.chunk_base;
    a.group_shift = J.group_shift;
    a.epoch = b.epoch;
    a.flag_epoch = 0;
    a.flags = nullptr;
    a.ticket = nullptr;
    a.final = J.final;
    return a;
}

// Batched range pass and offsets pre-pass.  The first b.dec.group_wgs
// workgroups each sum a group of tiles of a decompress job (as
// dec_groups_kernel), or several one after the other.  The others reduce segments (kSegElems elements of one
// compress job, a partial each) and clear the batch's chunk flags for the
// kernel that follows.
__global__ __launch_bounds__(kStatsThreads) void batch_stats_kernel(BatchArgs b)
{
    static_assert(kStatsThreads == kGroupThreads, "both parts of the launch");
    if (blockIdx.x == 0 && threadIdx.x == 0 && b.h_done)  // the job table's copy is done with its staging
        __hip_atomic_store(b.h_done, b.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (blockIdx.x < b.dec.group_wgs) {
        for (uint64_t g = blockIdx.x; g < b.dec.total_groups; g += b.dec.group_wgs) {
            const uint32_t job = __builtin_amdgcn_readfirstlane(find_job(b.dec.group_end, b.dec.njobs, g));
            if (job >= b.dec.njobs) return;
            const BatchJob &J = b.dec.jobs[job];
            DecompressArgs a = batch_decompress_args(b, J);
            group_sums<kBlocksPerTile, 1>(a, g - J.seg_base, J.group_passes, b.dec.tpc_log2,
                                          b.dec.offsets + J.chunk_base, b.dec.groups + J.seg_base);
            lds_barrier();  // its shared slots are reused by the next group
        }
        return;
    }
    const uint64_t wg = blockIdx.x - b.dec.group_wgs, nwg = gridDim.x - b.dec.group_wgs;
    for (uint64_t i = wg * kStatsThreads + threadIdx.x; i < b.nflags; i += nwg * kStatsThreads) b.flags[i] = 0;
    // workgroups loop over segments (one partial each), so the job search and
    // the workgroup start are paid once per several segments
    for (uint64_t seg = wg; seg < b.total_segs; seg += nwg) {
        const uint32_t job = __builtin_amdgcn_readfirstlane(find_job(b.seg_end, b.njobs, seg));
        if (job >= b.njobs) return;
        const BatchJob &J = b.jobs[job];
        const g_f32 *x = (const g_f32 *)J.src;
        const uint64_t e0 = (seg - J.seg_base) * kSegElems;
        const uint64_t e1 = J.n - e0 < (uint64_t)kSegElems ? J.n : e0 + kSegElems;
        RangeAcc acc;
        const int tid = threadIdx.x;
        // 16-byte loads, four in flight per thread; the elements before the
        // segment's first and after its last 16-byte boundary singly
        const uint32_t head = (uint32_t)min((uint64_t)align_head((const void *)J.src), e1 - e0);
        const g_f4 *x4 = (const g_f4 *)(x + e0 + head);
        const uint32_t nv = (uint32_t)((e1 - e0 - head) / 4);
        if (nv == kSegElems / 4) {
#pragma unroll 2
            for (int k = 0; k < kSegElems / (4 * kStatsThreads); k += 4) {
                const f4 f0 = __builtin_nontemporal_load(x4 + (k + 0) * kStatsThreads + tid);
                const f4 f1 = __builtin_nontemporal_load(x4 + (k + 1) * kStatsThreads + tid);
                const f4 f2 = __builtin_nontemporal_load(x4 + (k + 2) * kStatsThreads + tid);
                const f4 f3 = __builtin_nontemporal_load(x4 + (k + 3) * kStatsThreads + tid);
                acc.take4(f0);
                acc.take4(f1);
                acc.take4(f2);
                acc.take4(f3);
            }
        } else {
            uint32_t k = tid;
            for (; k + 3 * kStatsThreads < nv; k += 4 * kStatsThreads) {
                const f4 f0 = __builtin_nontemporal_load(x4 + k);
                const f4 f1 = __builtin_nontemporal_load(x4 + k + kStatsThreads);
                const f4 f2 = __builtin_nontemporal_load(x4 + k + 2 * kStatsThreads);
                const f4 f3 = __builtin_nontemporal_load(x4 + k + 3 * kStatsThreads);
                acc.take4(f0);
                acc.take4(f1);
                acc.take4(f2);
                acc.take4(f3);
            }
            for (; k < nv; k += kStatsThreads) acc.take4(f4(x4[k]));
        }
        if ((uint32_t)tid < head) acc.take(x[e0 + tid]);
        const uint64_t t = e0 + head + 4ull * nv + tid;
        if (t < e1) acc.take(x[t]);
        const StatsPartial p = acc.reduce();
        if (tid == 0) b.partials[seg] = p;
        __syncthreads();  // the reduction's shared slots are reused by the next segment
    }
}

// Per-job fold of the batched range pass (one workgroup per job) and the job's
// bound.
template <int THREADS>
__device__ __forceinline__ void fold_job_stats(const BatchArgs &b, uint32_t job)
{
    const BatchJob &J = b.jobs[job];
    float mn = INFINITY, mx = -INFINITY, ma = 0.0f;
    uint32_t nf = 0;
    for (uint64_t i = threadIdx.x; i < J.nsegs; i += THREADS)
        stats_combine(mn, mx, ma, nf, b.partials[J.seg_base + i]);
    const StatsPartial p = stats_block_reduce<THREADS>(mn, mx, ma, nf);
    if (threadIdx.x == 0)
        b.bounds[job] = resolve_bound(fsz_stats{p.xmin, p.xmax, p.maxabs, p.flags}, J.mode, J.value, J.n);
}

__global__ __launch_bounds__(kStatsThreads) void batch_stats_final_kernel(BatchArgs b)
{
    fold_job_stats<kStatsThreads>(b, blockIdx.x);
}

// Batched decompression: one (job, chunk) item per workgroup, as
// decompress_direct_kernel.  The range-pass launch has placed every chunk in
// its group (group_sums), so no item waits on another.  The first b.njobs
// workgroups fold the range pass of the batch's compress jobs, whose kernel
// comes next: a mixed batch has no launch more than a compression.  64 fields of 16 K to
// 16 M elements (125 M together): 117 us per call, where a persistent grid
// with tickets and a lookback per job took 221.
template <bool ALIGNED, int W>
__global__ __launch_bounds__(W * 64) void batch_dec_kernel(BatchArgs b)
{
    __shared__ DecompressShared<W> sh;
    __shared__ __attribute__((aligned(16))) uint32_t stage[W * kStageWaveDwords];
    if (blockIdx.x < b.njobs) {
        fold_job_stats<W * 64>(b, blockIdx.x);
        return;
    }
    const uint64_t t = blockIdx.x - b.njobs;
    const uint32_t job = __builtin_amdgcn_readfirstlane(find_job(b.dec.chunk_end, b.dec.njobs, t));
    if (job >= b.dec.njobs) return;
    const BatchJob &J = b.dec.jobs[job];
    decompress_one<ALIGNED, W, false, kByGroupsOnce>(batch_decompress_args(b, J), t - J.chunk_base, sh,
                                                     stage + (threadIdx.x >> 6) * kStageWaveDwords);
}

}  // namespace

hipError_t launch_stats_partials(const StatsArgs &a, uint32_t *nparts, hipStream_t s)
{
    // 512 threads from 2^21 elements on; below, 256 (and the same 16 elements
    // per thread) reach more CUs (2^20 13.0 against 13.3 us per compression)
    const bool small = a.n <= (1ull << 21);
    const uint64_t want = ceil_div(a.n, (small ? 256ull : 512ull) * 16);
    *nparts = (uint32_t)(want < 1 ? 1 : (want > kRangeMaxBlocks ? kRangeMaxBlocks : want));
    if (small)
        hipLaunchKernelGGL(stats_partial_kernel<256>, dim3(*nparts), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(stats_partial_kernel<512>, dim3(*nparts), dim3(512), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_stats(const StatsArgs &a, hipStream_t s)
{
    uint32_t nparts = 0;
    const hipError_t e = launch_stats_partials(a, &nparts, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(stats_final_kernel, dim3(1), dim3(kStatsThreads), 0, s, a, nparts);
    return hipGetLastError();
}

// ------------------------------------------------------------------ batched pipelined compression
//
// The compress jobs of a batch: the control-wave pipeline of
// compress_ctrl_kernel over the batch's work items.  Tickets are global item
// ids in job order; every item in flight carries its job, whose arguments
// (input, output, flag range, bound) come from the job table where they are
// needed, so one pipeline runs across job boundaries.  Items of a job whose
// bound does not resolve stay in the pipeline as empty items (no flags, no
// stores); the job's last item reports its status.  Each job's bytes equal a
// plain call's.

struct BItem {
    uint64_t t;    // global item id (>= total_chunks: none)
    uint32_t job;  // job index (njobs: none)
    uint64_t c;    // chunk index inside the job
};

// An item's job is the same in every lane and nothing writes the tables while
// the kernel runs: read through the constant address space, a job's record
// and bound come by scalar loads, into scalar registers and from the scalar
// cache.  (Copies of the records in LDS went through vector registers and took
// the room of an eleventh data wave.)
typedef __attribute__((address_space(4))) BatchJob c_job;
typedef __attribute__((address_space(4))) Resolved c_resolved;

__device__ __forceinline__ Resolved job_bound(const BatchArgs &b, uint32_t job)
{
    const c_resolved *r = (const c_resolved *)(b.bounds + job);
    return Resolved{r->E, r->inv, r->flags, r->status};
}

// The arguments of a job's chunks, as the whole-field kernels take them.
__device__ __forceinline__ CompressArgs batch_compress_args(const BatchArgs &b, uint32_t job)
{
    const c_job *J = (const c_job *)(b.jobs + job);
    CompressArgs a;
    a.x = static_cast<const float *>(J->src);
    a.n = J->n;
    a.ntiles = J->ntiles;
    a.nblocks = J->nblocks;
    a.nchunks = J->nchunks;
    a.data0 = J->data0;
    a.out = static_cast<uint8_t *>(J->dst);
    a.capacity = J->dst_capacity;
    a.stats = nullptr;
    a.partials = nullptr;
    a.nparts = 0;
    a.value = J->value;
    a.mode = J->mode;
    a.features = kFeaturesAll;
    a.cfg_flags = 0;
    a.epoch = b.epoch;
    a.flag_epoch = 1;
    a.flags = b.flags + J->chunk_base * kFlagStride;
    a.ticket = nullptr;
    a.final = J->final;
    return a;
}

__device__ __forceinline__ BItem batch_item(const BatchArgs &b, uint64_t t, uint32_t job)
{
    BItem it;
    it.t = uniform(t);
    it.job = uniform(t < b.total_chunks && job < b.njobs ? job : b.njobs);
    it.c = it.job < b.njobs ? it.t - ((const c_job *)(b.jobs + it.job))->chunk_base : 0;
    return it;
}

__device__ __forceinline__ BItem batch_item_of(const BatchArgs &b, const uint64_t *chunk_end, uint64_t t)
{
    return batch_item(b, t, t < b.total_chunks ? find_job(chunk_end, b.njobs, t) : b.njobs);
}

template <int W>
__device__ __forceinline__ void batch_fetch(const BatchArgs &b, const BItem &it, uint32_t *qb,
                                            int w, int lane)
{
    chunk_fetch<W>(batch_compress_args(b, it.job), it.c, qb, w, lane);
}

// Rate pass of item B (as compress_rates), or an empty state and
// the same barrier for an item whose job has no valid bound.
template <int W>
__device__ __forceinline__ ChunkState batch_rates(const BatchArgs &b, const BItem &it,
                                                  int (&x)[32], int slot, CompressShared<W> &sh)
{
    const Resolved R = job_bound(b, it.job);
    if (R.status == FSZ_OK) {
        ChunkState cs = compress_rates<W>(batch_compress_args(b, it.job), R, it.c, x, slot, sh);
        cs.chunk = it.c;
        return cs;
    }
    ChunkState cs{};
    cs.chunk = it.c;
    if ((threadIdx.x & 63) == 0) sh.wave_total[slot][threadIdx.x >> 6] = 0;
    lds_barrier();
    return cs;
}

// A data wave's step of the batched pipeline: as pipe2_step, with A, B, C and
// the new item each in its own job.
template <int W>
__device__ __forceinline__ BItem batch_pipe_step(const BatchArgs &b, const BItem &iA,
                                                 const ChunkState &ca, int (&xa)[32], int sa, const BItem &iB,
                                                 int (&yb)[32], ChunkState &cb, const BItem &iC, uint32_t *qb,
                                                 uint32_t *pb, CompressShared<W> &sh, const uint32_t (&s_job)[2], int w)
{
    const uint64_t N = b.total_chunks;
    const int lane = threadIdx.x & 63;
    const int j = lane & 7;
    if (iB.t < N) cb = batch_rates<W>(b, iB, yb, sa ^ 1, sh);
    uint32_t wave_base, chunk_total;
    chunk_totals<W>(sh, sa, w, wave_base, chunk_total);
    lds_barrier();  // the control wave has A's offset and the new ticket
    const uint64_t base = uniform((uint64_t)sh.base[sa]);
    const BItem iD = batch_item(b, sh.ticket[sa], s_job[sa]);

    const CompressArgs aA = batch_compress_args(b, iA.job);
    const bool liveA = job_bound(b, iA.job).status == FSZ_OK;
    const uint64_t tile0 = iA.c * (kTilesPerWave * W) + (uint64_t)w * kTilesPerWave;
    const bool ok = liveA && aA.data0 + base + chunk_total <= aA.capacity && tile0 < aA.ntiles;
    uint32_t *wave_out = reinterpret_cast<uint32_t *>(aA.out + aA.data0 + base + wave_base);
    uint32_t *ps = pb + (((uint32_t)(uintptr_t)wave_out >> 2) & 3u);  // staging at the output's 16-byte phase
    if (ok) pipe2_stage<false>(ca, xa, ps);  // fits: a batch computes its own statistics
    if (iC.t < N) chunk_read(qb, lane, xa);
    if (iD.t < N) {
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the read of qb is done before it is overwritten
        batch_fetch<W>(b, iD, qb, w, lane);
    }
    if (liveA && ca.vm != 0)
        ((g_u8 *)aA.out)[kHeaderBytes + (tile0 + (lane >> 3)) * kBlocksPerTile + j] = (uint8_t)ca.rbyte;
    if (ok) {
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        wave_store_staged_phased(wave_out, ps, ca.wave_total >> 2, lane);
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    return iD;
}

template <int W>
__device__ __forceinline__ void batch_pipe_run(const BatchArgs &b, const uint64_t *chunk_end, CompressShared<W> &sh,
                                               const uint32_t (&s_job)[2], uint32_t *qb, uint32_t *pb, int w)
{
    const int lane = threadIdx.x & 63;
    const uint64_t N = b.total_chunks;
    const uint64_t takes = N + gridDim.x;
    int tslot = 0;
    BItem iA = batch_item_of(b, chunk_end, next_ticket(b.ticket, takes, sh, tslot));
    if (iA.t >= N) return;
    batch_fetch<W>(b, iA, qb, w, lane);
    BItem iB = batch_item_of(b, chunk_end, next_ticket(b.ticket, takes, sh, tslot));
    int x[32], y[32];
    chunk_read(qb, lane, x);
    if (iB.t < N) {
        __builtin_amdgcn_s_waitcnt(0xC07F);
        batch_fetch<W>(b, iB, qb, w, lane);
    }
    ChunkState ca = batch_rates<W>(b, iA, x, 0, sh);
    ChunkState cb = ca;
    BItem iC = batch_item(b, N, b.njobs);
    if (iB.t < N) {
        iC = batch_item_of(b, chunk_end, next_ticket(b.ticket, takes, sh, tslot));
        chunk_read(qb, lane, y);
        if (iC.t < N) {
            __builtin_amdgcn_s_waitcnt(0xC07F);
            batch_fetch<W>(b, iC, qb, w, lane);
        }
    }
    // loop invariant: A rate-passed in x (slot 0), B read into y, C in flight
    for (;;) {
        const BItem iD = batch_pipe_step<W>(b, iA, ca, x, 0, iB, y, cb, iC, qb, pb, sh, s_job, w);
        if (iB.t >= N) return;
        const BItem iE = batch_pipe_step<W>(b, iB, cb, y, 1, iC, x, ca, iD, qb, pb, sh, s_job, w);
        if (iC.t >= N) return;
        iA = iC;
        iB = iD;
        iC = iE;
    }
}

// The control wave (as ctrl_run): tickets, their jobs, and the lookback of the
// item rate-passed in the previous step.  Passes every barrier of the data
// waves.
template <int W>
__device__ __forceinline__ void batch_ctrl_run(const BatchArgs &b, const uint64_t *chunk_end, CompressShared<W> &sh,
                                               uint32_t (&s_job)[2])
{
    const uint64_t N = b.total_chunks;
    const uint64_t takes = N + gridDim.x;
    const int lane = __lane_id();
    __builtin_amdgcn_s_setprio(3);  // as ctrl_run
    int tslot = 0;
    BItem iA = batch_item_of(b, chunk_end, next_ticket(b.ticket, takes, sh, tslot));
    if (iA.t >= N) return;
    BItem iB = batch_item_of(b, chunk_end, next_ticket(b.ticket, takes, sh, tslot));
    lds_barrier();  // the rate pass of A
    BItem iC = batch_item(b, N, b.njobs);
    if (iB.t < N) iC = batch_item_of(b, chunk_end, next_ticket(b.ticket, takes, sh, tslot));
    for (int sa = 0;; sa ^= 1) {
        const bool take = iC.t < N;
        unsigned long long traw = 0;
        if (take && lane == 0) traw = atomicAdd(b.ticket, 1ull);
        uint32_t chunk_total = 0;
#pragma unroll
        for (int k = 0; k < W; k++) chunk_total += sh.wave_total[sa][k];  // A's, from the previous step
        const CompressArgs aA = batch_compress_args(b, iA.job);
        const Resolved RA = job_bound(b, iA.job);
        Prefix pre{0, false};
        if (RA.status == FSZ_OK) pre = lookback_wait(aA.flags, iA.c, aA.flag_epoch, chunk_total, false);
        const unsigned long long tk = take ? uniform((uint64_t)traw) : N;
        const uint32_t jobD = tk < N ? find_job(chunk_end, b.njobs, tk) : b.njobs;
        if (iB.t < N) lds_barrier();  // the data waves' rate pass of B
        if (lane == 0) {
            if (take && tk == takes - 1)
                __hip_atomic_store(b.ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sh.base[sa] = pre.excl;
            sh.ticket[sa] = tk;
            s_job[sa] = jobD;
            if (iA.c == aA.nchunks - 1) {
                if (RA.status == FSZ_OK)
                    finish_stream(aA, RA, pre, chunk_total);
                else
                    write_final(aA.final, 0, (uint32_t)RA.status, aA.epoch);
            }
        }
        lds_barrier();  // the offset and the ticket go out
        if (iB.t >= N) return;
        iA = iB;
        iB = iC;
        iC = batch_item(b, tk, jobD);
    }
}

// W data waves (8 tiles each per item) and a control wave, one workgroup per
// CU (compress_batch_waves).  LDSJOBS (njobs <= kPipeLdsJobs): the jobs' chunk
// ends are copied to LDS at the start for the control wave's searches.  64
// fields of 125 M elements: 219 us per call with the range pass, where groups of 4
// waves whose wave 0 walked the lookback beside its data took 309 and such
// groups of 8 waves 266.
constexpr uint32_t kPipeLdsJobs = 512;
template <int W, bool LDSJOBS>
__global__ __launch_bounds__((W + 1) * 64) void batch_pipe_kernel(BatchArgs b)
{
    __shared__ CompressShared<W> sh;
    __shared__ uint32_t s_job[2];  // the job of the ticket in the same slot of sh
    __shared__ __attribute__((aligned(16))) uint32_t inbuf[W * kPipeInDwords];
    __shared__ __attribute__((aligned(16))) uint32_t stbuf[W * kPipeOutDwords];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
    uint32_t *qb = inbuf + w * kPipeInDwords;
    uint32_t *pb = stbuf + w * kPipeOutDwords;
    if (LDSJOBS) {
        __shared__ uint64_t lend[kPipeLdsJobs];
        for (uint32_t k = threadIdx.x; k < b.njobs; k += blockDim.x) lend[k] = b.chunk_end[k];
        lds_barrier();
        if (w < W)
            batch_pipe_run<W>(b, lend, sh, s_job, qb, pb, w);
        else
            batch_ctrl_run<W>(b, lend, sh, s_job);
    } else {
        if (w < W)
            batch_pipe_run<W>(b, b.chunk_end, sh, s_job, qb, pb, w);
        else
            batch_ctrl_run<W>(b, b.chunk_end, sh, s_job);
    }
}

// ------------------------------------------------------------------ tile configurations
//
// The tile-configuration sweep of Sec. VI-C (Table V): blocks of B = 32 HB
// elements (HB = 1 or 2) and tiles of T blocks, recorded in header flags bits
// 2-4.  As in the default kernels a lane holds one 32-element segment; a block
// spans HB lanes and a tile L = HB T lanes (4 to 32), so the cross-block chain
// runs over L lanes.  A 64-element block's words (sign map, planes) are 64
// bits with element i at bit 63 - i, written most-significant byte first:
// the stored words of its two halves side by side, so the lane of half h
// writes its word k at byte 8k + 4h of the block.  The decoder runs one chunk
// of kCfgDecWaves waves per workgroup.

// a decoding wave's staging area: padded output rows (64 x 36 dwords)
constexpr int kCfgStageDwords = 64 * kStageRowDwords;

// Sum over aligned groups of L lanes, in every lane of the group.  For binary32
// values the butterfly adds the groups' halves in index order at each level,
// so it reproduces the pairwise tree bit for bit (addition is commutative).
template <int L, typename V>
__device__ __forceinline__ V lane_group_sum(V v)
{
#pragma unroll
    for (int k = 1; k < L; k <<= 1) v = v + __shfl_xor(v, k);
    return v;
}

// Inclusive prefix sum over aligned runs of `run` lanes (a power of two, at
// most L); pos = the lane's index inside its group of L lanes.
template <int L>
__device__ __forceinline__ uint32_t lane_run_incl_scan(uint32_t v, int pos, int run)
{
#pragma unroll
    for (int k = 1; k < L; k <<= 1) {
        const uint32_t t = __shfl_up(v, k);
        if (k < run && (pos & (run - 1)) >= k) v += t;
    }
    return v;
}

// Rate pass of one chunk of W waves in a tile configuration (for TileCfg): tile mean,
// quantization, cross-block extrema, four-way evaluation and selection, and
// the offsets of the lane's words inside its wave (blk_off, with the lane's
// half h of a 64-element block at byte 4 h).  One workgroup barrier; wave 1
// publishes the chunk's aggregate.  On return x holds the LZ1 residuals.
template <int HB, int L, int W>
__device__ __forceinline__ ChunkState cfg_rates(const CompressArgs &a, const Resolved &R, uint64_t chunk,
                                                int (&x)[32], int slot, CompressShared<W> &sh)
{
    const int tid = threadIdx.x;
    const int w = tid >> 6;
    const int lane = tid & 63;
    const int tl = lane % L;  // lane inside the tile
    const int h = tl % HB;    // half of a 64-element block
    const uint64_t seg0 = (chunk * W + (uint64_t)w) * 64;  // the wave's first segment
    const uint64_t seg = seg0 + lane;
    const uint64_t e0 = seg * 32;
    const int cnt = e0 >= a.n ? 0 : (a.n - e0 >= 32 ? 32 : (int)(a.n - e0));
    const bool tile_ok = seg / L < a.ntiles;
    const bool full = (seg0 + 64) * 32 <= a.n;  // wave-uniform
    ChunkState cs;
    cs.chunk = chunk;
    cs.vm = cnt >= 32 ? 0xFFFFFFFFu : ((1u << cnt) - 1u);

    // ---- tile mean: pairwise binary32 tree over the B T slots, times 1/(B T)
    float s16[16];
#pragma unroll
    for (int i = 0; i < 16; i++) s16[i] = __int_as_float(x[2 * i]) + __int_as_float(x[2 * i + 1]);
#pragma unroll
    for (int i = 0; i < 8; i++) s16[i] = s16[2 * i] + s16[2 * i + 1];
#pragma unroll
    for (int i = 0; i < 4; i++) s16[i] = s16[2 * i] + s16[2 * i + 1];
#pragma unroll
    for (int i = 0; i < 2; i++) s16[i] = s16[2 * i] + s16[2 * i + 1];
    const float ts = lane_group_sum<L>(s16[0] + s16[1]);
    const float mean_q = (ts * (1.0f / (float)(32 * L))) * R.inv;
    const bool centre_ok = __builtin_isfinite(mean_q);
    const int mu = centre_ok ? (int)__builtin_rintf(mean_q) : 0;
    cs.mu = mu;

    // ---- quantize (biased), cross-block state from the previous lane of the tile
#pragma unroll
    for (int i = 0; i < 32; i++) x[i] = __float_as_int(__int_as_float(x[i]) * R.inv + kQMagic);
    const int p31 = __shfl_up(x[31], 1);
    const int p30 = __shfl_up(x[30], 1);
    const bool first = tl == 0;  // the tile start: the prediction restarts
    cs.first = first;
    const int carry_b = first ? kQBias : p31;
    cs.carry_l1 = first ? 0 : p31 - p30;
    uint32_t a1, a2;
    int l2_1;
    if (full)
        block_extrema<true>(x, carry_b, cs.carry_l1, first ? 0 : 1, cs.vm, a1, a2, l2_1);
    else
        block_extrema<false>(x, carry_b, cs.carry_l1, first ? 0 : 1, cs.vm, a1, a2, l2_1);

    // ---- four-way evaluation (Eq. (3)-(4)) and selection
    uint32_t m0 = a1, m1 = a2, m2 = a1, m3 = a2;
    if (first) {
        const int q0 = x[0];  // d[0] = q[0] at a tile start
        const int d1 = cnt >= 2 ? l2_1 : 0;  // q1 - 2 q0
        const int c0 = q0 - mu;
        const int c1 = cnt >= 2 ? l2_1 + mu : 0;
        m0 = max(uabs(q0), a1);
        m1 = max(max(uabs(q0), uabs(d1)), a2);
        m2 = max(uabs(c0), a1);
        m3 = max(max(uabs(c0), uabs(c1)), a2);
    }
    if (cnt == 0) m0 = m1 = m2 = m3 = 0;  // segments past the end of the field
    if (HB == 2) {
        m0 = max(m0, (uint32_t)__shfl_xor((int)m0, 1));
        m1 = max(m1, (uint32_t)__shfl_xor((int)m1, 1));
        m2 = max(m2, (uint32_t)__shfl_xor((int)m2, 1));
        m3 = max(m3, (uint32_t)__shfl_xor((int)m3, 1));
    }
    const uint32_t r0 = bitlen(m0), r1 = bitlen(m1), r2 = bitlen(m2), r3 = bitlen(m3);
    const uint32_t Ca = lane_group_sum<L>(h == 0 ? (uint32_t)HB * block_bytes(r0) : 0u);
    const uint32_t Cb = lane_group_sum<L>(h == 0 ? (uint32_t)HB * block_bytes(r1) : 0u);
    const uint32_t Cc = lane_group_sum<L>(h == 0 ? (uint32_t)HB * block_bytes(r2) : 0u) + 4u;
    const uint32_t Cd = lane_group_sum<L>(h == 0 ? (uint32_t)HB * block_bytes(r3) : 0u) + 4u;
    int best = 0;
    uint32_t C = Ca, r = r0;
    if (Cb < C) {
        best = 1;
        C = Cb;
        r = r1;
    }
    if (centre_ok) {
        if (Cc < C) {
            best = 2;
            C = Cc;
            r = r2;
        }
        if (Cd < C) {
            best = 3;
            C = Cd;
            r = r3;
        }
    }
    if (!tile_ok) {
        best = 0;
        C = 0;
        r = 0;
    }
    cs.order2 = best & 1;
    cs.cent = best >> 1;
    cs.r = r;
    cs.rbyte = first ? (r | (uint32_t)cs.order2 << 7 | (uint32_t)cs.cent << 6) : r;

    // ---- offsets: the lane's block inside the tile, the tile inside the wave
    const uint32_t S = block_bytes(r);  // this lane's words: 4 (1 + r) bytes
    const uint32_t pre = lane_run_incl_scan<L>(S, tl, L) - S;
    const int incl = wave_incl_scan(first ? (int)C : 0);
    cs.tile_excl = (uint32_t)incl - C;
    cs.wave_total = (uint32_t)__builtin_amdgcn_readlane(incl, 63);
    cs.blk_off = cs.tile_excl + 4u * (uint32_t)cs.cent + pre - (uint32_t)h * S + 4u * (uint32_t)h;
    if (lane == 0) sh.wave_total[slot][w] = cs.wave_total;
    lds_barrier();
    if (tid == 64) {
        uint32_t chunk_total = 0;
#pragma unroll
        for (int k = 0; k < W; k++) chunk_total += sh.wave_total[slot][k];
        publish_aggregate(a.flags, chunk, a.flag_epoch, chunk_total, false);
    }
    return cs;
}

// Residual codes and bit planes of one wave's segments into its staging area
// (word k of the lane's half h of a block at dword blk_off / 4 + HB k).
template <int HB>
__device__ __forceinline__ void cfg_stage(const ChunkState &cs, int (&B)[32], uint32_t *st)
{
    if (cs.vm != 0 && cs.first && cs.cent) st[cs.tile_excl >> 2] = (uint32_t)cs.mu;
    block_codes(B, cs.carry_l1, cs.first ? 0 : 1, cs.order2, cs.cent, cs.mu);
    const uint32_t keep = __builtin_bswap32(__builtin_bitreverse32(cs.vm));
    const uint32_t nwords = cs.r ? cs.r + 1 : 0;
    uint32_t *words = st + (cs.blk_off >> 2);
    for (uint32_t g = 0; __ballot(8 * g < nwords) != 0; g++) {
        uint32_t Rg[8];
#pragma unroll
        for (int rho = 0; rho < 8; rho++)
            Rg[rho] = pack_byte_g((uint32_t)B[7 - rho], (uint32_t)B[15 - rho], (uint32_t)B[23 - rho],
                                  (uint32_t)B[31 - rho], g);
        transpose8(Rg);
#pragma unroll
        for (int p = 0; p < 8; p++)
            if (8 * g + p < nwords) words[HB * (8 * g + p)] = Rg[p] & keep;
    }
}

// Tile geometry of a configuration for the compression pipeline: HB lanes
// per block, L lanes per tile (a wave's 64 segments hold 64 / L tiles).
template <int HB, int L>
struct TileCfg {
    static constexpr int kLanes = L, kWordStride = HB;
    template <int W, bool FEAT>
    static __device__ __forceinline__ ChunkState rates(const CompressArgs &a, const Resolved &R, uint64_t chunk,
                                                       int (&x)[32], int slot, CompressShared<W> &sh)
    {
        static_assert(!FEAT, "the configuration kernels run the full method");
        return cfg_rates<HB, L, W>(a, R, chunk, x, slot, sh);
    }
    template <bool FEAT>
    static __device__ __forceinline__ void stage(const ChunkState &cs, int (&B)[32], uint32_t *st)
    {
        cfg_stage<HB>(cs, B, st);
    }
    template <int W>
    static __device__ __forceinline__ bool wave_live(const CompressArgs &a, uint64_t chunk, int w)
    {
        return (chunk * W + (uint64_t)w) * 64 / L < a.ntiles;
    }
    template <int W>
    static __device__ __forceinline__ void store_rate(const CompressArgs &a, const ChunkState &cs, int w, int lane)
    {
        if (cs.vm != 0 && lane % HB == 0)
            ((g_u8 *)a.out)[kHeaderBytes + ((cs.chunk * W + (uint64_t)w) * 64 + lane) / HB] = (uint8_t)cs.rbyte;
    }
};

// Pipelined compressor of a tile configuration: compress_ctrl_kernel's
// pipeline (8 data waves, one control wave, persistent workgroups, chunks of
// 8 x 64 segments from the ticket counter) over the configuration's tiles.
// a.nchunks counts chunks of kCfgPipeChunkSegs segments.
template <int HB, int L>
__global__ __launch_bounds__(9 * 64) void compress_cfg_pipe_kernel(CompressArgs a)
{
    __shared__ CompressShared<8> sh;
    __shared__ __attribute__((aligned(16))) uint32_t inbuf[8 * kPipeInDwords];
    __shared__ __attribute__((aligned(16))) uint32_t stbuf[8 * kPipeOutDwords];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
    Resolved R;
    uint64_t A;
    int tslot;
    if (!pipe_start<9 * 64, 8>(a, sh, inbuf + w * kPipeInDwords, w, R, A, tslot)) return;
    if (w < 8)
        pipe2_run<false, 8, false, TileCfg<HB, L>>(a, R, sh, inbuf + w * kPipeInDwords,
                                                    stbuf + w * kPipeOutDwords, w, A, tslot);
    else
        ctrl_run<8>(a, R, sh, A, tslot);
}

// WV waves per workgroup, chunks of 64 WV segments (4 waves: a wider grid,
// which small fields need, and several workgroups per CU to hide the lookback
// and the tile loads; 16 in the lookback form of fields above 2^21 elements,
// whose chain the larger chunks halve twice).  PRESCAN: the chunk offsets come from
// dec_groups_kernel<64 WV / L, L / HB, HB>: chunk = workgroup, no lookback.
template <bool ALIGNED, int HB, int L, bool PRESCAN = false, int WV = kCfgDecWaves>
__global__ __launch_bounds__(WV * 64) void decompress_cfg_kernel(DecompressArgs a)
{
    __shared__ DecompressShared<WV> sh;
    __shared__ __attribute__((aligned(16))) uint32_t stage[WV * kCfgStageDwords];
    const int tid = threadIdx.x;
    const int w = tid >> 6;
    const int lane = tid & 63;
    const int tl = lane % L;
    const int h = tl % HB;

    // ---- header: as dec_header, with the configuration bits of this kernel
    const uint32_t *hw = reinterpret_cast<const uint32_t *>(a.cmp);
    const uint32_t h1 = hw[1];
    int hst = FSZ_OK;
    if (hw[0] != 0x315A5346u || (h1 & 0xFFFFu) != 1u || ((h1 >> 16) & 0xFFu) > 1u || ((h1 >> 24) & ~0x1Fu) != 0u ||
        ((h1 >> 24) & 0x1Cu) != a.cfg_flags)
        hst = FSZ_ERR_CORRUPT;
    else if (((uint64_t)hw[3] << 32 | hw[2]) != a.n)
        hst = FSZ_ERR_SIZE_MISMATCH;
    const bool indep = ((h1 >> 25) & 1u) != 0;  // flags bit 1: prediction restarts at every block
    const float E = __uint_as_float(hw[4]);
    const uint64_t total = (uint64_t)hw[7] << 32 | hw[6];
    if (hst == FSZ_OK && (!__builtin_isfinite(E) || !(E > 0.0f) || total > a.cmp_size || total < a.data0))
        hst = FSZ_ERR_CORRUPT;
    if (hst != FSZ_OK) {
        if (tid == 0 && blockIdx.x == 0) write_final(a.final, 0, hst, a.epoch);
        return;
    }
    int tslot = 0;
    GroupCursor gc;
    const uint64_t chunk = PRESCAN ? (uint64_t)blockIdx.x : next_ticket(a.ticket, a.nchunks, sh, tslot);
    if (chunk >= a.nchunks) return;

    // ---- steps 1-2: rate bytes -> block, tile and wave sizes
    const uint64_t seg0 = (chunk * WV + w) * 64;
    const uint64_t seg = seg0 + lane;
    const bool tile_ok = seg / L < a.ntiles;
    const uint64_t blk = seg / HB;
    const bool blk_ok = tile_ok && blk < a.nblocks;
    const bool first = tl == 0;
    const uint32_t rb = blk_ok ? a.cmp[kHeaderBytes + blk] : 0u;
    const bool bad = blk_ok && h == 0 && (first ? (rb & 0x20u) : (rb & 0xE0u)) != 0;
    const uint32_t head = (uint32_t)__shfl((int)rb, lane - tl);  // the tile's first rate byte
    const int order2 = tile_ok ? (int)((head >> 7) & 1u) : 0;
    const int cent = tile_ok ? (int)((head >> 6) & 1u) : 0;
    const uint32_t r = rb & 31u;
    const uint32_t S = block_bytes(r);  // this lane's words
    const uint32_t Z = lane_group_sum<L>(S) + 4u * (uint32_t)cent;
    const uint32_t pre = lane_run_incl_scan<L>(S, tl, L) - S;
    const uint32_t blk_rel = 4u * (uint32_t)cent + pre - (uint32_t)h * S;
    const int incl = wave_incl_scan(first ? (int)Z : 0);
    const uint32_t tile_excl = (uint32_t)incl - Z;
    const uint32_t wave_total = (uint32_t)__builtin_amdgcn_readlane(incl, 63);
    const bool wave_bad = __ballot(bad) != 0;
    if (lane == 0) {
        sh.wave_total[0][w] = wave_total;
        sh.wave_total[1][w] = wave_bad ? 1u : 0u;
    }
    uint64_t base = 0;
    if (PRESCAN) {
        gc.next = chunk >> a.group_shift;
        base = a.offsets[chunk];
        if (a.groups_scanned) {  // the groups hold running sums already
            const unsigned long long t = a.groups[gc.next];
            base += t & ~kGroupBad;
            gc.bad = (t & kGroupBad) != 0;
        } else {
            bool seen;
            const unsigned long long share = groups_share<WV * 64>(a, (uint32_t)gc.next, seen);
            const bool wave_seen = __ballot(seen) != 0;
            if (lane == 0) {
                sh.wave_prefix[w] = share;
                sh.wave_bad[w] = wave_seen ? 1u : 0u;
            }
        }
    }
    lds_barrier();
    uint32_t chunk_total = 0, wave_base = 0;
    bool any_bad = false;
#pragma unroll
    for (int k = 0; k < WV; k++) {
        if (k < w) wave_base += sh.wave_total[0][k];
        chunk_total += sh.wave_total[0][k];
        any_bad = any_bad || sh.wave_total[1][k] != 0;
    }
    if (PRESCAN) {
        if (!a.groups_scanned) {
#pragma unroll
            for (int k = 0; k < WV; k++) {
                base += sh.wave_prefix[k];
                gc.bad = gc.bad || sh.wave_bad[k] != 0;
            }
        }
        if (w == 0 && chunk == a.nchunks - 1) 
            finish_decode<false>(a, gc.bad || (a.groups[gc.next] & kGroupBad) != 0, base + chunk_total, total);
    } else {
        if (tid == 0) publish_aggregate(a.flags, chunk, a.flag_epoch, chunk_total, any_bad);
        if (w == 0) {
            const Prefix pre_c = lookback_wait(a.flags, chunk, a.flag_epoch, chunk_total, any_bad);
            if (lane == 0) {
                sh.base = pre_c.excl;
                if (chunk == a.nchunks - 1) {  // the sizes add up to the stream's total, padding is zero
                    bool good = !pre_c.err && a.data0 + pre_c.excl + chunk_total == total;
                    for (uint64_t k = kHeaderBytes + a.nblocks; good && k < a.data0; k++) good = a.cmp[k] == 0;
                    write_final(a.final, total, good ? (uint32_t)FSZ_OK : (uint32_t)FSZ_ERR_CORRUPT, a.epoch);
                }
            }
        }
        lds_barrier();
        base = sh.base;
    }
    if (any_bad || a.data0 + base + chunk_total > total || seg0 / L >= a.ntiles) return;

    // ---- steps 3-5: bit-unshuffle, inverse prediction, x' = (float)q * E
    const uint8_t *wave_data = a.cmp + a.data0 + base + wave_base;
    int mu = 0;
    if (cent) mu = (int)*reinterpret_cast<const uint32_t *>(wave_data + tile_excl);
    // the sign map folded into the magnitude planes, as in dec_decode: a
    // residual is x + sign (1 - 2^(8 G)) (mod 2^32)
    uint32_t code[32];
#pragma unroll
    for (int i = 0; i < 32; i++) code[i] = 0;
    const uint32_t rp = blk_ok ? r : 0;  // magnitude planes
    const uint32_t *words = reinterpret_cast<const uint32_t *>(wave_data + tile_excl + blk_rel) + h;
    const uint32_t sw = rp ? words[0] : 0u;  // the lane's half of the sign map
    uint32_t G = 0;
    for (uint32_t g = 0; __ballot(8 * g < rp) != 0; g++) {
        uint32_t Rg[8];
#pragma unroll
        for (int p = 0; p < 8; p++) Rg[p] = (8 * g + p < rp ? words[HB * (1 + 8 * g + p)] : 0u) ^ sw;
        transpose8(Rg);
        // Rg[rho] byte k = byte g of x of element 8k + 7 - rho
#pragma unroll
        for (int rho = 0; rho < 8; rho++) {
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint32_t sel = (0x03020100u & ~(0xFFu << (8 * g))) | ((4u + k) << (8 * g));
                code[8 * k + 7 - rho] = __builtin_amdgcn_perm(Rg[rho], code[8 * k + 7 - rho], sel);
            }
        }
        G = g + 1;
    }
    const uint32_t M = G < 4 ? 1u - (1u << (8 * G)) : 1u;  // 1 - 2^(8 G) mod 2^32
    uint32_t acc = 0;
#pragma unroll
    for (int i = 0; i < 32; i++) {
        const uint32_t ns = (uint32_t)((int)(sw << (31 - (i ^ 7))) >> 31);  // -sign
        acc += code[i] + (ns & M);
        code[i] = acc;  // first running sum inside the segment
    }
    // carries from the earlier lanes of the prediction run (the tile, or the
    // block when every block restarts)
    const int run = indep ? HB : L;
    const uint32_t start1 = lane_run_incl_scan<L>(acc, tl, run) - acc;
    uint32_t acc2 = 0;
#pragma unroll
    for (int i = 0; i < 32; i++) acc2 += code[i] + start1;
    const uint32_t start2 = lane_run_incl_scan<L>(acc2, tl, run) - acc2;
    float xo[32];
    {
        // the tile mean enters the start of the running sum that is the result
        const uint32_t s1 = start1 + (order2 ? 0u : (uint32_t)mu);
        uint32_t run2 = start2 + (order2 ? (uint32_t)mu : 0u);
#pragma unroll
        for (int i = 0; i < 32; i++) {
            const uint32_t d1 = code[i] + s1;  // first running sum with the carry
            run2 += d1;                        // second running sum
            xo[i] = (float)(int)(order2 ? run2 : d1) * E;
        }
    }
    // ---- write back through LDS with coalesced stores (the wave's 2048 elements)
    uint32_t *st = stage + w * kCfgStageDwords;
#pragma unroll
    for (int k = 0; k < 8; k++)
        *reinterpret_cast<float4 *>(st + lane * kStageRowDwords + 4 * k) =
            make_float4(xo[4 * k], xo[4 * k + 1], xo[4 * k + 2], xo[4 * k + 3]);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const uint64_t w0 = seg0 * 32;
    const bool fullw = w0 + 2048 <= a.n;
    if (ALIGNED) {
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int p = k * 64 + lane;
            const uint64_t e = w0 + 4ull * p;
            const f4 f = *reinterpret_cast<const f4 *>(st + (p >> 3) * kStageRowDwords + (p & 7) * 4);
            if (fullw || e + 4 <= a.n) {
                __builtin_nontemporal_store(f, reinterpret_cast<f4 *>(a.out + e));
            } else {
                if (e + 0 < a.n) a.out[e + 0] = f.x;
                if (e + 1 < a.n) a.out[e + 1] = f.y;
                if (e + 2 < a.n) a.out[e + 2] = f.z;
                if (e + 3 < a.n) a.out[e + 3] = f.w;
            }
        }
    } else {
        // 16-byte stores between the output's 16-byte boundaries, the elements
        // before the first and after the last one singly.  32 stores of 4 bytes
        // kept the workgroup's end waiting for their issue, and every addition
        // before them showed: 512^3 at offset 1, us per call, 32/4 150 with a
        // ticketed pre-pass, 164 with the group totals, 119 with these stores (115
        // aligned); 64/16 158, 173 and 125 (121).
        const uint32_t cnt = fullw ? 2048u : (uint32_t)(a.n - w0);
        const uint32_t head = min(align_head(a.out), cnt), nq = (cnt - head) / 4;  // w0 is a multiple of 2048
        const uint32_t tail = head + 4 * nq;
        g_f32 *out = (g_f32 *)a.out + w0;
        auto staged = [&](uint32_t p) { return __uint_as_float(st[(p >> 5) * kStageRowDwords + (p & 31)]); };
        if ((uint32_t)lane < head) out[lane] = staged(lane);
        if ((uint32_t)lane < cnt - tail) out[tail + lane] = staged(tail + lane);
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const uint32_t q = k * 64 + lane, p = head + 4 * q;
            if (q < nq) {
                const f4 f = {staged(p), staged(p + 1), staged(p + 2), staged(p + 3)};
                __builtin_nontemporal_store(f, (g_f4 *)(out + p));
            }
        }
    }
}

// Workgroups of a persistent grid: enough to fill every CU at the kernel's
// occupancy, never more than there are chunks.
template <typename K>
static unsigned persistent_grid(K kernel, uint64_t nchunks, int threads = kThreads)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || cus <= 0 ||
        per_cu <= 0) {
        cus = 256;
        per_cu = 2;
    }
    const uint64_t g = (uint64_t)cus * (uint64_t)per_cu * (uint64_t)tuning().grid_factor;
    return (unsigned)(nchunks < g ? nchunks : g);
}

// Enqueues the offsets pre-pass for chunks of TPC tiles and names its results
// in a: `words` holds kMaxGroupWords group totals, then an offset per chunk.
template <int TPC, int T = kBlocksPerTile, int HB = 1>
static hipError_t launch_dec_groups(DecompressArgs &a, unsigned long long *words, bool scan, hipStream_t s)
{
    static_assert(TPC % kGroupTilesPerThread == 0, "a chunk starts at a thread's first tile");
    const uint32_t passes = group_passes(a.tile_end);
    const uint64_t ngroups = a.tile_end ? ceil_div(a.tile_end, (uint64_t)kGroupTiles * passes) : 1;
    a.groups = words;
    a.offsets = words + kMaxGroupWords;
    a.group_shift = (uint32_t)__builtin_ctz(kGroupTiles / TPC * passes);
    hipLaunchKernelGGL((dec_groups_kernel<T, HB>), dim3((unsigned)ngroups), dim3(kGroupThreads), 0, s, a,
                       words + kMaxGroupWords, words, passes, (uint32_t)__builtin_ctz(TPC));
    a.groups_scanned = scan;
    if (scan) hipLaunchKernelGGL(dec_groups_scan_kernel, dim3(1), dim3(512), 0, s, words, (uint32_t)ngroups);
    return hipGetLastError();
}

template <bool ALIGNED, bool RANGE, bool PREZERO>
static hipError_t launch_decompress_persistent(const DecompressArgs &a, hipStream_t s)
{
    static const unsigned cap = persistent_grid(decompress_kernel<ALIGNED, 8, RANGE, PREZERO>, ~0ull, 512);
    const uint64_t chunks = a.nchunks - a.chunk_begin;
    hipLaunchKernelGGL((decompress_kernel<ALIGNED, 8, RANGE, PREZERO>), dim3((unsigned)(chunks < cap ? chunks : cap)),
                       dim3(512), 0, s, a);
    return hipGetLastError();
}

// Chunks of tpc tiles that hold the decoded tiles, counted from the field's
// first tile or from the first decoded one.  An empty decode still has one, to
// report the outcome: the one that ends where its data would start.
static void chunk_span(DecompressArgs &a, uint64_t tpc, bool from_begin)
{
    const uint64_t t0 = from_begin ? 0 : a.tile_begin;
    const uint64_t t1 = from_begin ? a.tile_end - a.tile_begin : a.tile_end;
    a.chunk_begin = (t1 > t0 ? t0 : t1 ? t1 - 1 : 0) / tpc;
    a.nchunks = t1 > t0 ? ceil_div(t1, tpc) : a.chunk_begin + 1;
}

template <bool ALIGNED, int W, bool RANGE, int OFF, bool PREZERO = false>
static hipError_t launch_decompress_direct(const DecompressArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL((decompress_direct_kernel<ALIGNED, W, RANGE, OFF, PREZERO>),
                       dim3((unsigned)(a.nchunks - a.chunk_begin)), dim3(W * 64), 0, s, a);
    return hipGetLastError();
}

template <bool ALIGNED, bool RANGE, bool PREZERO = false>
static hipError_t launch_decompress_t(const DecompressArgs &a, unsigned long long *words, hipStream_t s)
{
    DecompressArgs p = a;
    const uint64_t tiles = a.tile_end - a.tile_begin;
    if (decode_by_prefix(a.tile_begin, a.tile_end)) {
        // chunks of 4 waves spread small decodes wider; from 2^21 elements
        // on 8 waves halve the reads of the rate bytes (2^21 GRF 7.4 against
        // 7.9 us, 2^22 9.9 against 9.0)
        const bool wide = tiles * kTile > (1ull << 21);
        chunk_span(p, (uint64_t)kTilesPerWave * (wide ? 8 : 4), true);
        return wide ? launch_decompress_direct<ALIGNED, 8, RANGE, kByPrefix, PREZERO>(p, s)
                    : launch_decompress_direct<ALIGNED, 4, RANGE, kByPrefix, PREZERO>(p, s);
    }
    const bool direct = !PREZERO && tiles * kTile < tuning().dec_direct_below;
    const hipError_t e = direct ? launch_dec_groups<kTilesPerWave * 4>(p, words, false, s)
                                : launch_dec_groups<kTilesPerWave * 8>(p, words, false, s);
    if (e != hipSuccess) return e;
    chunk_span(p, (uint64_t)kTilesPerWave * (direct ? 4 : 8), false);
    if (direct) return launch_decompress_direct<ALIGNED, 4, RANGE, kByGroupsOnce>(p, s);
    return launch_decompress_persistent<ALIGNED, RANGE, PREZERO>(p, s);
}

hipError_t launch_decompress(const DecompressArgs &a, unsigned long long *words, bool out_aligned16, bool range,
                             hipStream_t s)
{
    if (range)
        return out_aligned16 ? launch_decompress_t<true, true>(a, words, s)
                             : launch_decompress_t<false, true>(a, words, s);
    return out_aligned16 ? launch_decompress_t<true, false>(a, words, s)
                         : launch_decompress_t<false, false>(a, words, s);
}

// +0.0 into out[0, n): 16-byte nontemporal stores from the first 16-byte
// boundary, 4-byte stores for the ragged ends.
__global__ __launch_bounds__(256) void fill_zero_kernel(float *out, uint64_t n)
{
    const uint64_t head = ((16u - (reinterpret_cast<uintptr_t>(out) & 15u)) & 15u) / 4u;
    const uint64_t h = head < n ? head : n;
    const uint64_t nv = (n - h) / 4;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    f4 *v = reinterpret_cast<f4 *>(out + h);
    for (uint64_t i = t; i < nv; i += stride) __builtin_nontemporal_store(f4{0.0f, 0.0f, 0.0f, 0.0f}, v + i);
    if (t < h) out[t] = 0.0f;
    const uint64_t tail = h + 4 * nv;
    if (t < n - tail) out[tail + t] = 0.0f;
}

hipError_t launch_decompress_prezero(const DecompressArgs &a, unsigned long long *words, bool out_aligned16,
                                     hipStream_t s)
{
    if (a.n) {
        const uint64_t want = ceil_div(a.n, 4ull * 256);
        const unsigned grid = (unsigned)(want < 4096 ? want : 4096);
        hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(256), 0, s, a.out, a.n);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return out_aligned16 ? launch_decompress_t<true, false, true>(a, words, s)
                         : launch_decompress_t<false, false, true>(a, words, s);
}

template <typename K>
static hipError_t launch_pipe(K kernel, unsigned cap, int waves, const CompressArgs &a, int data_waves, hipStream_t s)
{
    // the pipeline's chunks are 8 tiles per data wave
    CompressArgs p = a;
    p.nchunks = p.ntiles ? ceil_div(p.ntiles, (uint64_t)kTilesPerWave * data_waves) : 1;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(p.nchunks < cap ? p.nchunks : cap)), dim3(waves * 64), 0, s, p);
    return hipGetLastError();
}

#define FSZ_LAUNCH_PIPE(K, WAVES, DATA)                                                \
    {                                                                                  \
        static const unsigned cap = persistent_grid(K, ~0ull, (WAVES) * 64);           \
        return launch_pipe(K, cap, WAVES, a, DATA, s);                                 \
    }

hipError_t launch_compress(const CompressArgs &a, hipStream_t s)
{
    if (a.features != kFeaturesAll)  // the ablation's feature subsets
        FSZ_LAUNCH_PIPE(compress_pipe2_kernel<8>, 8, 8)
    // 11 data waves and a control wave; fewer where the smaller workgroup's
    // start and the finer spread count for more (4 / 8 / 11 data waves in us
    // per call, each with the same range pass: 2^14 9.8 / 10.5 / -, 2^18 10.8 / 12.1 / -,
    // 2^20 13.3 / 13.6 / 16.0, 2^21 17.6 / 15.3 / -, 2^22 - / 22.3 / 22.7, 6 M
    // - / 26.5 / 26.9, 2^23 - / 30.9 / 30.3, 2^25 - / 76.9 / 74.5)
    // A field without a range pass (self_range) takes the least that holds it.
    if (a.n >= (1ull << 23)) FSZ_LAUNCH_PIPE(compress_ctrl_kernel<11>, 12, 11)
    if (a.n <= (a.self_range ? 4 * kWaveElems : 1ull << 20)) FSZ_LAUNCH_PIPE(compress_ctrl_kernel<4>, 5, 4)
    FSZ_LAUNCH_PIPE(compress_ctrl_kernel<8>, 9, 8)
}

hipError_t launch_compress_naive(const CompressArgs &a, const NaiveTables &t, bool in_aligned16, hipStream_t s)
{
    const unsigned grid = (unsigned)a.nchunks;
    for (int v = 0; v < 4; v++) {
        if (in_aligned16)
            hipLaunchKernelGGL(naive_eval_kernel<true>, dim3(grid), dim3(kThreads), 0, s, a, t, v);
        else
            hipLaunchKernelGGL(naive_eval_kernel<false>, dim3(grid), dim3(kThreads), 0, s, a, t, v);
    }
    if (in_aligned16)
        hipLaunchKernelGGL(naive_encode_kernel<true>, dim3(grid), dim3(kThreads), 0, s, a, t);
    else
        hipLaunchKernelGGL(naive_encode_kernel<false>, dim3(grid), dim3(kThreads), 0, s, a, t);
    return hipGetLastError();
}

// Tile configurations (Sec. VI-C): (B, T) -> (HB, L) = (B / 32, T B / 32).
template <bool ALIGNED, int WV>
static hipError_t launch_decompress_cfg_w(const DecompressArgs &a, int block, int tile_blocks, hipStream_t s)
{
    const dim3 grid((unsigned)a.nchunks), threads(WV * 64);
    const int key = block * 100 + tile_blocks;
    switch (key) {
    case 3204: hipLaunchKernelGGL((decompress_cfg_kernel<ALIGNED, 1, 4, false, WV>), grid, threads, 0, s, a); break;
    case 3208: hipLaunchKernelGGL((decompress_cfg_kernel<ALIGNED, 1, 8, false, WV>), grid, threads, 0, s, a); break;
    case 3216: hipLaunchKernelGGL((decompress_cfg_kernel<ALIGNED, 1, 16, false, WV>), grid, threads, 0, s, a); break;
    case 6404: hipLaunchKernelGGL((decompress_cfg_kernel<ALIGNED, 2, 8, false, WV>), grid, threads, 0, s, a); break;
    case 6408: hipLaunchKernelGGL((decompress_cfg_kernel<ALIGNED, 2, 16, false, WV>), grid, threads, 0, s, a); break;
    case 6416: hipLaunchKernelGGL((decompress_cfg_kernel<ALIGNED, 2, 32, false, WV>), grid, threads, 0, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Lookback form: a.nchunks counts chunks of 64 cfg_dec_lookback_waves(n) segments.
template <bool ALIGNED>
static hipError_t launch_decompress_cfg_t(const DecompressArgs &a, int block, int tile_blocks, hipStream_t s)
{
    return cfg_dec_lookback_waves(a.n) == kCfgDecWideWaves
               ? launch_decompress_cfg_w<ALIGNED, kCfgDecWideWaves>(a, block, tile_blocks, s)
               : launch_decompress_cfg_w<ALIGNED, kCfgDecWaves>(a, block, tile_blocks, s);
}

// Persistent workgroups of 8 data
// waves and a control wave, chunks of kCfgPipeChunkSegs segments.
template <int HB, int L>
static hipError_t launch_compress_cfg_pipe_t(const CompressArgs &a, hipStream_t s)
{
    static const unsigned cap = persistent_grid(compress_cfg_pipe_kernel<HB, L>, ~0ull, 9 * 64);
    hipLaunchKernelGGL((compress_cfg_pipe_kernel<HB, L>), dim3((unsigned)(a.nchunks < cap ? a.nchunks : cap)),
                       dim3(9 * 64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_compress_cfg(const CompressArgs &a, int block, int tile_blocks, hipStream_t s)
{
    CompressArgs p = a;
    p.nchunks = a.n ? ceil_div(ceil_div(a.n, (uint64_t)kBlock), (uint64_t)kCfgPipeChunkSegs) : 1;
    switch (block * 100 + tile_blocks) {
    case 3204: return launch_compress_cfg_pipe_t<1, 4>(p, s);
    case 3208: return launch_compress_cfg_pipe_t<1, 8>(p, s);
    case 3216: return launch_compress_cfg_pipe_t<1, 16>(p, s);
    case 6404: return launch_compress_cfg_pipe_t<2, 8>(p, s);
    case 6408: return launch_compress_cfg_pipe_t<2, 16>(p, s);
    case 6416: return launch_compress_cfg_pipe_t<2, 32>(p, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_decompress_cfg(const DecompressArgs &a, int block, int tile_blocks, bool out_aligned16,
                                 hipStream_t s)
{
    return out_aligned16 ? launch_decompress_cfg_t<true>(a, block, tile_blocks, s)
                         : launch_decompress_cfg_t<false>(a, block, tile_blocks, s);
}

// Offsets pre-pass (chunks of kCfgDecChunkSegs segments = kCfgDecChunkSegs / L
// tiles), then one chunk per workgroup without lookback.
template <bool ALIGNED, int HB, int L>
static hipError_t launch_decompress_cfg_prescan_t(const DecompressArgs &a, unsigned long long *words, hipStream_t s)
{
    DecompressArgs p = a;
    // From 2^26 elements on a small launch turns the group totals into running
    // sums, so that no workgroup adds them up (512^3 from a cold cache, REL 1e-3,
    // 32/4 138 against 156 us, 64/16 147 / 157; 25 M elements 37.3 / 37.0, 40.9 /
    // 40.7).  That brings large fields back to where a pre-pass with tickets and
    // a lookback over the totals had them (135 us), which cost smaller ones more.
    const hipError_t e = launch_dec_groups<kCfgDecChunkSegs / L, L / HB, HB>(p, words, a.n >= (1ull << 26), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((decompress_cfg_kernel<ALIGNED, HB, L, true>), dim3((unsigned)a.nchunks),
                       dim3(kCfgDecWaves * 64), 0, s, p);
    return hipGetLastError();
}

template <bool ALIGNED>
static hipError_t launch_decompress_cfg_prescan_a(const DecompressArgs &a, unsigned long long *words, int block,
                                                  int tile_blocks, hipStream_t s)
{
    switch (block * 100 + tile_blocks) {
    case 3204: return launch_decompress_cfg_prescan_t<ALIGNED, 1, 4>(a, words, s);
    case 3208: return launch_decompress_cfg_prescan_t<ALIGNED, 1, 8>(a, words, s);
    case 3216: return launch_decompress_cfg_prescan_t<ALIGNED, 1, 16>(a, words, s);
    case 6404: return launch_decompress_cfg_prescan_t<ALIGNED, 2, 8>(a, words, s);
    case 6408: return launch_decompress_cfg_prescan_t<ALIGNED, 2, 16>(a, words, s);
    case 6416: return launch_decompress_cfg_prescan_t<ALIGNED, 2, 32>(a, words, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_decompress_cfg_prescan(const DecompressArgs &a, unsigned long long *words, int block,
                                         int tile_blocks, bool out_aligned16, hipStream_t s)
{
    return out_aligned16 ? launch_decompress_cfg_prescan_a<true>(a, words, block, tile_blocks, s)
                         : launch_decompress_cfg_prescan_a<false>(a, words, block, tile_blocks, s);
}

constexpr size_t kLdsPerCu = 160 * 1024;

// Dynamic LDS that caps resident workgroups per CU at `groups` (0 = none);
// returns false when the cap needs more LDS per workgroup than allowed or
// would change nothing.
template <typename K>
static bool batch_lds_pad(K kernel, int groups, size_t *pad)
{
    *pad = 0;
    if (groups <= 0) return true;
    hipFuncAttributes attr{};
    int dev = 0, max_lds = 0;
    if (hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(kernel)) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return false;
    const size_t per = kLdsPerCu / (size_t)groups;
    const size_t want = per > attr.sharedSizeBytes ? (per - attr.sharedSizeBytes) / 256 * 256 : 0;
    if (want == 0) return false;  // the kernel's own LDS already allows no more than `groups`
    if (attr.sharedSizeBytes + want > (size_t)max_lds) return false;
    // the pad must make the next workgroup not fit
    if ((size_t)(groups + 1) * (attr.sharedSizeBytes + want) <= kLdsPerCu) return false;
    *pad = want;
    return true;
}

template <int W, bool LDSJOBS>
static hipError_t launch_batch_pipe(const BatchArgs &b, hipStream_t s)
{
    static const unsigned cap = persistent_grid(batch_pipe_kernel<W, LDSJOBS>, ~0ull, (W + 1) * 64);
    const unsigned grid = (unsigned)(b.total_chunks < cap ? b.total_chunks : cap);
    hipLaunchKernelGGL((batch_pipe_kernel<W, LDSJOBS>), dim3(grid), dim3((W + 1) * 64), 0, s, b);
    return hipGetLastError();
}

static hipError_t launch_batch_compress(const BatchArgs &b, hipStream_t s)
{
    const bool lds = b.njobs <= kPipeLdsJobs;
    if (b.waves == 11) return lds ? launch_batch_pipe<11, true>(b, s) : launch_batch_pipe<11, false>(b, s);
    if (b.waves == 4) return lds ? launch_batch_pipe<4, true>(b, s) : launch_batch_pipe<4, false>(b, s);
    return lds ? launch_batch_pipe<8, true>(b, s) : launch_batch_pipe<8, false>(b, s);
}

template <bool ALIGNED, int W>
static hipError_t launch_batch_decompress(const BatchArgs &b, int groups, hipStream_t s)
{
    size_t pad = 0;
    if (!batch_lds_pad(batch_dec_kernel<ALIGNED, W>, groups, &pad)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((batch_dec_kernel<ALIGNED, W>), dim3((unsigned)(b.njobs + b.dec.total_chunks)),
                       dim3(W * 64), pad, s, b);
    return hipGetLastError();
}

template <int W>
static hipError_t launch_batch_w(const BatchArgs &b, bool aligned_out, int groups, hipStream_t s)
{
    hipError_t e = hipSuccess;
    if (b.dec.njobs) {
        e = aligned_out ? launch_batch_decompress<true, W>(b, groups, s)
                          : launch_batch_decompress<false, W>(b, groups, s);
    } else {
        hipLaunchKernelGGL(batch_stats_final_kernel, dim3(b.njobs), dim3(kStatsThreads), 0, s, b);
        e = hipGetLastError();
    }
    if (e == hipSuccess && b.njobs)
        e = launch_batch_compress(b, s);
    return e;
}

bool batch_shape_supported(const BatchShape &shape)
{
    if (shape.groups_per_cu < 0 || shape.groups_per_cu > 8) return false;
    size_t pad = 0;
    switch (shape.waves) {
    case 2: return batch_lds_pad(batch_dec_kernel<true, 2>, shape.groups_per_cu, &pad);
    case 4: return batch_lds_pad(batch_dec_kernel<true, 4>, shape.groups_per_cu, &pad);
    case 8: return batch_lds_pad(batch_dec_kernel<true, 8>, shape.groups_per_cu, &pad);
    default: return false;
    }
}

hipError_t launch_batch(const BatchArgs &b, bool aligned_out, const BatchShape &shape, hipStream_t s)
{
    // workgroups loop over segments; enough of them to clear the flags
    uint64_t grid = b.total_segs < 2048 ? b.total_segs : 2048;
    const uint64_t clear = ceil_div(b.nflags, kStatsThreads);
    if (grid < clear) grid = clear < kStatsMaxBlocks ? clear : kStatsMaxBlocks;
    grid += b.dec.group_wgs;
    hipLaunchKernelGGL(batch_stats_kernel, dim3((unsigned)grid), dim3(kStatsThreads), 0, s, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    switch (shape.waves) {
    case 2: return launch_batch_w<2>(b, aligned_out, shape.groups_per_cu, s);
    case 4: return launch_batch_w<4>(b, aligned_out, shape.groups_per_cu, s);
    case 8: return launch_batch_w<8>(b, aligned_out, shape.groups_per_cu, s);
    default: return hipErrorInvalidValue;
    }
}

// ------------------------------------------------------------------ allocation-free compression
//
// fsz_compress_noalloc_async keeps its chunk flags, ticket and range-pass
// partials in one fixed device array instead of the per-stream workspace.
// Layout: [0, 16 KiB) range-pass partials, then the field stats (16 bytes)
// and the ticket (8 bytes, 128 bytes further), then from byte 16640 the flag
// words (kFlagStride words per chunk) of the smallest chunk any compress
// kernel uses (8 tiles, 2048 elements), enough for n <= kNoAllocMaxElements.
// Each call clears the flag words it uses and the ticket with a fill kernel
// (no memset node, so the call may be captured in a graph and replayed).
constexpr uint64_t kNoAllocMaxElements = 1ull << 30;
constexpr size_t kNoAllocStatsOff = sizeof(StatsPartial) * kStatsMaxBlocks;
constexpr size_t kNoAllocTicketOff = kNoAllocStatsOff + 128;
constexpr size_t kNoAllocFlagsOff = kNoAllocStatsOff + 256;
constexpr uint64_t kNoAllocMaxFlags = kNoAllocMaxElements / ((uint64_t)kTile * kTilesPerWave);
constexpr size_t kNoAllocScratchBytes = kNoAllocFlagsOff + kNoAllocMaxFlags * kFlagStride * sizeof(unsigned long long);
static_assert(kNoAllocScratchBytes == 16640 + 32 * 524288, "scratch layout");

static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

// Device address of `scratch` on the current device, looked up once per
// device (each device holds its own copy of the array).  Host code passes
// this address, never the array's name, to kernels.
static unsigned char *scratch_address(int dev)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static unsigned char *addr[kMaxDevices] = {};
    if (dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> g(mu);
    if (!addr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
        addr[dev] = static_cast<unsigned char *>(ptr);
    }
    return addr[dev];
}

__global__ __launch_bounds__(256) void zero_words_kernel(unsigned long long *p, uint64_t count,
                                                         unsigned long long *one)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) p[i] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) *one = 0;
}

fsz_status compress_noalloc(const float *d_in, uint64_t n, int mode, double value, const fsz_stats *d_stats,
                            void *d_out, uint64_t cap, fsz_result *d_result, hipStream_t s)
{
    if (n > kNoAllocMaxElements) return FSZ_ERR_TOO_LARGE;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return FSZ_ERR_DEVICE;
    unsigned char *base = scratch_address(dev);
    if (!base) return FSZ_ERR_DEVICE;
    StatsPartial *partials = reinterpret_cast<StatsPartial *>(base);
    fsz_stats *stats = reinterpret_cast<fsz_stats *>(base + kNoAllocStatsOff);
    unsigned long long *ticket = reinterpret_cast<unsigned long long *>(base + kNoAllocTicketOff);
    unsigned long long *flags = reinterpret_cast<unsigned long long *>(base + kNoAllocFlagsOff);

    CompressArgs a{};
    a.x = d_in;
    a.n = n;
    a.ntiles = ceil_div(n, kTile);
    a.nblocks = ceil_div(n, kBlock);
    a.nchunks = a.ntiles ? ceil_div(a.ntiles, kTilesPerChunk) : 1;
    a.data0 = kHeaderBytes + pad16(a.nblocks);
    a.out = static_cast<uint8_t *>(d_out);
    a.capacity = cap;
    a.value = value;
    a.mode = mode;
    a.features = kFeaturesAll;
    a.epoch = 1;       // flags start cleared at every call, so one epoch serves
    a.flag_epoch = 1;  // every call
    a.flags = flags;
    a.ticket = ticket;
    a.final = d_result;
    const uint64_t nflags = (a.ntiles ? ceil_div(a.ntiles, kTilesPerWave) : 1) * kFlagStride;  // words
    const uint64_t want = ceil_div(nflags, 256);
    const unsigned grid = (unsigned)(want < 1024 ? want : 1024);
    hipLaunchKernelGGL(zero_words_kernel, dim3(grid), dim3(256), 0, s, flags, nflags, ticket);
    if (hipGetLastError() != hipSuccess) return FSZ_ERR_DEVICE;
    if (!d_stats) {
        const StatsArgs sa{d_in, n, stats, partials};
        if (launch_stats_partials(sa, &a.nparts, s) != hipSuccess) return FSZ_ERR_DEVICE;
        a.partials = partials;
    }
    a.stats = d_stats;
    if (launch_compress(a, s) != hipSuccess) return FSZ_ERR_DEVICE;
    return FSZ_OK;
}

}  // namespace fsz
