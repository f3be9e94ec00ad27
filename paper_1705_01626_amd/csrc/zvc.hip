// Zero-value compression (ZVC) for AMD gfx950 (wave64): kernels and C ABI.
//
// The operation is the one of the paper's section 5.1: one 32-bit presence mask
// per 32 consecutive elements plus the non-zero elements packed in order.  The
// paper builds it as a fixed-function pipeline beside the memory controllers
// (section 5.2); this file is a GPU kernel design instead:
//
//   * one pass over the input.  A workgroup owns a tile of 16 to 64 KB of input;
//     each lane loads one dword at a time (a wave instruction covers 256
//     contiguous bytes), so the 64-lane ballot of the zero test is two finished
//     masks and its mbcnt the packed position of the lane's element (the GPU
//     form of the paper's per-sector prefix sum over mask bits);
//   * the offset of a tile's first kept element in the packed stream -- where
//     the next mask goes, a serial chain in the paper's hardware -- is a
//     device-wide exclusive scan of per-tile counts done in the same pass:
//     every tile publishes its count, every 512th tile a running prefix, and a
//     tile adds the counts between the nearest published prefix and itself;
//   * kept elements are staged by each wave in an LDS queue in packed order and
//     leave as whole 128-byte lines; masks leave as one contiguous run per wave.
//
// Decompression: where a span's stored elements start depends on the masks
// alone, so a small pre-pass over the masks computes it for every 32 masks; the
// expand kernel's waves then work independently: each stages its packed run in
// LDS with aligned 16-byte loads and rebuilds 16 bytes of output per lane from
// "bit ? next stored element : zero".  Below some tens of megabytes a tensor decodes in one launch that
// uses the encoder's scan instead of the pre-pass, and the smallest without either.
//
// Three variants share these kernels: a fused ReLU + ZVC encoder
// (pre-activations in, stream of ReLU(x) out), an encoder that writes into a
// buffer below the worst case and never past it (section 9: streams kept in GPU
// memory), and the paper's own stream order (a group's mask, then its non-zeros)
// in independently decodable windows of 1 KB to 64 KB with an offset table.

#include "zvc.h"

#include <hip/hip_runtime.h>

#include <mutex>
#include <tuple>
#include <utility>
#include <cstdint>
#include <cstring>
#include <type_traits>

namespace {

// ------------------------------------------------------------------ geometry
constexpr int kThreads = 256;                 // 4 waves of 64 lanes
constexpr int kWaveSize = 64;
constexpr int kWaves = kThreads / kWaveSize;
constexpr int kFinishLanes = 64;              // arrival counters, one 128-byte line each
constexpr size_t kHeaderBytes = 256 + 128 * (kFinishLanes + 1);  // header, then the scan state
constexpr int kMinLoads = 4;                  // smallest tile: 16 KB (sizes the workspace)
constexpr int kStageLoads = 4;                // 16-byte loads a wave stages through LDS at a time
constexpr int kBlockShift = 9;                // one running prefix is published per 512 tiles (or more, see block_shift_of)
constexpr int kMaxDevices = 64;                // GPUs per process that per-GPU host state is kept for
constexpr unsigned kDefaultPatience = 2000;   // polls a waiting tile makes before it computes a missing count itself
constexpr int kPollSleep = 8;                 // s_sleep units (64 clocks each) between polls

// The decoder's tile: LOADS 16-byte stores per lane, 256 * 16 * LOADS bytes of output.
template <int W, int LOADS>
struct Geometry {
    static constexpr int kElemsPerLane = 16 / W;                 // per 16-byte store: 4 | 8
    static constexpr int kLanesPerGroup = 32 / kElemsPerLane;    // lanes covering one mask: 8 | 4
    static constexpr int kGroupsPerLoad = kWaveSize / kLanesPerGroup;  // masks per KB of output: 8 | 16
    // per-wave LDS staging buffer: kStageLoads wave-loads, 16 bytes so that the slice can mirror the
    // run's alignment, and up to 31 elements that a shifted piece stages without writing them
    static constexpr int kStageSteps = LOADS / kStageLoads;
    static constexpr int kWaveStageBytes = kStageLoads * kWaveSize * 16 + 16 + 32 * W;
    // decompress_kernel: zeros, the waves' slices, a sum per wave
    static constexpr unsigned kDecodeLdsBytes = 16 + kWaves * kWaveStageBytes + 4 * kWaves;
    static_assert(LOADS % kStageLoads == 0, "tile is staged in whole steps");
};

// The encoder's tile.  A wave reads its part of the tensor one dword per lane
// (a chunk: 256 bytes, 64 fp32 or 128 16-bit elements, 2 or 4 masks), CH chunks
// per wave, WV waves per tile (the workgroup): WV x CH / 4 KB.  With one
// element (or one pair) per lane a ballot of the zero test is two masks as they
// stand and its mbcnt is the packed position, so a chunk costs a handful of
// vector instructions.  Streaming 4-byte accesses measure as fast as 16-byte
// ones on this memory system (each wave instruction still covers whole
// 128-byte lines).
constexpr int kChunkBytes = 4 * kWaveSize;
constexpr int kStepChunks = 8;                // chunks a wave stages between two flushes: 2 KB of input
template <int W, int CH, int WV>
struct EncoderGeometry {
    static constexpr int kChunkElems = kChunkBytes / W;          // 64 | 128
    static constexpr int kChunkGroups = kChunkElems / 32;        // masks per chunk: 2 | 4
    static constexpr int kWaveElems = CH * kChunkElems;
    static constexpr int kWaveGroups = CH * kChunkGroups;
    static constexpr int kTileBytes = WV * CH * kChunkBytes;
    static constexpr int kTileElems = WV * kWaveElems;
    static constexpr int kTileGroups = WV * kWaveGroups;
    static constexpr int kSteps = CH / kStepChunks;
    static constexpr int kMaskRegs = (kWaveGroups + kWaveSize - 1) / kWaveSize;
    static constexpr int kStepGroups = kStepChunks * kChunkGroups;
    // the most a step can add to the wave's queue (windowed stream: its masks too)
    static constexpr int kStepMaxBytes = kStepChunks * kChunkBytes + 4 * kStepGroups;
    // A wave's LDS queue.  What is in it when the tile learns where its run
    // begins has cost the tile no time; what does not fit waits for that moment.
    // Room for half the wave's input (a tensor that is at most half non-zero is
    // staged whole before the scan ends) plus a little, never less than a
    // carried-over partial line plus a step.  (More workgroups per CU with a
    // smaller queue measure the same or worse.)
    // The smallest tile's queues hold all of it (eight workgroups still fit a CU): no step waits
    // for the scan, however dense the tensor is (4 MB fp32 without a zero: 6.20 -> 5.52 us).
    static constexpr bool kHoldsAll = CH == 16;
    static constexpr int kQueueBytes =
        kHoldsAll ? CH * kChunkBytes + 4 * kWaveGroups :
        CH == 64 ? 8704 : (CH * kChunkBytes / 2 > kStepMaxBytes ? CH * kChunkBytes / 2 : kStepMaxBytes) + 256;
    static_assert(kQueueBytes >= 128 + kStepMaxBytes, "a step always fits behind a carried-over partial line");
    static_assert(CH % kStepChunks == 0, "a wave's chunks are staged in whole steps");
    static_assert(kTileElems <= 0x4000, "tile totals fit the arrival word and the scan's");
};

// Workspace header.  Lives at the start of the caller's workspace.
struct WsHeader {
    unsigned long long patience_plus_one;   // 0: default; else polls before a waiting tile helps itself, plus one
    unsigned long long scan_word;  // the scan's calls so far, see ScanCalls
    unsigned long long size_word;  // compressed size for zvc_offload's read-back
    unsigned long long helped;     // predecessor counts computed by a waiting tile since the workspace's init
    unsigned long long helped_here;   // not 0: a waiting tile of the present call has computed a predecessor's count
    unsigned long long wide_calls;    // so far, see ScanCalls
    unsigned long long pad[26];
    // The scan's running prefixes, and arrival counters, zero between calls.  Decoder's pre-pass: the
    // workgroup that completes a counter bumps finish_top, the one that completes finish_top is
    // the last.  Count-only pass: the same, with `sum` collecting the counts.
    // One counter per 128-byte line keeps the atomics on one address (about
    // 11 ns each) far apart in time.
    struct alignas(128) Line {
        unsigned value;
        unsigned pad;
        unsigned long long sum;
        unsigned long long prefix[14];
    } finish[kFinishLanes], finish_top;
};
static_assert(sizeof(WsHeader) == kHeaderBytes, "header size");

// Scan state.
//   counts   : a word per tile, behind the header: the call's number, a bit that the tile itself wrote it, and the
//              tile's own count of kept elements (15 bits).  32 bits with the number's lowest 15, or (a
//              wide call) 64 with all that matter;
//   prefixes : a 64-bit word per block of tiles, in the header's lines: a tag of two bits, 1 and 2 in turn
//              from call to call, and the kept elements in all tiles up to and including the block's last.
// A count holds if it has the call's number, so nothing that earlier calls left there has to be cleared,
// neither by them nor by a later one, which may be a tiny one or have been told of fewer bytes than they.  15 bits tell apart
// the calls of two terms of 2^14 calls; what lies behind the tiles of a term's last call may be older than that in the term
// after.  A call that has more tiles than that one, and than every such call since, is a wide one.  Its
// counts have the number of wide calls so far, of which there cannot be 2^45.  Neither kind passes for the other, nor what the
// decoder's pre-pass leaves in the same bytes for either: the two highest bits of each 32 are 1x in a count of 32 bits,
// 0x and 01 in the lower and upper half of one of 64, 00 in the pre-pass's arrays.
// A call's prefixes replace what the one before left.
// The last tile zeroes the few that only that one had, and counts the call in the header: it has every tile's count by then, and a tile's count is out
// after its waves have read the word there, so nobody reads it later.  (If counts were
// computed by waiting tiles, the last tile first sees to it that their owners have started, see
// scan_end.)  So no tile waits for its stores or counts itself finished, and the call does not end with
// a clean-up.  us with words that the last tile zeroed once all had counted themselves finished | now, the other
// changes of the scan included: fp32 256 KB 4.63 | 4.02, 6.4 MB 6.12 | 5.38, 24 MB 9.4 | 9.1, 100 MB 29.3 | 28.4, 300 MB
// 77.0 | 75.2; bf16 4 MB 5.9 | 5.4, 200 MB 58.9 | 57.0, 600 MB 163.6 | 156.1.  (A call that zeroes what only the call
// before it had: 16 KB after 800 MB 27 us instead of 6.2.)
constexpr int kCallShift = 16;                // of a count's word; of a wide one the number's lowest bits
constexpr int kCallBits = 15, kTermBits = kCallBits - 1;
constexpr unsigned kCountOwner = 1u << 15, kCountBits = kCountOwner - 1u;
constexpr int kTagShift = 62;                 // of a prefix
constexpr unsigned kLinePrefixes = 14, kMostPrefixes = kLinePrefixes * kFinishLanes;

__host__ __device__ inline unsigned narrow_mark(unsigned call) { return 1u << 31 | call << kCallShift; }
__host__ __device__ inline unsigned long long wide_mark(unsigned long long number) {
    return 1ull << 62 | (number >> kCallBits & ((1ull << 30) - 1ull)) << 32 | (number & ((1ull << kCallBits) - 1ull)) << kCallShift;
}

// hdr->scan_word; zero in a new workspace.
struct ScanCalls {
    unsigned call;                 // the next one's number, its lowest 15 bits
    unsigned prefixes;             // that the last call left
    unsigned limit;                // a call with more tiles is a wide one; 0: none is
    __host__ __device__ explicit ScanCalls(unsigned long long word)
        : call(static_cast<unsigned>(word) & ((1u << kCallBits) - 1u)), prefixes(static_cast<unsigned>(word) >> kCallBits),
          limit(static_cast<unsigned>(word >> 32)) {
        // (a workspace that was never initialised is at worst scanned wrongly, and nothing outside it written)
        if (prefixes > kMostPrefixes) prefixes = kMostPrefixes;
    }
    __host__ __device__ unsigned long long word() const {
        return static_cast<unsigned long long>(limit) << 32 | prefixes << kCallBits | call;
    }
    __host__ __device__ bool wide(unsigned tiles) const { return limit - 1u < tiles - 1u; }
    __host__ __device__ ScanCalls next(unsigned tiles, unsigned prefixes_left) const {
        ScanCalls after = *this;
        after.call = (call + 1u) % (1u << kCallBits);
        after.prefixes = prefixes_left;
        if (after.call % (1u << kTermBits) == 0u || wide(tiles)) after.limit = tiles;
        return after;
    }
};

__host__ __device__ inline size_t div_up(size_t a, size_t b) { return a / b + (a % b != 0); }

inline size_t tiles_for(size_t n, int w, int loads) {
    const size_t tile_elems = static_cast<size_t>(kThreads * 16 * loads / w);
    return div_up(n, tile_elems);
}
inline size_t scan_state_bytes(size_t tiles) { return 8 * tiles; }     // (a wide call's)
// log2 of the tiles per block: 9, or more where the header has not room for that many prefixes (from 458752 tiles up)
__host__ __device__ inline int block_shift_of(unsigned tiles) {
    int shift = kBlockShift;
    while (tiles >> shift > kMostPrefixes) ++shift;
    return shift;
}
// The decoder's pre-pass arrays sit at the end of the workspace; where it is no larger than it has to be, in bytes
// that the scan state of other calls takes as well.
inline size_t pad256(size_t b) { return div_up(b, 256) * 256; }
inline size_t decoder_area_bytes(size_t chunks) {   // chunk_prefix, chunk_total, unit_end
    return pad256(8 * chunks) + pad256(4 * chunks) + pad256(4 * 128 * chunks);
}

// A prefix of the pre-pass: 30 bits in each half, so that neither passes for a tile's count.
__host__ __device__ inline unsigned long long in_halves(unsigned long long v) { return v >> 30 << 32 | (v & 0x3FFFFFFFull); }
__host__ __device__ inline unsigned long long from_halves(unsigned long long v) { return v >> 32 << 30 | (v & 0x3FFFFFFFull); }

// ------------------------------------------------------------ device helpers
__device__ inline unsigned long long load64(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline unsigned load32(const unsigned* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store64(unsigned long long* p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store32(unsigned* p, unsigned v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The same as an exchange, whose old value nobody waits for.  It reaches the memory that all XCDs see sooner
// than a store does: calls whose tiles wait for words written so take 3 to 5 % less below 20 MB (us,
// store | exchange: 256 KB 4.20 | 4.00, 6.4 MB 6.17 | 5.95, decoding 6.4 MB 5.89 | 5.57).
__device__ inline void exchange64(unsigned long long* p, unsigned long long v) {
    (void)__hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void exchange32(unsigned* p, unsigned v) {
    (void)__hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// acc + number of set bits of `ballot` in lanes below the calling lane.
__device__ inline unsigned lanes_below(unsigned long long ballot, unsigned acc) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(ballot >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(ballot), acc));
}

__device__ inline unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
    for (int off = 1; off < kWaveSize; off <<= 1) v += __shfl_xor(v, off);
    return v;
}

// A value that is the same in every lane, moved to scalar registers so that
// address arithmetic built on it stays scalar.
__device__ inline unsigned uniform(unsigned v) {
    return static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
}
__device__ inline unsigned long long uniform(unsigned long long v) {
    return (static_cast<unsigned long long>(uniform(static_cast<unsigned>(v >> 32))) << 32) |
           uniform(static_cast<unsigned>(v));
}

// Lane `src` (wave-uniform) of v.
__device__ inline unsigned lane_value(unsigned v, int src) {
    return static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(v), src));
}
__device__ inline unsigned long long lane_value(unsigned long long v, int src) {
    return (static_cast<unsigned long long>(lane_value(static_cast<unsigned>(v >> 32), src)) << 32) |
           lane_value(static_cast<unsigned>(v), src);
}

// Sum over the wave of one value per lane (each below 2^26), wave-uniform
// result.  DPP adds within each row of 16 lanes (pairs, quads, half-row mirror,
// row mirror), then the four row sums are read out and added on the scalar
// unit: a dozen instructions and no lane-index registers, which matters where
// the caller holds a tile's data in registers and every cycle of the scan is
// waited for by the tile's other waves.
__device__ inline unsigned wave_sum_small(unsigned v) {
    v += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0xB1, 0xF, 0xF, true));
    v += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x4E, 0xF, 0xF, true));
    v += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x141, 0xF, 0xF, true));
    v += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x140, 0xF, 0xF, true));
    return lane_value(v, 0) + lane_value(v, 16) + lane_value(v, 32) + lane_value(v, 48);
}

// Streaming 16-byte accesses, for what a call touches exactly once: the
// uncompressed tensor (read by the encoder, written by the decoder) and the
// encoder's output.  The non-temporal hint keeps such data from displacing other
// data in the caches (a plain copy kernel gains about 10 % from it here).  The
// decoder's reads of the compressed stream are ordinary loads: the masks are
// read twice (pre-pass, then expand), and the value runs of neighbouring waves
// share cache lines; with the hint those re-reads went back to memory, which
// cost 10-25 % of the decoder's time at low density.
typedef unsigned int vec4u __attribute__((ext_vector_type(4)));
typedef vec4u vec4u_at4 __attribute__((aligned(4)));
typedef vec4u vec4u_at2 __attribute__((aligned(2)));
__device__ inline uint4 load16_stream(const void* p) {
    const vec4u v = __builtin_nontemporal_load(reinterpret_cast<const vec4u*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ inline void store16_stream(void* p, const uint4& d) {
    vec4u v;
    v.x = d.x; v.y = d.y; v.z = d.z; v.w = d.w;
    __builtin_nontemporal_store(v, reinterpret_cast<vec4u*>(p));
}

// The same 16 bytes to an address that is a multiple of W only: one store whatever
// the address (the memory pipeline takes unaligned vector stores), through the
// caches, because a wave's 1 KB then shares its first and last line with its
// neighbours.  Against a store per element: 44.5 -> 21.2 us for 29 M fp16 elements at
// an odd element (aligned: 18.9), 49 -> 32.7 us for 26 M fp32 ones (24.4), 307 ->
// 126 us for 206 M bf16 ones (109).
template <int W>
__device__ inline void store16_loose(void* p, const uint4& d) {
    vec4u v;
    v.x = d.x; v.y = d.y; v.z = d.z; v.w = d.w;
    if (W == 4) *reinterpret_cast<vec4u_at4*>(p) = v;
    else *reinterpret_cast<vec4u_at2*>(p) = v;
}

// A raw buffer's descriptor word (32-bit data, no swizzle), the non-temporal bit of a buffer load.
constexpr int kRawBuffer = 0x00020000;
constexpr int kNonTemporal = 2;

// LDS written by some lanes of a wave is read by other lanes of the same wave:
// order the accesses (LDS operations of one wave execute in order).
__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 16 bytes of input from a 16-byte boundary on, for the lane whose first element
// is e0.  Elements at or past n read as zero.  A chunk that holds at least one
// element of the tensor is loaded whole: an aligned 16-byte chunk never straddles
// a page, so the access is as safe as the load of that element, and the bytes
// past the tensor's end are cleared in registers.
template <int W>
__device__ inline uint4 load_chunk(const unsigned char* __restrict__ in, size_t e0, size_t n) {
    constexpr int E = 16 / W;
    unsigned d[4];
    if (e0 >= n) return make_uint4(0u, 0u, 0u, 0u);
    const uint4 v = load16_stream(in + e0 * W);
    if (e0 + E <= n) return v;
    const unsigned valid_bytes = static_cast<unsigned>(n - e0) * W;   // 1 .. 15
    const unsigned raw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const unsigned lo = 4u * k;
        d[k] = valid_bytes >= lo + 4u ? raw[k]
             : valid_bytes > lo      ? raw[k] & ((1u << (8u * (valid_bytes - lo))) - 1u)
                                     : 0u;
    }
    return make_uint4(d[0], d[1], d[2], d[3]);
}

// Which elements are kept.  Plain ZVC (RELU = false) keeps the elements that are
// non-zero as integers (section 5.2: words compared to zero form the mask
// bits).  The fused ReLU + ZVC encoder (RELU = true) reads pre-activation
// values (IEEE-style, sign in the top bit: fp32, fp16, bf16) and keeps those
// whose sign bit is clear and which are not +0, i.e. the non-zeros of ReLU(x);
// as signed integers those are exactly the words greater than zero.
template <int W, bool RELU>
__device__ inline bool element_kept(const uint4& v, int c) {
    const unsigned d[4] = {v.x, v.y, v.z, v.w};
    if (W == 4) return RELU ? static_cast<int>(d[c]) > 0 : d[c] != 0u;
    if (c & 1) return RELU ? static_cast<int>(d[c >> 1]) > 0xFFFF : d[c >> 1] > 0xFFFFu;
    const unsigned low = d[c >> 1] & 0xFFFFu;
    return RELU ? (low - 1u) < 0x7FFFu : low != 0u;
}

// Kept-element bits of the lane's 16 bytes: bit c set <=> element c is kept.
template <int W, bool RELU>
__device__ inline unsigned presence_bits(const uint4& v) {
    unsigned bits = 0;
#pragma unroll
    for (int c = 0; c < 16 / W; ++c) bits |= (element_kept<W, RELU>(v, c) ? 1u : 0u) << c;
    return bits;
}

// A dword of a wave's LDS queue at any offset that is a multiple of W (with
// 16-bit elements the queue need not sit at the destination's offset modulo 4).
template <int W>
__device__ inline unsigned queue_dword(const unsigned char* p) {
    if (W == 4) return *reinterpret_cast<const unsigned*>(p);
    return static_cast<unsigned>(*reinterpret_cast<const unsigned short*>(p)) |
           (static_cast<unsigned>(*reinterpret_cast<const unsigned short*>(p + 2)) << 16);
}

// Writes out what a wave has staged so far.  The wave's packed run goes through
// its LDS slice like through a queue: slice offset p holds the byte that belongs
// at global address gzero + p (gzero is wave-uniform and a multiple of W; nothing
// before offset lo is ever dereferenced), and [lo, end) is staged but not yet
// written.  Every store instruction covers one 256-byte aligned block of the
// destination, a dword per lane, so whole 128-byte lines leave as whole lines
// wherever the run begins (partial-line writes cost the memory system about as
// much as whole lines).  Unless `last`, the bytes after the run's last line
// boundary stay behind: they move to the front of the slice, where the next
// step continues them, so a wave writes two partial lines per tile, not two per
// step.  Updates gzero, lo and end.
template <int W>
__device__ inline void wave_flush(unsigned char*& gzero, unsigned char* stage, unsigned& lo,
                                  unsigned& end, bool last, int lane) {
    const uintptr_t g = reinterpret_cast<uintptr_t>(gzero);
    // slice offsets of the bytes to write: [first, tail)
    int first = static_cast<int>(lo);
    const int keep_back = last ? 0 : static_cast<int>((g + end) & 127u);   // bytes after the last line boundary
    const int tail = static_cast<int>(end) - keep_back;
    if (tail <= first) {       // no line completed yet (or, with `last`, nothing staged)
        if (last) lo = end;
        return;
    }
    int stop = tail;
    if (W == 2) {
        // odd halves at either end, so that what is left is whole dwords of the destination
        if ((g + first) & 2u) {
            if (lane == 0)
                *reinterpret_cast<unsigned short*>(gzero + first) =
                    *reinterpret_cast<const unsigned short*>(stage + first);
            first += 2;
        }
        if (((g + stop) & 2u) && stop > first) {
            if (lane == 0)
                *reinterpret_cast<unsigned short*>(gzero + (stop - 2)) =
                    *reinterpret_cast<const unsigned short*>(stage + (stop - 2));
            stop -= 2;
        }
    }
    // one 256-byte aligned block of the destination per store instruction, four blocks at a
    // time so that the LDS reads of a round are under way together
    constexpr int kRound = 4;
    for (int block = first - static_cast<int>((g + first) & 255u); block < stop; block += 256 * kRound) {
        unsigned v[kRound];
#pragma unroll
        for (int j = 0; j < kRound; ++j) {
            const int at = block + 256 * j + 4 * lane;
            v[j] = 0u;
            if (at >= first && at < stop) v[j] = queue_dword<W>(stage + at);
        }
#pragma unroll
        for (int j = 0; j < kRound; ++j) {
            const int at = block + 256 * j + 4 * lane;
            if (at >= first && at < stop)
                __builtin_nontemporal_store(v[j], reinterpret_cast<unsigned*>(gzero + (block + 256 * j)) + lane);
        }
    }
    if (last) {
        lo = end;
        return;
    }
    // the unfinished line moves to the front of the slice (all lanes read before any writes:
    // source and destination may overlap)
    const unsigned rem = static_cast<unsigned>(keep_back);          // below 128
    unsigned keep = 0;
    const bool mine = static_cast<unsigned>(W * lane) < rem;
    if (mine) {
        if (W == 4) keep = *reinterpret_cast<const unsigned*>(stage + tail + W * lane);
        else keep = *reinterpret_cast<const unsigned short*>(stage + tail + W * lane);
    }
    wave_lds_sync();
    if (mine) {
        if (W == 4) *reinterpret_cast<unsigned*>(stage + W * lane) = keep;
        else *reinterpret_cast<unsigned short*>(stage + W * lane) = static_cast<unsigned short>(keep);
    }
    gzero += tail;
    lo = 0;
    end = rem;
}

// Global bytes [0, end) at gbase (16-byte aligned, the same in all lanes) into LDS at
// `stage`, by one wave, without a register in between: 1 KB per instruction, lane i's 16
// bytes behind lane i - 1's.  A slot that holds nothing is left out by a scalar branch.  A
// 16-byte chunk is loaded whole even where the run begins or ends inside it: an aligned
// chunk never straddles a page, so the access is as safe as that of the bytes wanted.
// stage_wait() before LDS is read.  (Through registers, with the bytes behind the run
// cleared, this was 110 of the expand kernel's 500 vector instructions per 4 KB of 16-bit
// output, and that kernel had the vector units busy 83 % of its time.)
constexpr unsigned kSlotBytes = kWaveSize * 16;
constexpr int kFetchSlots = kStageLoads + 1;      // a run of 4 KB that begins anywhere in a chunk

// Slot at byte AT behind gbase and stage (an immediate of the instruction, for both).
template <bool STREAMING, unsigned AT>
__device__ __forceinline__ void stage_slot(unsigned char* stage, const unsigned char* gbase, unsigned end, int lane) {
    if (AT >= end) return;                                               // uniform
    if (AT + 16u * lane < end)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) unsigned*)(gbase + 16u * lane),
                                         (__attribute__((address_space(3))) unsigned*)stage, 16, AT,
                                         STREAMING ? kNonTemporal : 0);
}
template <bool STREAMING>
__device__ __forceinline__ void wave_stage(unsigned char* stage, const unsigned char* gbase, unsigned end, int lane) {
    static_assert(kStageLoads == 4 && kFetchSlots == 5 && 4 * kSlotBytes == 4096, "immediates are below 4096");
    stage_slot<STREAMING, 0>(stage, gbase, end, lane);
    stage_slot<STREAMING, kSlotBytes>(stage, gbase, end, lane);
    stage_slot<STREAMING, 2 * kSlotBytes>(stage, gbase, end, lane);
    stage_slot<STREAMING, 3 * kSlotBytes>(stage, gbase, end, lane);
    if (end > 4 * kSlotBytes) stage_slot<STREAMING, 0>(stage + 4 * kSlotBytes, gbase + 4 * kSlotBytes, end - 4 * kSlotBytes, lane);
}
__device__ __forceinline__ void stage_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// 16 bytes of output: element c is "bit c of `field` ? next stored element : 0", and the
// next stored element is at `at` in `lds`, whose first 16 bytes are zero (an absent
// element is read from there).  Three instructions per element beside its LDS read: the
// bit as 0 or -1, the address (at & that), the next address (at - W * that).  Selecting
// address and value by comparison took 8.  With the staging above: 202 vector
// instructions per 4 KB of 16-bit output instead of 499 (32-bit: 108, 303), the expand
// kernel 13.8 -> 12.4 us for 51 MB bf16; 822 MB fp32, bound by memory, 158 either way.
template <int W>
__device__ __forceinline__ uint4 expand_lane(const unsigned char* lds, unsigned at, unsigned field) {
    unsigned d[4], half[2];
#pragma unroll
    for (int c = 0; c < 16 / W; ++c) {
        const int bit = __builtin_amdgcn_sbfe(static_cast<int>(field), c, 1);
        const unsigned from = at & static_cast<unsigned>(bit);
        if (W == 4) d[c] = *reinterpret_cast<const unsigned*>(lds + from);
        else half[c % 2] = *reinterpret_cast<const unsigned short*>(lds + from);
        if (W == 2 && c % 2 == 1) {
            asm("" : "+v"(half[0]), "+v"(half[1]));         // (or the compiler goes on in 16 bits, an instruction more)
            d[c / 2] = half[1] << 16 | half[0];
        }
        if (c + 1 < 16 / W) asm("v_mad_i32_i24 %0, %1, %2, %0" : "+v"(at) : "v"(bit), "n"(-W));
    }
    return make_uint4(d[0], d[1], d[2], d[3]);
}

// Inclusive sum over the first LANES lanes (whole wave active; later lanes: unspecified).
template <int LANES>
__device__ __forceinline__ unsigned wave_scan_small(unsigned v) {
    static_assert(LANES == 32 || LANES == 64, "two or four rows of lanes");
    v += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x111, 0xF, 0xF, true));
    v += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x112, 0xF, 0xF, true));
    v += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x114, 0xF, 0xF, true));
    v += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x118, 0xF, 0xF, true));
    // a row's last lane to the whole next row, the second row's last to the third and fourth
    v += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x142, 0xA, 0xF, false));
    if (LANES == 64) v += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x143, 0xC, 0xF, false));
    return v;
}

// Adds to the tile's arrival word in LDS, by one lane, and returns what was there.
__device__ __forceinline__ unsigned arrive(unsigned* word, unsigned v) {
    unsigned none = 0;
    asm("" : "+v"(none));          // (or the compiler makes code for a sum over many lanes)
    return __hip_atomic_fetch_add(word + none, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One call's view of the scan state.
struct ScanState {
    WsHeader* hdr;
    ScanCalls calls;               // before this one
    unsigned wide;                 // 0 | 1
    unsigned mark0, mark1;         // what the call's counts have beside count and owner, in the words with even and odd index:
                                   // two tiles', or one's lower and upper half
    int block_shift;
    // The word's load, which goes out behind the tile's own and is waited for when those have arrived.  (On
    // the vector unit: a scalar load would be waited for at the next barrier.  One of 8 bytes: every wave of the
    // call asks for it, and a second one costs the decoder 0.5 to 1.7 us from 20 MB up.)
    __device__ static unsigned long long ask(const WsHeader* header) {
        unsigned none = 0;
        asm("" : "+v"(none));
        return load64(reinterpret_cast<const unsigned long long*>(reinterpret_cast<const unsigned char*>(&header->scan_word) + none));
    }
    // Every wave builds its ScanState before it counts itself in at the tile's arrival word: the last tile writes the
    // next word once it has every tile's count, and a tile's count is out once its waves have arrived.  The load
    // has returned when the asm statement is reached, and no later access to memory is moved before it.
    __device__ ScanState(WsHeader* header, unsigned num_tiles, unsigned long long asked)
        : hdr(header), calls(settled(asked)), wide(calls.wide(num_tiles) ? 1u : 0u), mark0(narrow_mark(calls.call)),
          mark1(mark0), block_shift(block_shift_of(num_tiles)) {
        if (__builtin_expect(wide != 0u, 0)) {
            const unsigned long long mark = wide_mark(settled(load64(&header->wide_calls)));
            mark0 = static_cast<unsigned>(mark);
            mark1 = static_cast<unsigned>(mark >> 32);
        }
    }
    __device__ static unsigned long long settled(unsigned long long word) {
        asm volatile("" : "+v"(word) : : "memory");
        return uniform(word);
    }
    __host__ __device__ unsigned* counts() const { return reinterpret_cast<unsigned*>(hdr + 1); }
    __host__ __device__ unsigned long long* wide_counts() const { return reinterpret_cast<unsigned long long*>(hdr + 1); }
    __host__ __device__ unsigned long long mark() const { return static_cast<unsigned long long>(mark1) << 32 | mark0; }
    // Whether the words with even and odd index are counts of this call.
    __host__ __device__ bool is_there0(unsigned word) const { return (word ^ mark0) >> kCallShift == 0u; }
    __host__ __device__ bool is_there1(unsigned word) const { return (word ^ mark1) >> (wide ? 0 : kCallShift) == 0u; }
    // Whether the tile has written its count itself.
    __device__ bool has_started(unsigned tile) const {
        return wide ? (load64(wide_counts() + tile) ^ (mark() | kCountOwner)) <= kCountBits
                    : (load32(counts() + tile) ^ (mark0 | kCountOwner)) <= kCountBits;
    }
    __device__ void publish(unsigned tile, unsigned kept) const {
        if (__builtin_expect(wide != 0u, 0)) exchange64(wide_counts() + tile, mark() | kCountOwner | kept);
        else exchange32(counts() + tile, mark0 | kCountOwner | kept);
    }
    // A count that another tile has computed, unless its owner has been there meanwhile.
    __device__ void publish_for(unsigned tile, unsigned kept) const {
        if (wide) {
            unsigned long long* const p = wide_counts() + tile;
            unsigned long long old = load64(p);
            while ((old ^ mark()) >> kCallShift != 0ull) {
                const unsigned long long seen = atomicCAS(p, old, mark() | kept);
                if (seen == old) break;
                old = seen;
            }
        } else {
            unsigned* const p = counts() + tile;
            unsigned old = load32(p);
            while (!is_there0(old)) {
                const unsigned seen = atomicCAS(p, old, mark0 | kept);
                if (seen == old) break;
                old = seen;
            }
        }
    }
    __host__ __device__ unsigned long long* prefix(unsigned block) const {
        return &hdr->finish[block / kLinePrefixes].prefix[block % kLinePrefixes];
    }
    __host__ __device__ unsigned long long tag() const { return 1ull + (calls.call & 1u); }
    __device__ void publish_prefix(unsigned tile, unsigned long long upto) const {
        exchange64(prefix(tile >> block_shift), tag() << kTagShift | upto);
    }
    __host__ __device__ bool ends_block(unsigned tile) const { return ((tile + 1u) & ((1u << block_shift) - 1u)) == 0u; }
    // The prefixes that only the call before had, by one wave.
    __host__ __device__ void zero_prefixes_left(unsigned num_tiles, int lane) const {
        for (unsigned i = (num_tiles >> block_shift) + lane; i < calls.prefixes; i += kWaveSize) *prefix(i) = 0ull;
    }
};

// Device-wide exclusive scan of the per-tile counts, single pass (the paper's
// offset at which the next mask goes, section 5.1, for a whole tile at a time).
//
// Protocol.  Every tile publishes its own count (the wave of the tile that
// finishes its zero tests last does).  The last tile of every block of 512 also
// publishes the running total up to and including itself.  A tile
// finds the nearest published block prefix behind it and adds the counts of the
// tiles between that block and itself, two counts per 8-byte load across the
// wave.  In steady state that is a few hundred counts and the walk takes one
// pass.
//
// Why this shape (measured on MI355X): a device-scope load of a line that other
// XCDs are still writing costs a coherence round trip and slows the streaming
// traffic around it, while lines that have gone quiet are served from the local
// L2.  Counts are written once and read afterwards; running prefixes, which are
// written late, are kept sparse so that few lines are ever read while hot.  A
// classic look-back that polls a status+value word per tile, or a ticket
// counter per tile (one same-address atomic costs about 11 ns here), holds the
// whole kernel to a third of memory speed.
//
// Tiles are numbered by workgroup id.  The hardware hands workgroups out in id
// order, so a predecessor is normally already running and publishes within
// microseconds.  The wait does not rely on that: after `patience` fruitless
// polls the waiting wave computes a missing predecessor's count itself
// (`count_tile`, a re-read of that tile's input) and publishes it, so the walk
// ends whatever the dispatch order.
//
// Called by one whole wave of the tile, when the tile's own zero tests are done
// (asking for the prefixes earlier, while the tile's loads are under way, saves
// a round trip but finds a prefix further back, and the extra counts to read
// cost more than the round trip).  PAUSE: see there.  Returns the number of kept elements in all
// tiles before `tile` (not 0).
constexpr int kNoPause = -1, kDecoderPause = 16;
template <int PAUSE, class CountTile>
__device__ inline unsigned long long scan_exclusive_prefix(const ScanState& st, unsigned tile, int lane,
                                                           const CountTile& count_tile) {
    const int t = static_cast<int>(tile);
    // nearest published block prefix
    int bb = (t >> st.block_shift) - 1;
    unsigned long long base = 0;
    int lo = 0;
    // Nothing is asked for one round trip to memory (patience is needed below) and PAUSE sleeps of 64 clocks, or
    // at once with kNoPause: a line of counts that many tiles read while others still write it costs all
    // of them more.  us, encoding, at once | a round trip later | 0.3 us asleep: fp32 6.4 MB 6.1 | 5.8 | 6.1, 64 MB
    // 20.4 | 17.3 | 19.5, 300 MB 73.8 | 70.7 | 73.6 (waiting for the tile in front first, alone: 6.9, 21.3, 75.8); with 8
    // sleeps more 6.4 MB 5.8 | 5.8, 12 MB 7.1 | 7.2.  Decoding, whose workgroups have their counts all at the same time, a round trip
    // and 14 | 16 | 18 | 20 sleeps: fp32 3 MB 4.42 | 4.47 | 4.52, 6.4 MB 4.78 | 4.83 | 4.89 | 4.94 (without any 5.6), 30 MB 9.48 | 9.30 | 9.23,
    // at an odd element 20 MB 7.58 | 7.50 | 7.44; 6.4 MB from memory, where the counts are less together, the kernel alone 6.92 | 6.88 |
    // 6.87 | 6.82.
    unsigned long long patience_word = 0;
    if (PAUSE != kNoPause) patience_word = uniform(load64(&st.hdr->patience_plus_one));
    if (PAUSE > 0) __builtin_amdgcn_s_sleep(PAUSE);
    while (bb >= 0) {
        const int idx = bb - lane;
        unsigned long long pv = 0;
        if (idx >= 0) pv = load64(st.prefix(static_cast<unsigned>(idx)));
        const unsigned long long have = __ballot(pv >> kTagShift == st.tag());
        if (have) {
            const int k = __ffsll(static_cast<long long>(have)) - 1;
            base = lane_value(pv, k) << 2 >> 2;
            lo = (bb - k + 1) << st.block_shift;   // first tile after that block
            break;
        }
        bb -= kWaveSize;
    }
    // Counts of tiles lo .. t-1, a pair (a wide one) per 8-byte load (lo is a multiple of the
    // block size: pairs are aligned), kScanBatch loads per lane in flight at a time
    // (256 tiles a batch; asking for more at once reads more of the newest counts while they are still being
    // written, which measures slower.  So do 64-bit words in every call: a batch is 16 lines then and not 8.  fp32 6.4 MB
    // 5.33 | 5.62 us, 16-bit 30 MB 12.6 | 13.5, decoding 40 MB 12.5 | 13.6).  The
    // loads of a batch are added in order as far as everything they cover is
    // published; a later round asks again only from the first load that found
    // something missing, so the waiting re-reads no more than the newest counts.
    constexpr int kScanBatch = 2;
    const int per = st.wide ? 1 : 2;              // tiles per 8 bytes
    const unsigned count_bits1 = st.wide ? 0u : kCountBits;
    int done_to = lo;              // wave-uniform: the counts of tiles lo .. done_to-1 are in `sum`
    unsigned sum = 0;              // a lane adds few counts, each below 2^16
    unsigned polls = 0;
    while (done_to < t) {
        unsigned long long pair[kScanBatch];
        const unsigned long long* const from =
            reinterpret_cast<const unsigned long long*>(st.counts() + (st.wide ? 2 * static_cast<size_t>(done_to) : done_to));
#pragma unroll
        for (int k = 0; k < kScanBatch; ++k) {
            const int i = done_to + per * (k * kWaveSize + lane);
            pair[k] = i < t ? load64(from + k * kWaveSize + lane) : 0ull;
        }
        int complete = 0;          // leading loads of the batch that found everything published
        int hole = -1;             // wave-uniform: the first tile found unpublished
#pragma unroll
        for (int k = 0; k < kScanBatch; ++k) {
            if (complete != k) continue;          // wave-uniform
            const int i = done_to + per * (k * kWaveSize + lane), i1 = i + per - 1;
            const unsigned c0 = static_cast<unsigned>(pair[k]), c1 = static_cast<unsigned>(pair[k] >> 32);
            const bool there0 = i >= t || st.is_there0(c0), there1 = i1 >= t || st.is_there1(c1);
            const unsigned long long missing = __ballot(!(there0 && there1));
            if (!missing) {
                sum += (i < t ? c0 & kCountBits : 0u) + (i1 < t ? c1 & count_bits1 : 0u);
                complete = k + 1;
            } else {
                const int first = __ffsll(static_cast<long long>(missing)) - 1;
                hole = done_to + per * (k * kWaveSize + first) + (st.is_there0(lane_value(c0, first)) ? per - 1 : 0);
            }
        }
        done_to += complete * per * kWaveSize;
        if (hole < 0) continue;                   // the whole batch was there: the next one, if any
        if (PAUSE == kNoPause && polls == 0) patience_word = uniform(load64(&st.hdr->patience_plus_one));
        const unsigned patience = patience_word != 0 ? static_cast<unsigned>(patience_word - 1) : kDefaultPatience;
        if (polls < patience) {
            ++polls;
            __builtin_amdgcn_s_sleep(kPollSleep);
            continue;
        }
        // help one unpublished predecessor, then look again without waiting anew.  The call's last tile must
        // know (scan_end): helped_here is written before the count can be seen.
        const unsigned helped_count = count_tile(static_cast<unsigned>(hole), lane);
        if (lane == 0) {
            store64(&st.hdr->helped_here, 1ull);
            atomicAdd(&st.hdr->helped, 1ull);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            st.publish_for(static_cast<unsigned>(hole), helped_count);
        }
    }
    // (halves, so that no partial sum can overflow whatever the distance walked)
    return base + wave_sum_small(sum & 0xFFFFu) +
           (static_cast<unsigned long long>(wave_sum_small(sum >> 16)) << 16);
}

// The end of a call, by the scan wave of its last tile once it has the counts of all tiles: the
// next call takes the next number.  A tile whose count was computed by another one may not have
// begun yet, and would then read the word of the next call: the last tile waits for such
// tiles (none of them waits for it).
__device__ inline void scan_end(const ScanState& st, unsigned num_tiles, int lane) {
    if (__builtin_expect(uniform(load64(&st.hdr->helped_here)) != 0ull, 0)) {
        for (unsigned tile = lane; tile + 1u < num_tiles; tile += kWaveSize)
            while (!st.has_started(tile)) __builtin_amdgcn_s_sleep(kPollSleep);
        if (lane == 0) store64(&st.hdr->helped_here, 0ull);
    }
    st.zero_prefixes_left(num_tiles, lane);
    if (lane != 0) return;
    store64(&st.hdr->scan_word, st.calls.next(num_tiles, num_tiles >> st.block_shift).word());
    if (__builtin_expect(st.wide != 0u, 0)) atomicAdd(&st.hdr->wide_calls, 1ull);
}

// ------------------------------------------------- encoder: loads and zero tests
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

__device__ inline unsigned load_stream(const unsigned* p) { return __builtin_nontemporal_load(p); }
__device__ inline unsigned load_stream(const unsigned short* p) { return __builtin_nontemporal_load(p); }

// Dword `index` of a run of dwords that starts at `base` (wave-uniform, inside
// the tensor) and of which only dwords 0 .. room belong to the tensor, the last
// one maybe only with its low half (half_tail: 16-bit elements, odd count).
// What lies past the tensor reads as zero.  The dword that holds the tensor's
// last element is loaded whole (an aligned dword never straddles a page, so
// that is as safe as loading the element) and later lanes are redirected to
// it, so the loads need no branch; the excess is cleared in registers.  SPLIT
// fetches halves and checks each.
template <bool SPLIT>
__device__ __forceinline__ unsigned load_dword_ragged(const unsigned char* base, unsigned index,
                                                      unsigned room, bool half_tail) {
    if (SPLIT) {
        const unsigned short* p = reinterpret_cast<const unsigned short*>(base);
        const unsigned lo = index <= room ? static_cast<unsigned>(load_stream(p + 2 * index)) : 0u;
        const unsigned hi = index < room || (index == room && !half_tail)
                                ? static_cast<unsigned>(load_stream(p + 2 * index + 1)) : 0u;
        return lo | (hi << 16);
    }
    unsigned x = load_stream(reinterpret_cast<const unsigned*>(base) + (index < room ? index : room));
    if (index > room) x = 0u;
    if (half_tail && index == room) x &= 0xFFFFu;
    return x;
}

// Which elements are kept.  Plain ZVC (RELU = false) keeps the elements that are
// non-zero as integers (section 5.2: words compared to zero form the mask
// bits).  The fused ReLU + ZVC encoder (RELU = true) reads pre-activation
// values (IEEE-style, sign in the top bit: fp32, fp16, bf16) and keeps those
// whose sign bit is clear and which are not +0, i.e. the non-zeros of ReLU(x);
// as signed integers those are exactly the words greater than zero.
// kept_first: the element in the dword's low W bytes; kept_second (16-bit
// elements only): the one in its high half.
template <int W, bool RELU>
__device__ inline bool kept_first(unsigned x) {
    if (W == 4) return RELU ? static_cast<int>(x) > 0 : x != 0u;
    const unsigned low = x & 0xFFFFu;
    return RELU ? (low - 1u) < 0x7FFFu : low != 0u;
}
template <bool RELU>
__device__ inline bool kept_second(unsigned x) {
    return RELU ? static_cast<int>(x) > 0xFFFF : x > 0xFFFFu;
}

// The 16 low bits of v moved apart: bit i goes to bit 2i.
__device__ inline unsigned spread_bits(unsigned v) {
    v = (v | (v << 8)) & 0x00FF00FFu;
    v = (v | (v << 4)) & 0x0F0F0F0Fu;
    v = (v | (v << 2)) & 0x33333333u;
    v = (v | (v << 1)) & 0x55555555u;
    return v;
}

// v in lane LANE := the wave-uniform value s (other lanes keep theirs).  The
// value usually comes straight from a vector compare; a vector instruction that
// reads such a freshly written scalar as an operand needs one wait state, which
// the compiler cannot know for an instruction it does not see, hence the s_nop.
template <int LANE>
__device__ __forceinline__ void set_lane(unsigned& v, unsigned s) {
    asm("s_nop 0\n\tv_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(s), "n"(LANE));
}
// The two halves of a ballot into lanes LANE0 and LANE1 of v (one wait state serves both).
template <int LANE0, int LANE1>
__device__ __forceinline__ void set_lanes(unsigned& v, unsigned long long ballot) {
    asm("s_nop 0\n\tv_writelane_b32 %0, %1, %3\n\tv_writelane_b32 %0, %2, %4"
        : "+v"(v)
        : "s"(static_cast<unsigned>(ballot)), "s"(static_cast<unsigned>(ballot >> 32)), "n"(LANE0), "n"(LANE1));
}

// Count of kept elements of input tile q, by one wave (scan self-help).
template <int W, int CH, int WV, bool RELU, bool SPLIT>
struct CountInputTile {
    const unsigned char* in;
    size_t n;
    __device__ unsigned operator()(unsigned q, int lane) const {
        constexpr unsigned kTileDwords = EncoderGeometry<W, CH, WV>::kTileBytes / 4;
        const size_t d0 = static_cast<size_t>(q) * kTileDwords;      // inside the tensor: q is a predecessor
        const size_t last = (n * W - 1) / 4;
        const unsigned room = last - d0 < kTileDwords ? static_cast<unsigned>(last - d0) : kTileDwords;
        const bool half_tail = W == 2 && (n & 1u) != 0u && room < kTileDwords;
        unsigned count = 0;
#pragma unroll 1
        for (unsigned i = 0; i < kTileDwords; i += kWaveSize) {
            const unsigned x = load_dword_ragged<SPLIT>(in + d0 * 4, i + lane, room, half_tail);
            count += kept_first<W, RELU>(x) ? 1u : 0u;
            if (W == 2) count += kept_second<RELU>(x) ? 1u : 0u;
        }
        return wave_sum_small(count);      // a lane counts at most 512 elements
    }
};

// ------------------------------------------------------------------- kernels

// Zeroes the workspace header and scan state (`words` 8-byte words).
__global__ void reset_kernel(unsigned long long* ws_words, size_t words) {
    for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < words;
         i += static_cast<size_t>(gridDim.x) * blockDim.x)
        ws_words[i] = 0ull;
}

__global__ void write_word_kernel(unsigned long long* dst, unsigned long long v) { *dst = v; }

// Workgroup barrier that orders LDS traffic only (__syncthreads() would also
// wait for the wave's outstanding global stores).
__device__ inline void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

struct EncoderArgs {
    const unsigned char* __restrict__ in;
    size_t n;
    unsigned* __restrict__ masks;
    unsigned char* __restrict__ values;
    WsHeader* hdr;
    unsigned long long* d_bytes;
    unsigned long long* h_bytes;     // where the size goes as well, in host memory that the GPU sees, or null
    unsigned num_tiles;
    size_t num_groups;
    unsigned long long cap_values;   // bytes that may be written at `values`
    unsigned long long* offsets;   // windowed stream only: byte offset of every window, then the total
    unsigned window_shift;         // windowed stream only: a window is 1 KB << window_shift of input
};

// Section 5.1 encoder.  One workgroup per tile; tile = workgroup id.  With
// RELU the input is the pre-activation tensor and the stream is that of
// ReLU(input): the dense ReLU output is never written or read.
//
// A wave owns CH consecutive chunks of the tile (256 bytes each, a dword per
// lane).  Its work, in the order in which it happens:
//
//   1. zero tests as the loads arrive: the ballot of a chunk's test is two
//      masks (fp32) or, zipped with the ballot of the lanes' second elements,
//      four (16-bit); its popcount adds to the wave's total.  The masks are
//      gathered into registers lane by lane and leave as coalesced stores.
//   2. the wave adds its total to the tile's arrival word in LDS; the wave that
//      arrives last publishes the tile's count for the tiles behind it, at once.
//   3. the wave stages its kept elements in its LDS queue in packed order
//      (position = ballot bits in lower lanes + kept elements of earlier
//      chunks), as many steps as the queue holds (some of them earlier, with
//      their tests, see kFusedSteps): that needs nothing from other tiles, and it
//      gives the tiles in front the time to publish their counts.
//   4. wave 0 does the device-wide scan, which it begins once its own steps are
//      staged; one barrier hands the result to the other waves.
//   5. every wave writes its queue out in whole lines (wave_flush), staging
//      whatever did not fit before.
//
// WINDOWED selects the paper's own stream order (section 5.1: a group's
// non-zeros are appended right after its mask), packed back to back, plus a
// table with the byte offset of every window of 1 KB << window_shift of input
// (section 6 uses 4 KB and tries up to 64 KB).  The stream's bytes do not depend
// on the window size: the kernel works in units of 1 KB, four chunks, and stores
// the offset of every unit that begins a window.  The only differences are where things go in the
// wave's queue -- a group's mask sits before the group's elements -- and that
// masks leave with the values instead of going to a mask area.  The scan is the
// same: a window's byte offset is 4 x (groups before it) + W x (kept elements
// before it).
//
// EARLY: fewer of the tile's steps are staged before its count is published, see kFusedSteps.
template <int W, int CH, int WV, bool RELU, bool WINDOWED, bool SPLIT, bool EARLY>
__global__ __launch_bounds__(WV * kWaveSize) void compress_kernel(EncoderArgs a) {
    using G = EncoderGeometry<W, CH, WV>;
    constexpr int CG = G::kChunkGroups;
    constexpr int kWindowChunks = 4;              // the windowed stream's unit: 1 KB of input
    // Steps that may be staged in the same pass as their tests, while the wave waits for its next
    // loads anyway.  The others are staged once the tile's count is published: the tiles behind
    // wait for the count, and staging then fills the time until the counts of the tiles in front
    // are there.  Windowed staging is long (a step ends with a scan for the places of its masks), so
    // none of it goes in front: us with all steps fused -> none, 1 MB fp32 6.5 -> 5.5, 25 MB 13.6 ->
    // 11.1, 103 MB 36.3 -> 33.6, 297 MB 87.6 -> 83.5; 206 MB bf16 76.7 -> 72.0, 51 MB 21.7 -> 21.9.
    // Planar (choose_early() says which tensors): half of them where EARLY, else all.
    constexpr int kFusedSteps = WINDOWED ? 0 : EARLY ? G::kSteps / 2 : G::kSteps;
    static_assert(W == 2 || !SPLIT, "only 16-bit elements can sit at an odd half dword");

    __shared__ __align__(16) unsigned char s_stage[WV][G::kQueueBytes];
    __shared__ unsigned s_wave_total[WV];
    __shared__ unsigned s_arrive;                 // waves arrived << 24 | kept elements so far
    __shared__ unsigned long long s_prefix;

    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = static_cast<int>(uniform(static_cast<unsigned>(tid / kWaveSize)));
    const unsigned tile = blockIdx.x;
    if (tid == 0) s_arrive = 0u;

    const size_t wave_elem0 = static_cast<size_t>(tile) * G::kTileElems + static_cast<size_t>(wave) * G::kWaveElems;
    const size_t wave_group0 = static_cast<size_t>(tile) * G::kTileGroups + static_cast<size_t>(wave) * G::kWaveGroups;
    const size_t wave_dword0 = wave_elem0 / (4 / W);

    // ---- 1. loads, zero tests, masks (section 5.2: words compared to zero form the mask
    //         bits) and, fused with them where the queue has room, 3. compaction (section
    //         5.2: shift non-zeros to their packed slots)
    unsigned cur[SPLIT ? CH + 1 : CH];
    unsigned mask_reg[G::kMaskRegs];
    unsigned second_reg[W == 2 ? G::kMaskRegs : 1];   // 16-bit elements: the ballots of the lanes' second elements
    unsigned step_total[G::kSteps];               // wave-uniform
#pragma unroll
    for (int r = 0; r < G::kMaskRegs; ++r) mask_reg[r] = 0u;
#pragma unroll
    for (int r = 0; r < (W == 2 ? G::kMaskRegs : 1); ++r) second_reg[r] = 0u;
#pragma unroll
    for (int h = 0; h < G::kSteps; ++h) step_total[h] = 0u;
    unsigned char* stage = s_stage[wave];
    unsigned q_lo = 0, q_end = 0;                 // the wave's queue: slice offsets, wave-uniform
    unsigned zero_local = 0;                      // offset within the wave's run of slice offset 0
    unsigned window_local = 0;                    // lane i: offset within the wave's run of its window i
    // groups of the tensor in this wave's part
    const unsigned groups_here =
        wave_group0 >= a.num_groups ? 0u
        : a.num_groups - wave_group0 < static_cast<size_t>(G::kWaveGroups) ? static_cast<unsigned>(a.num_groups - wave_group0)
                                                                           : static_cast<unsigned>(G::kWaveGroups);
    // Windowed: every chunk leaves room for all the masks it could have.  Groups past the tensor's end have
    // none, and their room, which is behind everything else, is given back before the queue is written out:
    // the queue's end when steps first .. upto - 1 have been staged since the last time.
    const auto queue_end = [&](unsigned first, unsigned upto) -> unsigned {
        const unsigned there = min(groups_here, upto * G::kStepGroups) - min(groups_here, first * G::kStepGroups);
        return q_end - 4u * ((upto - first) * G::kStepGroups - there);
    };
    // 16-bit elements: masks from a register with 32 bits of the first elements' ballot in every even
    // lane and one with the same 32 bits of the second elements' ballot.  An even lane zips the low
    // halves into its mask, its odd neighbour (which reads them with a DPP row shift) the high halves
    // into the next mask.
    const auto zip_ballot_lanes = [&](unsigned first, unsigned second) __attribute__((always_inline)) -> unsigned {
        // (a DPP read of a register needs two wait states after the instruction that wrote it;
        // the compiler sees the lane writes only as opaque statements)
        asm volatile("s_nop 1" : "+v"(first), "+v"(second));
        const unsigned first_prev =
            static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(first), 0x111, 0xF, 0xF, true));
        const unsigned second_prev =
            static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(second), 0x111, 0xF, 0xF, true));
        const bool odd_lane = (lane & 1) != 0;
        return spread_bits(odd_lane ? first_prev >> 16 : first & 0xFFFFu) |
               (spread_bits(odd_lane ? second_prev >> 16 : second & 0xFFFFu) << 1);
    };

    // One chunk.  TEST: its masks and its share of the totals.  STAGE: its kept
    // elements into the queue at q_end.  Both use the same ballots.
    const auto chunk = [&](auto kc, auto test_c, auto stage_c) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        constexpr bool TEST = decltype(test_c)::value, STAGE = decltype(stage_c)::value;
        if constexpr (SPLIT && TEST) {
            // the next lane's dword: lanes shifted by one, the last lane's from the next chunk's first
            const int next = __builtin_amdgcn_update_dpp(__builtin_amdgcn_readfirstlane(static_cast<int>(cur[k + 1])),
                                                         static_cast<int>(cur[k]), 0x130, 0xF, 0xF, false);
            cur[k] = __builtin_amdgcn_alignbit(static_cast<unsigned>(next), cur[k], 16);
        }
        // Windowed: staged in a pass of its own, the chunk is tested again.  Kept from the first pass, the
        // ballots of all chunks are more than the scalar registers hold: they went to vector registers and
        // back, one by one.  us before | now: 16-bit 30 MB 15.0 | 13.8, 100 MB 38.8 | 36.2, 300 MB 92.8 |
        // 83.3; fp32 100 MB 28.4 | 27.3, 784 MB 174.7 | 170.1.
        if constexpr (WINDOWED && STAGE && !TEST) asm("" : "+v"(cur[k]));
        const unsigned x = cur[k];
        if (STAGE && WINDOWED && k % kWindowChunks == 0)
            set_lane<k / kWindowChunks>(window_local, zero_local + q_end);
        // (windowed: the lane's group has its mask, and the masks of the chunk's earlier groups, before it;
        // write_step_masks() puts the masks there)
        if constexpr (W == 4) {
            const bool keep = kept_first<4, RELU>(x);
            const unsigned long long b = __ballot(keep);
            const unsigned kept = static_cast<unsigned>(__popcll(b));
            if (TEST) {
                step_total[k / kStepChunks] += kept;
                // (now: the compiler would count when the totals are needed, and keep every ballot until then)
                if constexpr (WINDOWED) asm volatile("" : "+s"(step_total[k / kStepChunks]));
                set_lanes<(2 * k) % kWaveSize, (2 * k + 1) % kWaveSize>(mask_reg[(2 * k) / kWaveSize], b);
            }
            if (STAGE) {
                const unsigned at = 4u * lanes_below(b, 0u) + q_end + (WINDOWED ? 4u + 4u * (lane >> 5) : 0u);
                if (__builtin_expect(keep, 1)) *reinterpret_cast<unsigned*>(stage + at) = x;   // predicated, no branch
                q_end += 4u * kept + (WINDOWED ? 4u * CG : 0u);
            }
        } else {
            const bool keep0 = kept_first<2, RELU>(x), keep1 = kept_second<RELU>(x);
            const unsigned long long be = __ballot(keep0), bo = __ballot(keep1);
            const unsigned kept = static_cast<unsigned>(__popcll(be)) + static_cast<unsigned>(__popcll(bo));
            if (TEST) {
                step_total[k / kStepChunks] += kept;
                if constexpr (WINDOWED) asm volatile("" : "+s"(step_total[k / kStepChunks]));   // (as above)
                // The ballots as they are, 32 bits each in lanes 4k and 4k+2 (two masks' worth of
                // first elements in mask_reg, of second elements in second_reg): they are zipped
                // into the four masks once per wave (windowed: once per step), on the vector unit,
                // which measures 8-15 % faster than zipping every chunk on the scalar unit.
                set_lanes<(4 * k) % kWaveSize, (4 * k + 2) % kWaveSize>(mask_reg[(4 * k) / kWaveSize], be);
                set_lanes<(4 * k) % kWaveSize, (4 * k + 2) % kWaveSize>(second_reg[(4 * k) / kWaveSize], bo);
            }
            if (STAGE) {
                const unsigned at = 2u * lanes_below(bo, lanes_below(be, 0u)) + q_end +
                                    (WINDOWED ? 4u + 4u * (lane >> 4) : 0u);
                if (__builtin_expect(keep0, 1)) *reinterpret_cast<unsigned short*>(stage + at) = static_cast<unsigned short>(x);
                if (__builtin_expect(keep1, 1)) *reinterpret_cast<unsigned short*>(stage + at + (keep0 ? 2u : 0u)) = static_cast<unsigned short>(x >> 16);
                q_end += 2u * kept + (WINDOWED ? 4u * CG : 0u);
            }
        }
    };
    // Windowed: the masks of step h, which was staged from queue offset q_step on, into the gaps that
    // its chunks left for them: a lane per mask, whose place is the sum of the sizes of the step's
    // groups before it (a scan over 16 or 32 lanes).  Per step instead of per chunk: 89.1 ->
    // 87.7 us for 297 MB fp32, 87.8 -> 59.9 us for 149 MB bf16 (whose chunks zipped their masks on
    // the scalar unit), 4 MB fp32 5.83 -> 5.74 (all the tests done by then, see kFusedSteps).
    const auto write_step_masks = [&](auto hc, unsigned q_step) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
        constexpr int reg = h * G::kStepGroups / kWaveSize, lane0 = h * G::kStepGroups % kWaveSize;
        static_assert(G::kStepGroups == 16 || G::kStepGroups == 32, "one or two rows of lanes");
        unsigned mask = mask_reg[reg];
        if (W == 2) mask = zip_ballot_lanes(mask, second_reg[W == 2 ? reg : 0]);
        else asm volatile("s_nop 1" : "+v"(mask));            // (as in zip_ballot_lanes)
        const unsigned size = 4u + W * static_cast<unsigned>(__popc(mask));
        unsigned upto = size;
        upto += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(upto), 0x111, 0xF, 0xF, true));
        upto += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(upto), 0x112, 0xF, 0xF, true));
        upto += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(upto), 0x114, 0xF, 0xF, true));
        upto += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(upto), 0x118, 0xF, 0xF, true));
        if (G::kStepGroups == 32)                             // the first row's sum to the second row (and the third's to the fourth)
            upto += static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(upto), 0x142, 0xA, 0xF, false));
        unsigned char* const at = stage + (q_step + upto - size);
        const int group = lane - lane0;
        if (group >= 0 && group < G::kStepGroups && static_cast<unsigned>(h * G::kStepGroups + group) < groups_here) {
            if (W == 4) {
                *reinterpret_cast<unsigned*>(at) = mask;
            } else {
                *reinterpret_cast<unsigned short*>(at) = static_cast<unsigned short>(mask);
                *reinterpret_cast<unsigned short*>(at + 2) = static_cast<unsigned short>(mask >> 16);
            }
        }
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};

    // All of the wave's loads are in flight from the start (measured: 3-6 % over 8 KB at a
    // time), and each chunk is tested as it arrives.  They are buffer loads: what lies past
    // the tensor reads as zero without a test, so the wave that holds the tensor's end runs
    // the same instructions as the others.  (With loads and tests of its own, that wave,
    // usually the call's last, fetched several KB of code that no other wave had: 5.9 against
    // 4.8 us for a call of 64,000 fp32 elements, 1.5 to 6 us on every size that is not a
    // multiple of the tile.)
    // In the smallest fp32 tile a wave that lies wholly inside the tensor takes plain loads: a
    // call of a few tiles per CU waits for its first loads, and these need no descriptor (us,
    // cold whole-tile tensors of 4 | 6 | 8 MB: 6.6 | 7.3 | 7.8, with buffer loads alone 7.0 |
    // 7.8 | 8.1).  The larger tiles gain nothing from it (30 MB: 11.5 against 11.3).
    if (W == 4 && CH == 16 && __builtin_expect(wave_elem0 + G::kWaveElems <= a.n, 1)) {
        const unsigned* base = reinterpret_cast<const unsigned*>(a.in) + wave_dword0;
        static_for<0, CH>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            cur[k] = load_stream(base + k * kWaveSize + lane);
            __builtin_amdgcn_sched_barrier(0);   // in the order in which the tests use them
        });
    } else {
        // Aligned dwords from the one that holds the tensor's first element to the one that holds
        // its last.  SPLIT: the tensor begins in the middle of the first of them, so a lane's two
        // elements are the halves of two of them, its own and the next lane's.
        const size_t bytes = div_up(a.n * W + (SPLIT ? 2 : 0), size_t{4}) * 4, wave_byte0 = wave_dword0 * 4;
        const unsigned most = CH * kChunkBytes + (SPLIT ? 4 : 0);
        // (in words of 32 bits, which the scalar unit compares: with 64-bit comparisons on the vector
        // unit the descriptor takes 0.2 to 0.8 us longer where a call waits for its first loads)
        const size_t left = bytes - wave_byte0;
        const int left_high = static_cast<int>(left >> 32);
        const unsigned readable = left_high < 0 ? 0u : left_high > 0 ? most : min(static_cast<unsigned>(left), most);
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<unsigned char*>(a.in) - (SPLIT ? 2 : 0) + wave_byte0, 0, static_cast<int>(readable), kRawBuffer);
        // The descriptor's range check covers the vector and the immediate offset, not the scalar one,
        // which is zero throughout: the immediate reaches 16 chunks, a register each takes the lanes to
        // the next 16.
        int lane_byte[CH / 16];
#pragma unroll
        for (int j = 0; j < CH / 16; ++j) lane_byte[j] = 4 * lane + j * 16 * kChunkBytes;
        static_for<0, CH>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            cur[k] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, lane_byte[k / 16] + k % 16 * kChunkBytes, 0, kNonTemporal);
            __builtin_amdgcn_sched_barrier(0);   // in the order in which the tests use them
        });
        if constexpr (SPLIT)
            cur[CH] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, CH * kChunkBytes, 0, 0);
        // the second half of the last dword is not the tensor's
        const size_t half = a.n / 2;             // the dword with element n - 1 (n odd), or with element n in its first half
        if (W == 2 && (a.n & 1u) != (SPLIT ? 1u : 0u) && half >= wave_dword0 && half - wave_dword0 < CH * kWaveSize) {
            const unsigned last = static_cast<unsigned>(half - wave_dword0);
#pragma unroll
            for (int k = 0; k < CH; ++k)
                if (static_cast<unsigned>(k * kWaveSize + lane) == last) cur[k] &= 0xFFFFu;
        }
    }
    const unsigned long long scan_word = ScanState::ask(a.hdr);
    lds_barrier();                                // the cleared arrival word, after the loads have been issued

    // One of the first kFusedSteps steps is compacted in the same pass while the queue is sure
    // to hold it whatever its density (the first always is): the compaction then happens while
    // the wave would otherwise wait for its loads, and needs nothing from other tiles.
    int staged = 0;                               // steps in the queue so far, wave-uniform
    static_for<0, G::kSteps>([&](auto hc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
        if (h < kFusedSteps &&
            (G::kHoldsAll || (staged == h && q_end + G::kStepMaxBytes <= static_cast<unsigned>(G::kQueueBytes)))) {
            const unsigned q_step = q_end;
            static_for<h * kStepChunks, (h + 1) * kStepChunks>([&](auto kc) __attribute__((always_inline)) {
                chunk(kc, yes, yes);
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (WINDOWED) write_step_masks(hc, q_step);
            staged = h + 1;
        } else {
            static_for<h * kStepChunks, (h + 1) * kStepChunks>([&](auto kc) __attribute__((always_inline)) {
                chunk(kc, yes, no);
                __builtin_amdgcn_sched_barrier(0);
            });
        }
    });
    unsigned wave_total = 0;
#pragma unroll
    for (int h = 0; h < G::kSteps; ++h) wave_total += step_total[h];

    // ---- 2. arrival: the last wave of the tile to get here publishes the tile's count
    const ScanState scan(a.hdr, a.num_tiles, scan_word);
    unsigned arrived = 0;
    if (lane == 0) {
        s_wave_total[wave] = wave_total;
        arrived = arrive(&s_arrive, (1u << 24) | wave_total);
    }
    arrived = uniform(arrived);
    const bool publisher = (arrived >> 24) == WV - 1;
    if (publisher && lane == 0)
        scan.publish(tile, (arrived & 0xFFFFFFu) + wave_total);

    if constexpr (!WINDOWED && W == 2) {
#pragma unroll
        for (int r = 0; r < G::kMaskRegs; ++r) mask_reg[r] = zip_ballot_lanes(mask_reg[r], second_reg[r]);
    }
    if (!WINDOWED) {
#pragma unroll
        for (int r = 0; r < G::kMaskRegs; ++r) {
            const size_t g = wave_group0 + static_cast<size_t>(r) * kWaveSize + lane;
            if (r * kWaveSize + lane < G::kWaveGroups && g < a.num_groups)
                __builtin_nontemporal_store(mask_reg[r], a.masks + g);
        }
    }

    // ---- 3. more of the compaction before the tile knows where its run begins: the steps left
    //         for now, and those that were not sure to fit but, now that their size is known, do
    const auto step_bytes = [&](int h) -> unsigned {
        return step_total[h] * W + (WINDOWED ? 4u * G::kStepGroups : 0u);
    };
    const auto stage_step = [&](auto hc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
        const unsigned q_step = q_end;
        static_for<h * kStepChunks, (h + 1) * kStepChunks>([&](auto kc) __attribute__((always_inline)) {
            chunk(kc, no, yes);
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (WINDOWED) write_step_masks(hc, q_step);
    };
    static_for<0, G::kSteps>([&](auto hc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
        if (G::kHoldsAll ? h >= kFusedSteps : staged == h && q_end + step_bytes(h) <= static_cast<unsigned>(G::kQueueBytes)) {
            stage_step(hc);
            staged = h + 1;
        }
    });

    // ---- 4. device-wide exclusive scan, wave 0
    if (wave == 0) {
        unsigned long long ex = 0;
        if (tile != 0) {
            const CountInputTile<W, CH, WV, RELU, SPLIT> count_tile{a.in, a.n};
            // (the smallest windowed tile has been staging its steps since it published its count: 1 MB fp32 4.92
            // us, with the pause 5.00; 30 MB 16-bit 14.15 | 14.23)
            ex = scan_exclusive_prefix<WINDOWED && CH == 16 ? kNoPause : 0>(scan, tile, lane, count_tile);
        }
        if (lane == 0) s_prefix = ex;
    }
    lds_barrier();
    const unsigned long long exclusive = uniform(s_prefix);
    unsigned wave_offset = 0, tile_total = 0;
#pragma unroll
    for (int v = 0; v < WV; ++v) {
        const unsigned t = uniform(s_wave_total[v]);
        if (v < wave) wave_offset += t;
        tile_total += t;
    }
    if (wave == 0 && lane == 0 && scan.ends_block(tile)) scan.publish_prefix(tile, exclusive + tile_total);

    //      A call with a buffer below the worst case (cap_values) writes a tile's
    //      run only if the run ends inside the buffer; the size is reported anyway.
    const unsigned long long tile_end_bytes =
        (exclusive + tile_total) * W +
        (WINDOWED ? 4ull * min(static_cast<size_t>(tile + 1) * G::kTileGroups, a.num_groups) : 0ull);
    if (tile_end_bytes <= a.cap_values) {
        unsigned char* const run_begin =
            a.values + (exclusive + wave_offset) * W +
            (WINDOWED ? 4 * (wave_group0 < a.num_groups ? wave_group0 : a.num_groups) : 0);
        unsigned char* gzero = run_begin;
        if (G::kHoldsAll || staged != 0) {
            if (WINDOWED) q_end = queue_end(0u, G::kHoldsAll ? G::kSteps : staged);
            wave_flush<W>(gzero, stage, q_lo, q_end, G::kHoldsAll || staged == G::kSteps, lane);
            zero_local = static_cast<unsigned>(gzero - run_begin);
            wave_lds_sync();
        }
        static_for<0, G::kSteps>([&](auto hc) __attribute__((always_inline)) {
            constexpr int h = decltype(hc)::value;
            if (!G::kHoldsAll && h >= staged) {
                stage_step(hc);
                if (WINDOWED) q_end = queue_end(h, h + 1);
                wave_lds_sync();
                wave_flush<W>(gzero, stage, q_lo, q_end, h == G::kSteps - 1, lane);
                zero_local = static_cast<unsigned>(gzero - run_begin);
                wave_lds_sync();
            }
        });
        if (WINDOWED && lane < CH / kWindowChunks) {
            // the byte offset of every window that exists: its masks before it, its kept elements before it
            const size_t unit = wave_group0 / (kWindowChunks * CG) + lane;     // 1 KB of input
            if (wave_group0 + static_cast<size_t>(lane) * (kWindowChunks * CG) < a.num_groups &&
                (unit & ((size_t{1} << a.window_shift) - 1)) == 0)
                a.offsets[unit >> a.window_shift] =
                    static_cast<unsigned long long>(run_begin - a.values) + window_local;
        }
    }

    // ---- section 5.4: the compressed size, reported by the last tile
    if (tile == a.num_tiles - 1 && tid == 0) {
        const unsigned long long total =
            4ull * a.num_groups + static_cast<unsigned long long>(W) * (exclusive + tile_total);
        *a.d_bytes = total;
        if (a.h_bytes != nullptr) __hip_atomic_store(a.h_bytes, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        if (WINDOWED)
            a.offsets[div_up(a.num_groups, static_cast<size_t>(kWindowChunks * CG) << a.window_shift)] = total;
    }

    if (tile == a.num_tiles - 1 && wave == 0)
        scan_end(scan, a.num_tiles, lane);
}

// With more than 80 scalar registers a SIMD holds seven waves, not eight, and the scan's state would make them 82 to 92.  us with
// them | with 80: windowed 16-bit 30 MB 15.05 | 14.7, 100 MB 37.6 | 36.8, 300 MB 89.5 | 87.2, fp32 64 MB 19.0 | 18.3; 16-bit 100 MB
// 32.0 | 32.6, 300 MB 82.4 | 81.6; decoding 16-bit 40 MB 13.3 | 13.0.  Not where a tile is staged early, which
// takes up to 106 and would save and reload them (fp32 24 MB 9.1 | 9.4).
#define ZVC_EIGHT_WAVES __attribute__((amdgpu_num_sgpr(80)))
#define ZVC_EIGHT_WAVES_ENCODER(W, CH, RELU, WINDOWED, SPLIT) \
    template __global__ ZVC_EIGHT_WAVES void compress_kernel<W, CH, 4, RELU, WINDOWED, SPLIT, false>(EncoderArgs)
#define ZVC_EIGHT_WAVES_ENCODERS(W, CH, SPLIT)                 \
    ZVC_EIGHT_WAVES_ENCODER(W, CH, false, false, SPLIT);       \
    ZVC_EIGHT_WAVES_ENCODER(W, CH, true, false, SPLIT);        \
    ZVC_EIGHT_WAVES_ENCODER(W, CH, false, true, SPLIT)
ZVC_EIGHT_WAVES_ENCODERS(2, 16, false);
ZVC_EIGHT_WAVES_ENCODERS(2, 16, true);
ZVC_EIGHT_WAVES_ENCODERS(2, 32, false);
ZVC_EIGHT_WAVES_ENCODERS(2, 32, true);
ZVC_EIGHT_WAVES_ENCODER(4, 16, false, true, false);
ZVC_EIGHT_WAVES_ENCODER(4, 32, false, true, false);

// Decoder pre-pass (section 5.2: the popcount of a mask span is the number of
// stored words the span consumes).  Where a span's stored elements start
// depends on the masks alone, which are 1/32 (fp32) or 1/16 (16-bit) of the
// tensor, so it is computed ahead of the decoder, whose waves then depend on
// nothing but their own part of the stream.  One workgroup takes a chunk of
// kChunkMasks consecutive masks with coalesced 16-byte loads and writes
//   unit_end[u]    = stored elements of the chunk up to and including unit u
//                    (a unit is 32 masks, 1024 elements),
//   chunk_total[c] = stored elements of the chunk.
// Unless chunk_prefix is null (few chunks, see kFewChunks), the workgroup that
// finishes last (arrival counters in the header, which it also resets) turns
// the totals into chunk_prefix[c] = stored elements before chunk c.
constexpr int kUnitMasks = 32;
constexpr int kChunkLoads = 4;                                 // 16-byte loads per thread
constexpr int kChunkMasks = kThreads * 4 * kChunkLoads;        // 4096 masks = 131072 elements
constexpr int kChunkUnits = kChunkMasks / kUnitMasks;          // 128
constexpr int kUnitLanes = kUnitMasks / 4;                     // 8 lanes of one load cover a unit
// Up to this many chunks (134M elements) the expand kernel's workgroups each add
// up the chunk totals before their own chunk; above, the pre-pass does it once.
constexpr unsigned kFewChunks = 1024;

__global__ __launch_bounds__(kThreads) void mask_prefix_kernel(
    const unsigned* __restrict__ masks, size_t num_groups, unsigned tail,
    unsigned* __restrict__ unit_end, unsigned* chunk_total,
    unsigned long long* __restrict__ chunk_prefix, WsHeader* hdr, unsigned num_chunks) {
    __shared__ unsigned s_unit[kChunkUnits];
    __shared__ unsigned s_wave_total[2];
    __shared__ unsigned long long s_wave_sum[kWaves];
    __shared__ unsigned s_last;
    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = tid / kWaveSize;
    const unsigned chunk = blockIdx.x;
    const size_t g_chunk = static_cast<size_t>(chunk) * kChunkMasks;

    // ---- load k covers masks [g_chunk + 1024 k, + 1024): 4 per thread, 4 KB per workgroup
    unsigned c[kChunkLoads];
    const bool whole = g_chunk + kChunkMasks <= num_groups &&
                       !(g_chunk + kChunkMasks == num_groups && tail != 0) &&
                       (reinterpret_cast<uintptr_t>(masks) & 15u) == 0;
    if (whole) {
#pragma unroll
        for (int k = 0; k < kChunkLoads; ++k) {
            const uint4 v = *reinterpret_cast<const uint4*>(masks + g_chunk + 1024 * k + 4 * tid);
            c[k] = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
        }
    } else {
#pragma unroll 1
        for (int k = 0; k < kChunkLoads; ++k) {
            unsigned sum = 0;
            for (int i = 0; i < 4; ++i) {
                const size_t g = g_chunk + 1024 * k + 4 * tid + i;
                if (g < num_groups) {
                    unsigned m = masks[g];
                    if (g == num_groups - 1 && tail != 0) m &= (1u << tail) - 1u;  // bits past n never count
                    sum += __popc(m);
                }
            }
            c[k] = sum;
        }
    }
    // ---- unit sums: 8 consecutive lanes of one load, two loads packed per register
    //      (a unit holds at most 1024 set bits)
#pragma unroll
    for (int q = 0; q < kChunkLoads / 2; ++q) {
        unsigned p = c[2 * q] | (c[2 * q + 1] << 16);
#pragma unroll
        for (int off = 1; off < kUnitLanes; off <<= 1) p += __shfl_xor(p, off);
        if (tid % kUnitLanes == 0) {
            s_unit[(2 * q) * (kThreads / kUnitLanes) + tid / kUnitLanes] = p & 0xFFFFu;
            s_unit[(2 * q + 1) * (kThreads / kUnitLanes) + tid / kUnitLanes] = p >> 16;
        }
    }
    __syncthreads();
    // ---- inclusive scan of the 128 unit sums (waves 0 and 1)
    const unsigned v = tid < kChunkUnits ? s_unit[tid] : 0u;
    unsigned incl = v;
#pragma unroll
    for (int off = 1; off < kWaveSize; off <<= 1) {
        const unsigned t = __shfl_up(incl, off);
        if (lane >= off) incl += t;
    }
    if (lane == kWaveSize - 1 && wave < 2) s_wave_total[wave] = incl;
    __syncthreads();
    if (tid < kChunkUnits)
        unit_end[static_cast<size_t>(chunk) * kChunkUnits + tid] =
            incl + (wave == 1 ? s_wave_total[0] : 0u);

    // ---- few chunks: the expand kernel's workgroups add up the totals before theirs
    //      themselves (a KB or so from L2 each), which costs less than the two memory
    //      round trips below
    if (chunk_prefix == nullptr) {
        if (tid == 0) chunk_total[chunk] = s_wave_total[0] + s_wave_total[1];
        return;
    }
    // ---- the last workgroup to get here prefixes the chunk totals
    if (tid == 0) {
        store32(chunk_total + chunk, s_wave_total[0] + s_wave_total[1]);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the total is out before the count moves
        // atomics on one address cost about 11 ns each here, so the arrivals are
        // spread over 64 counters with one on top
        const unsigned slot = chunk % kFinishLanes;
        const unsigned quota = num_chunks / kFinishLanes + (slot < num_chunks % kFinishLanes ? 1u : 0u);
        unsigned last = 0;
        if (atomicAdd(&hdr->finish[slot].value, 1u) == quota - 1) {
            const unsigned slots_used = num_chunks < kFinishLanes ? num_chunks : kFinishLanes;
            last = atomicAdd(&hdr->finish_top.value, 1u) == slots_used - 1 ? 1u : 0u;
        }
        s_last = last;
    }
    __syncthreads();
    if (s_last == 0u) return;
    // 8 consecutive totals per thread and round, all loads of a round in flight together
    constexpr int kPerThread = 8;
    unsigned long long carry = 0;
    for (size_t base = 0; base < num_chunks; base += kThreads * kPerThread) {
        const size_t c0 = base + static_cast<size_t>(tid) * kPerThread;   // chunk_total is 256-byte aligned
        unsigned long long pair[kPerThread / 2];
#pragma unroll
        for (int k = 0; k < kPerThread / 2; ++k)
            pair[k] = c0 + 2 * k < num_chunks
                          ? load64(reinterpret_cast<const unsigned long long*>(chunk_total + c0 + 2 * k))
                          : 0ull;
        unsigned t[kPerThread];
        unsigned long long mine = 0;
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            t[k] = c0 + k < num_chunks ? static_cast<unsigned>(pair[k / 2] >> (32 * (k % 2))) : 0u;
            mine += t[k];
        }
        unsigned long long inc = mine;
#pragma unroll
        for (int off = 1; off < kWaveSize; off <<= 1) {
            const unsigned long long up = __shfl_up(inc, off);
            if (lane >= off) inc += up;
        }
        __syncthreads();   // s_wave_sum of the previous round has been read
        if (lane == kWaveSize - 1) s_wave_sum[wave] = inc;
        __syncthreads();
        unsigned long long before = carry + inc - mine, all = 0;
#pragma unroll
        for (int w2 = 0; w2 < kWaves; ++w2) {
            const unsigned long long ws = s_wave_sum[w2];
            if (w2 < wave) before += ws;
            all += ws;
        }
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            if (c0 + k < num_chunks) chunk_prefix[c0 + k] = in_halves(before);
            before += t[k];
        }
        carry += all;
    }
    // ready for the next call
    if (tid < kFinishLanes) hdr->finish[tid].value = 0u;
    if (tid == 0) hdr->finish_top.value = 0u;
}

// How an output is written.  kAligned: 16 bytes a lane from a 16-byte boundary on.  kLoose: the same from
// any element.  kShifted: pieces begin with a line of the output, see PieceShift.
enum class Output { kAligned, kLoose, kShifted };

// 4 KB of output by one wave: 16 bytes per lane and store, which `piece(jj)` rebuilds for the jj-th
// store.  Of the output only elements 0 .. left - 1 are the tensor's (`left` is the same in all lanes).
template <int W, bool ALIGNED, class Piece>
__device__ __forceinline__ void store_piece(const Piece& piece, unsigned left, unsigned char* __restrict__ to, int lane) {
    constexpr int E = Geometry<W, kMinLoads>::kElemsPerLane;
    const bool whole = left >= kStageLoads * kWaveSize * E;             // uniform
    uint4 v[kStageLoads];
#pragma unroll
    for (int jj = 0; jj < kStageLoads; ++jj) {
        v[jj] = piece(jj);
        if (__builtin_expect(whole, 1)) {
            if (ALIGNED) store16_stream(to + (jj * kWaveSize + lane) * 16, v[jj]);
            else store16_loose<W>(to + (jj * kWaveSize + lane) * 16, v[jj]);
        }
        // Each store goes as soon as its 16 bytes are there: all four at the end cost the largest
        // tensors about 1 % (822 MB fp32 at density 0.5: 210.4 us against 207.8).
        __builtin_amdgcn_sched_barrier(0);
    }
    if (__builtin_expect(whole, 1)) return;
#pragma unroll
    for (int jj = 0; jj < kStageLoads; ++jj) {
        const unsigned e0 = static_cast<unsigned>(jj * kWaveSize + lane) * E;
        if (e0 + E <= left) {
            if (ALIGNED) store16_stream(to + e0 * W, v[jj]);
            else store16_loose<W>(to + e0 * W, v[jj]);
        } else if (e0 < left) {                                         // the tensor's last elements
            const unsigned d[4] = {v[jj].x, v[jj].y, v[jj].z, v[jj].w};
#pragma unroll
            for (int c = 0; c + 1 < E; ++c) {
                if (e0 + c < left) {
                    if (W == 4) reinterpret_cast<unsigned*>(to)[e0 + c] = d[c];
                    else reinterpret_cast<unsigned short*>(to)[e0 + c] = static_cast<unsigned short>(d[c >> 1] >> (16 * (c & 1)));
                }
            }
        }
    }
}

// A piece that begins with a mask's first bit: lane i holds mask i of the 32 (64) and the offset in `lds`
// of its first stored element.  `lds` begins with 16 bytes that belong to nothing else.
template <int W, bool ALIGNED>
__device__ __forceinline__ void expand_piece(unsigned char* lds, unsigned mask, unsigned mask_at, unsigned left,
                                             unsigned char* __restrict__ to, int lane) {
    using G = Geometry<W, kMinLoads>;
    constexpr int LPG = G::kLanesPerGroup;
    // (every wave writes the zeros itself: LDS operations of one wave execute in order)
    if (lane == 0) *reinterpret_cast<uint4*>(lds) = make_uint4(0u, 0u, 0u, 0u);
    wave_lds_sync();
    const unsigned bit0 = static_cast<unsigned>(lane % LPG) * G::kElemsPerLane, lower = (1u << bit0) - 1u;
    const auto piece = [&](int jj) __attribute__((always_inline)) -> uint4 {
        const int from = 4 * (jj * G::kGroupsPerLoad + lane / LPG);     // the lane's mask
        const unsigned gm = static_cast<unsigned>(__builtin_amdgcn_ds_bpermute(from, static_cast<int>(mask)));
        const unsigned at = static_cast<unsigned>(__builtin_amdgcn_ds_bpermute(from, static_cast<int>(mask_at)));
        return expand_lane<W>(lds, at + W * static_cast<unsigned>(__popc(gm & lower)), gm >> bit0);
    };
    store_piece<W, ALIGNED>(piece, left, to, lane);
}

// The same for a piece that begins with bit `bits` of lane 0's mask.  Lane i holds mask i of the piece and,
// in `next`, the one behind; the stored elements of all masks follow each other in `lds`.  `to` is the
// beginning of a line.
template <int W>
__device__ __forceinline__ void expand_shifted_piece(unsigned char* lds, unsigned mask, unsigned mask_at, unsigned next,
                                                     unsigned bits, unsigned left, unsigned char* __restrict__ to, int lane) {
    using G = Geometry<W, kMinLoads>;
    constexpr int E = G::kElemsPerLane;
    constexpr int LPG = G::kLanesPerGroup;
    if (lane == 0) *reinterpret_cast<uint4*>(lds) = make_uint4(0u, 0u, 0u, 0u);
    wave_lds_sync();
    // the lane's elements begin with bit `bit0` of its mask and the next, taken as one word of 64 bits
    const unsigned bit0 = static_cast<unsigned>(lane % LPG) * E + bits;              // below 64 - E
    const unsigned long long lower = (1ull << bit0) - 1ull;
    const unsigned lower_mask = static_cast<unsigned>(lower), lower_next = static_cast<unsigned>(lower >> 32);
    const auto piece = [&](int jj) __attribute__((always_inline)) -> uint4 {
        const int from = 4 * (jj * G::kGroupsPerLoad + lane / LPG);
        const unsigned gm = static_cast<unsigned>(__builtin_amdgcn_ds_bpermute(from, static_cast<int>(mask)));
        const unsigned gn = static_cast<unsigned>(__builtin_amdgcn_ds_bpermute(from, static_cast<int>(next)));
        const unsigned at = static_cast<unsigned>(__builtin_amdgcn_ds_bpermute(from, static_cast<int>(mask_at)));
        const unsigned before = static_cast<unsigned>(__popc(gm & lower_mask)) + static_cast<unsigned>(__popc(gn & lower_next));
        const unsigned long long both = static_cast<unsigned long long>(gn) << 32 | gm;
        return expand_lane<W>(lds, at + W * before, static_cast<unsigned>(both >> bit0));
    };
    store_piece<W, true>(piece, left, to, lane);
}

// `total` stored elements from element `first` of the value area on into LDS, by one wave, with aligned
// 16-byte loads; what lies past values_avail elements reads as zero.  `lds` + `slice` is 16-byte aligned;
// the run begins `shift` bytes behind it.  In two parts, so that the caller has something to do meanwhile.
template <int W>
struct StagedRun {
    unsigned shift, valid, wanted;         // bytes
    __device__ __forceinline__ StagedRun(unsigned char* at, const unsigned char* __restrict__ values,
                                         unsigned long long values_avail, unsigned long long first, unsigned total,
                                         bool stream_values, int lane) {
        const unsigned char* src = values + first * W;
        shift = static_cast<unsigned>(reinterpret_cast<uintptr_t>(src) & 15u);
        unsigned long long readable = values_avail > first ? values_avail - first : 0ull;
        if (readable > total) readable = total;
        wanted = total * W;
        valid = static_cast<unsigned>(readable) * W;
        const unsigned end = valid != 0u ? shift + valid : 0u;
        if (stream_values) wave_stage<true>(at, src - shift, end, lane);
        else wave_stage<false>(at, src - shift, end, lane);
    }
    __device__ __forceinline__ void wait(unsigned char* at, int lane) const {
        stage_wait();
        if (__builtin_expect(valid < wanted, 0)) {           // the stream is cut short
            wave_lds_sync();
            for (unsigned i = shift + valid + W * lane; i < shift + wanted; i += W * kWaveSize) {
                if (W == 4) *reinterpret_cast<unsigned*>(at + i) = 0u;
                else *reinterpret_cast<unsigned short*>(at + i) = 0;
            }
        }
    }
};

// One step of the decoder, by one wave: 4 KB of output from `m` (lane i holds
// the step's mask i, bits past n cleared) and the step's `step_total` stored
// elements, which begin at element `first` of the value area.  Stages them in
// the wave's slice of `lds` (at offset `slice`; see expand_piece) with aligned 16-byte
// loads, never past values_avail elements: anything the masks ask for beyond that
// decodes as zero.  `first`, `step_total` and `slice` are the same in all lanes.
template <int W, bool ALIGNED>
__device__ __forceinline__ void expand_step(unsigned char* lds, unsigned slice, const unsigned char* __restrict__ values,
                                            unsigned long long values_avail, unsigned long long first,
                                            unsigned step_total, unsigned m, size_t wave_elem0, size_t n,
                                            unsigned char* __restrict__ out, bool stream_values, int lane) {
    using G = Geometry<W, kMinLoads>;
    constexpr int kStepMasks = kStageLoads * G::kGroupsPerLoad;   // 32 | 64 masks per step
    constexpr unsigned kStepElems = kStageLoads * kWaveSize * G::kElemsPerLane;
    const StagedRun<W> run(lds + slice, values, values_avail, first, step_total, stream_values, lane);
    // stored elements of the step before each of its masks, while the loads are under way
    const unsigned cnt = static_cast<unsigned>(__popc(m));
    const unsigned mask_at = slice + run.shift + W * (wave_scan_small<kStepMasks>(cnt) - cnt);
    run.wait(lds + slice, lane);
    const unsigned left = n - wave_elem0 < kStepElems ? static_cast<unsigned>(n - wave_elem0) : kStepElems;
    expand_piece<W, ALIGNED>(lds, m, mask_at, left, out + wave_elem0 * W, lane);
}

// Outputs that do not begin with a 128-byte line.  A wave that writes from a group's beginning on then
// shares the lines at both ends of each of its stores with other stores, and where the output is not
// 16-byte aligned every store is split as well.  So a wave's piece begins SHIFT elements later, SHIFT the
// elements up to the first line: its masks then begin with bit SHIFT mod 32 and end in the mask behind,
// and the first wave writes the SHIFT elements before the first piece.  us, stores that follow the
// output's alignment | shifted, at an odd element: fp16 52 MB 19.3 | 17.6 (aligned: 16.6); fp32 100 MB 32.9 | 25.9,
// 300 MB 80.8 | 74.9 (71.4), 784 MB 238 | 206, of density 0.05 201 | 136.  planar_output() says which are shifted.
constexpr unsigned kLineBytes = 128;
template <int W>
struct PieceShift {
    using G = Geometry<W, kMinLoads>;
    static constexpr int kStepMasks = kStageLoads * G::kGroupsPerLoad;       // 32 | 64
    unsigned elements, groups, bits;                 // bits: of the first mask that belong to the piece before
    __device__ explicit PieceShift(const unsigned char* out) {
        elements = static_cast<unsigned>(-reinterpret_cast<uintptr_t>(out) % kLineBytes) / W;
        groups = elements / 32u;                     // 0 | 0 or 1
        bits = elements % 32u;
    }
};
// Lane i's masks for a shifted piece that begins with mask g0 before the shift: mask g0 + i, the mask that
// the piece has there, and the one behind that.  `masks_of(g)`: mask g, 0 past the tensor's end.
template <int W, class MasksOf>
struct ShiftedMasks {
    unsigned own, mask, next;
    __device__ __forceinline__ ShiftedMasks(const PieceShift<W>& shift, size_t g0, int lane, const MasksOf& masks_of) {
        own = masks_of(g0 + lane);
        next = masks_of(g0 + 1 + lane);
        mask = own;
        if (W == 2 && shift.groups != 0) {           // uniform
            mask = next;
            next = masks_of(g0 + 2 + lane);
        }
    }
};

// expand_step for a shifted piece: `first` is the stored element that the piece's first mask begins
// with (its bits before the piece included).
template <int W>
__device__ __forceinline__ void expand_shifted_step(unsigned char* lds, unsigned slice,
                                                    const unsigned char* __restrict__ values,
                                                    unsigned long long values_avail, unsigned long long first,
                                                    unsigned mask, unsigned next, const PieceShift<W>& shift,
                                                    size_t elem0, size_t n, unsigned char* __restrict__ out,
                                                    bool stream_values, int lane) {
    using G = Geometry<W, kMinLoads>;
    constexpr int kStepMasks = kStageLoads * G::kGroupsPerLoad;
    constexpr unsigned kStepElems = kStageLoads * kWaveSize * G::kElemsPerLane;
    const unsigned cnt = lane < kStepMasks ? static_cast<unsigned>(__popc(mask)) : 0u;
    const unsigned upto = wave_scan_small<kStepMasks>(cnt);
    const unsigned total = lane_value(upto, kStepMasks - 1) +
                           static_cast<unsigned>(__popc(lane_value(next, kStepMasks - 1) & ((1u << shift.bits) - 1u)));
    const StagedRun<W> run(lds + slice, values, values_avail, first, total, stream_values, lane);
    const unsigned left = n - elem0 < kStepElems ? static_cast<unsigned>(n - elem0) : kStepElems;
    run.wait(lds + slice, lane);
    expand_shifted_piece<W>(lds, mask, slice + run.shift + W * (upto - cnt), next, shift.bits, left, out + elem0 * W, lane);
}

// The elements before the first piece, by the first wave: a lane each.
template <int W>
__device__ inline void expand_head(const unsigned char* __restrict__ values, unsigned long long values_avail, unsigned mask0,
                                   unsigned mask1, unsigned count, unsigned char* __restrict__ out, int lane) {
    if (static_cast<unsigned>(lane) >= count) return;
    const unsigned mask = lane < 32 ? mask0 : mask1, bit = static_cast<unsigned>(lane) % 32u;
    const unsigned at = (lane < 32 ? 0u : static_cast<unsigned>(__popc(mask0))) +
                        static_cast<unsigned>(__popc(mask & ((1u << bit) - 1u)));
    const bool stored = (mask >> bit & 1u) != 0u && at < values_avail;
    if (W == 4) reinterpret_cast<unsigned*>(out)[lane] = stored ? reinterpret_cast<const unsigned*>(values)[at] : 0u;
    else reinterpret_cast<unsigned short*>(out)[lane] = stored ? reinterpret_cast<const unsigned short*>(values)[at] : 0;
}

// A wave's part of a shifted output: its piece and, for the first wave, what lies before it.  `first` is the
// first stored element of the part before the shift, whose masks are `own`.
template <int W>
__device__ __forceinline__ void expand_shifted(unsigned char* lds, unsigned slice, const unsigned char* __restrict__ values,
                                               unsigned long long values_avail, unsigned long long first, unsigned own,
                                               unsigned mask, unsigned next, const PieceShift<W>& shift, size_t elem0, size_t n,
                                               unsigned char* __restrict__ out, bool stream_values, int lane) {
    if (elem0 == 0 && shift.elements != 0)
        expand_head<W>(values, values_avail, lane_value(own, 0), lane_value(own, 1),
                       shift.elements, out, lane);      // (a shifted output is larger than that, see planar_output)
    if (elem0 + shift.elements >= n) return;
    if (W == 2 && shift.groups != 0) first += static_cast<unsigned>(__popc(lane_value(own, 0)));
    expand_shifted_step<W>(lds, slice, values, values_avail, first, mask, next, shift, elem0 + shift.elements, n, out,
                           stream_values, lane);
}

// Mask g of the tensor: none past its end, and bits past n never count (tail = n % 32).
__device__ __forceinline__ auto masks_within(const unsigned* __restrict__ masks, size_t num_groups, unsigned tail) {
    return [=](size_t g) __attribute__((always_inline)) -> unsigned {
        unsigned v = 0;
        if (g < num_groups) {
            v = masks[g];
            if (tail != 0 && g == num_groups - 1) v &= (1u << tail) - 1u;
        }
        return v;
    };
}

// Section 5.2 decoder.  Every wave works on its own: it expands one step, 4 KB
// of output, and knows from the pre-pass where the step's stored elements begin
// and end (expand_step does the rest).
template <int W, int LOADS, Output OUTPUT>
__global__ __launch_bounds__(kThreads) void decompress_kernel(
    const unsigned* __restrict__ masks, const unsigned char* __restrict__ values,
    unsigned long long values_avail, size_t n, unsigned char* __restrict__ out,
    const unsigned* __restrict__ unit_end, const unsigned long long* __restrict__ chunk_prefix,
    const unsigned* __restrict__ chunk_total, size_t num_groups, bool stream_values, bool interleave) {
    using G = Geometry<W, LOADS>;
    constexpr int E = G::kElemsPerLane;
    constexpr int kStepMasks = kStageLoads * G::kGroupsPerLoad;   // 32 | 64 masks per step
    constexpr int kStepUnits = kStepMasks / kUnitMasks;           // 1 | 2
    constexpr int kSteps = G::kStageSteps;
    static_assert(kChunkMasks % (LOADS * G::kGroupsPerLoad) == 0, "a wave's masks lie in one chunk");

    __shared__ __align__(16) unsigned char s_stage[16 + kWaves * G::kWaveStageBytes];   // (16: see expand_piece)

    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = static_cast<int>(uniform(static_cast<unsigned>(tid / kWaveSize)));
    const unsigned tile = blockIdx.x;
    // Which part of the tensor (LOADS KB) the wave expands.  In a row: workgroup i
    // takes parts 4i .. 4i+3, so the eight XCDs (workgroup i runs on XCD i mod 8)
    // write 16 KB apiece side by side.  Interleaved: the waves of workgroup i take
    // parts that are i mod 8 modulo 8, so the XCDs write neighbouring 4 KB blocks at
    // the same time.  The memory system takes a stream of writes with few reads
    // among them up to 15 % faster in the second order (the host chooses).
    const size_t part = interleave ? (static_cast<size_t>(tile / 8) * kWaves + wave) * 8 + tile % 8
                                   : static_cast<size_t>(tile) * kWaves + wave;
    const size_t wave_elem0 = part * (static_cast<size_t>(LOADS) * kWaveSize * E);
    const size_t wave_group0 = wave_elem0 / 32;
    const size_t chunk = wave_group0 / kChunkMasks;     // the same for all waves of the workgroup
    const unsigned tail = static_cast<unsigned>(n % 32);

    // ---- few chunks: the workgroup adds up the totals of the chunks before its own.  These loads go
    //      out first, they are waited for first; the masks' latency then hides behind the sum (17.5
    //      -> 17.0 us for 51 MB bf16, 79.2 -> 78.7 for 297 MB fp32; with the masks
    //      asked for first 8 M fp32 elements take 12.5 us instead of 12.0)
    static_assert(kFewChunks == 4 * kThreads, "four totals per thread");
    unsigned total = 0;                            // of chunks with at most 2^17 stored elements each
    if (chunk_prefix == nullptr) {
        const unsigned before = static_cast<unsigned>(
            min(chunk, div_up(num_groups, static_cast<size_t>(kChunkMasks))));   // (a workgroup past the tensor's end)
        const unsigned c = 4u * tid;               // (the array is padded to whole 256 bytes)
        if (c < before) {
            const uint4 t = *reinterpret_cast<const uint4*>(chunk_total + c);
            total = t.x + (c + 1u < before ? t.y : 0u) + (c + 2u < before ? t.z : 0u) + (c + 3u < before ? t.w : 0u);
        }
    }
    // ---- the step's masks and where it begins and ends within its chunk, on their way meanwhile
    static_assert(kSteps == 1, "a wave expands one step");
    unsigned m = 0, next = 0, own = 0, step_begin = 0, step_end = 0;
    const PieceShift<W> shift(out);
    if (wave_elem0 < n) {
        const auto mask_of = masks_within(masks, num_groups, tail);
        if constexpr (OUTPUT != Output::kShifted) {
            if (lane < kStepMasks) m = mask_of(wave_group0 + lane);
        } else {
            const ShiftedMasks<W, decltype(mask_of)> got(shift, wave_group0, lane, mask_of);
            m = got.mask;
            next = got.next;
            own = got.own;
        }
        const size_t u = wave_group0 / kUnitMasks;
        step_begin = u % kChunkUnits != 0 ? unit_end[u - 1] : 0u;
        if (OUTPUT != Output::kShifted) step_end = unit_end[u + kStepUnits - 1];
    }

    // ---- stored elements before the wave's chunk: the sum (below 2^27), or from the pre-pass
    unsigned long long before_chunk = 0;
    if (chunk_prefix == nullptr) {
        __shared__ __align__(16) unsigned s_before[kWaves];
        static_assert(sizeof(s_stage) + sizeof(s_before) == G::kDecodeLdsBytes, "as the host counts it");
        const unsigned wave_part = wave_sum_small(total);
        if (lane == 0) s_before[wave] = wave_part;
        lds_barrier();
        unsigned sum = 0;
#pragma unroll
        for (int v = 0; v < kWaves; ++v) sum += s_before[v];
        before_chunk = uniform(sum);
    }
    if (wave_elem0 >= n) return;                  // nothing of the tensor in this wave's part
    if (chunk_prefix != nullptr) before_chunk = from_halves(chunk_prefix[chunk]);

    if constexpr (OUTPUT != Output::kShifted) {
        expand_step<W, OUTPUT == Output::kAligned>(s_stage, 16u + wave * G::kWaveStageBytes, values, values_avail, before_chunk + step_begin,
                       step_end - step_begin, m, wave_elem0, n, out, stream_values, lane);
    } else {
        expand_shifted<W>(s_stage, 16u + wave * G::kWaveStageBytes, values, values_avail, before_chunk + step_begin, own, m,
                          next, shift, wave_elem0, n, out, stream_values, lane);
    }
}

// The same decoder in one launch, for small tensors: no pre-pass.  A workgroup
// expands 16 or 32 KB of output, in stream order.  Where its stored elements begin is
// the number of set bits in all masks before its own, which it gets the way the
// encoder's tiles get their offsets: it publishes the popcount of its own
// masks and runs the device-wide scan over the workgroups before it
// (scan_exclusive_prefix; same scan state in the workspace, same numbers, same
// self-help if a predecessor has not been dispatched).  A
// workgroup knows its count after one small load, so the scan's chain is short;
// below a few tens of megabytes one launch beats the pre-pass's extra kernel,
// above that the pre-pass wins because its expand kernel touches no shared state.
struct CountMaskTile {
    const unsigned* masks;
    size_t num_groups;
    unsigned tail;                 // n % 32
    int tile_masks;                // masks per workgroup: 128 to 512
    // set bits in the masks of workgroup q, wave-uniform
    __device__ unsigned operator()(unsigned q, int lane) const {
        unsigned count = 0;
        for (int i = lane; i < tile_masks; i += kWaveSize) {
            const size_t g = static_cast<size_t>(q) * tile_masks + i;
            if (g < num_groups) {
                unsigned m = __builtin_nontemporal_load(masks + g);
                if (g == num_groups - 1 && tail != 0) m &= (1u << tail) - 1u;
                count += __popc(m);
            }
        }
        return wave_sum_small(count);
    }
};

//
// STREAM: the stored elements are read with the streaming hint.  A template's parameter, because the code of both ways
// in one kernel (6.2 KB for 5.8) is fetched on every call: us with the same pause, both | one, fp32 3 MB 4.59 | 4.39, 6.4 MB 4.95 |
// 4.71, 16-bit 3 MB 4.74 | 4.60, at an odd element 51 MB 16.2 | 16.0.
template <int W, Output OUTPUT, int WV, bool STREAM>
__global__ __launch_bounds__(WV * kWaveSize) ZVC_EIGHT_WAVES void decompress_scan_kernel(
    const unsigned* __restrict__ masks, const unsigned char* __restrict__ values,
    unsigned long long values_avail, size_t n, unsigned char* __restrict__ out, WsHeader* hdr,
    unsigned num_tiles, size_t num_groups) {
    using G = Geometry<W, kMinLoads>;
    constexpr int E = G::kElemsPerLane;
    constexpr int kStepMasks = kStageLoads * G::kGroupsPerLoad;   // masks per wave: 32 | 64
    static_assert(G::kStageSteps == 1, "a wave expands one step");

    __shared__ __align__(16) unsigned char s_stage[16 + WV * G::kWaveStageBytes];   // (16: see expand_piece)
    __shared__ unsigned s_wave_total[WV];
    __shared__ unsigned s_arrive;                 // waves arrived << 24 | set bits so far
    __shared__ unsigned long long s_prefix;

    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = static_cast<int>(uniform(static_cast<unsigned>(tid / kWaveSize)));
    const unsigned tile = blockIdx.x;
    if (tid == 0) s_arrive = 0u;
    const size_t wave_elem0 = (static_cast<size_t>(tile) * WV + wave) * (static_cast<size_t>(kMinLoads) * kWaveSize * E);
    const size_t wave_group0 = wave_elem0 / 32;
    const unsigned tail = static_cast<unsigned>(n % 32);

    // ---- the wave's masks (lane i holds mask i) and their set bits
    unsigned own = 0, m = 0, next = 0;
    const PieceShift<W> shift(out);
    const auto mask_of = masks_within(masks, num_groups, tail);
    if constexpr (OUTPUT != Output::kShifted) {
        if (lane < kStepMasks) own = mask_of(wave_group0 + lane);
    } else {
        const ShiftedMasks<W, decltype(mask_of)> got(shift, wave_group0, lane, mask_of);
        own = got.own;
        m = got.mask;
        next = got.next;
    }
    const unsigned long long scan_word = ScanState::ask(hdr);
    lds_barrier();                                // the cleared arrival word, after the loads have been issued
    const unsigned wave_total = wave_sum_small(lane < kStepMasks ? static_cast<unsigned>(__popc(own)) : 0u);

    // ---- the workgroup's count, published by the wave that arrives last; the scan, by wave 0
    const ScanState scan(hdr, num_tiles, scan_word);
    unsigned arrived = 0;
    if (lane == 0) {
        s_wave_total[wave] = wave_total;
        arrived = arrive(&s_arrive, (1u << 24) | wave_total);
    }
    arrived = uniform(arrived);
    const bool publisher = (arrived >> 24) == WV - 1;
    if (publisher && lane == 0)
        scan.publish(tile, (arrived & 0xFFFFFFu) + wave_total);
    if (wave == 0) {
        unsigned long long ex = 0;
        if (tile != 0) {
            const CountMaskTile count_tile{masks, num_groups, tail, WV * kStepMasks};
            ex = scan_exclusive_prefix<kDecoderPause>(scan, tile, lane, count_tile);
        }
        if (lane == 0) s_prefix = ex;
    }
    lds_barrier();
    const unsigned long long exclusive = uniform(s_prefix);
    unsigned wave_offset = 0, tile_total = 0;
#pragma unroll
    for (int v = 0; v < WV; ++v) {
        const unsigned t = uniform(s_wave_total[v]);
        if (v < wave) wave_offset += t;
        tile_total += t;
    }
    if (wave == 0 && lane == 0 && scan.ends_block(tile)) scan.publish_prefix(tile, exclusive + tile_total);

    if (wave_elem0 < n) {
        if constexpr (OUTPUT != Output::kShifted)
            expand_step<W, OUTPUT == Output::kAligned>(s_stage, 16u + wave * G::kWaveStageBytes, values, values_avail, exclusive + wave_offset,
                           wave_total, own, wave_elem0, n, out, STREAM, lane);
        else
            expand_shifted<W>(s_stage, 16u + wave * G::kWaveStageBytes, values, values_avail, exclusive + wave_offset, own,
                              m, next, shift, wave_elem0, n, out, STREAM, lane);
    }

    if (tile == num_tiles - 1 && wave == 0) scan_end(scan, num_tiles, lane);
}

// And without any scan, for the smallest tensors: a workgroup counts the bits of all masks before its own
// itself, 16 bytes a thread and eight of them on their way at a time.  That is one round trip to memory where the scan takes
// three (count, wait, look), and it is work that grows with the square of the tensor.  Workgroups begin
// at different places, so that they do not all ask the same channel of the L2 at a time (a cold 4 MB
// stream 6.3 -> 5.9 us).  us, scan | here with 4 | 8 waves: fp32 0.25 MB 4.1 | 3.4 | 3.5, 1 MB 4.2 | 3.6 | 3.65, 2 MB 4.3 | 3.9 |
// 3.9, 2.5 MB 4.4 | 4.4 | 4.3, 3 MB 4.4 | 4.55 | 4.4, 4 MB 4.5 | 5.15 | 4.5 (from memory 5.1 | 5.9 | 5.4); 16-bit 0.25 MB 4.3 | 3.5 |
// 3.7, 1 MB 4.4 | 4.0 | 4.0, 1.25 MB 4.4 | 4.4 | 4.3, 2 MB 4.4 | 5.1 | 4.6, 4 MB 4.65 | 7.35 | 5.9.
template <int W, Output OUTPUT, int WV>
__global__ __launch_bounds__(WV * kWaveSize) void decompress_direct_kernel(
    const unsigned* __restrict__ masks, const unsigned char* __restrict__ values,
    unsigned long long values_avail, size_t n, unsigned char* __restrict__ out, size_t num_groups, bool stream_values) {
    static_assert(OUTPUT != Output::kShifted, "small outputs are written as they lie");
    using G = Geometry<W, kMinLoads>;
    constexpr int E = G::kElemsPerLane;
    constexpr int kStepMasks = kStageLoads * G::kGroupsPerLoad;   // masks per wave: 32 | 64
    constexpr unsigned kTogether = 8, kWorkers = WV * kWaveSize;

    __shared__ __align__(16) unsigned char s_stage[16 + WV * G::kWaveStageBytes];   // (16: see expand_piece)
    __shared__ unsigned s_before[WV], s_wave_total[WV];

    const unsigned tid = threadIdx.x;
    const int lane = static_cast<int>(tid & (kWaveSize - 1));
    const int wave = static_cast<int>(uniform(tid / kWaveSize));
    const unsigned tile = blockIdx.x;
    const size_t wave_elem0 = (static_cast<size_t>(tile) * WV + wave) * (static_cast<size_t>(kMinLoads) * kWaveSize * E);

    // ---- the masks of the workgroups before, four at a time, from some place on and around
    const unsigned before = tile * (WV * kStepMasks / 4), from = __umulhi(tile * 2654435761u, before);
    unsigned count = 0;
    for (unsigned at = tid; at < before; at += kTogether * kWorkers) {
        vec4u v[kTogether];
#pragma unroll
        for (unsigned k = 0; k < kTogether; ++k) {
            unsigned i = at + k * kWorkers;
            v[k] = vec4u{0u, 0u, 0u, 0u};
            if (i < before) {
                i += from;
                if (i >= before) i -= before;
                v[k] = *reinterpret_cast<const vec4u_at4*>(masks + 4 * i);
            }
        }
#pragma unroll
        for (unsigned k = 0; k < kTogether; ++k)
            count += static_cast<unsigned>(__popc(v[k].x) + __popc(v[k].y) + __popc(v[k].z) + __popc(v[k].w));
    }
    const auto mask_of = masks_within(masks, num_groups, static_cast<unsigned>(n % 32));
    const unsigned m = lane < kStepMasks ? mask_of(wave_elem0 / 32 + lane) : 0u;
    const unsigned counted = wave_sum_small(count), wave_total = wave_sum_small(static_cast<unsigned>(__popc(m)));
    if (lane == 0) {
        s_before[wave] = counted;
        s_wave_total[wave] = wave_total;
    }
    lds_barrier();
    unsigned first = 0;
#pragma unroll
    for (int v = 0; v < WV; ++v) {
        first += uniform(s_before[v]);
        if (v < wave) first += uniform(s_wave_total[v]);
    }
    if (wave_elem0 < n)
        expand_step<W, OUTPUT == Output::kAligned>(s_stage, 16u + wave * G::kWaveStageBytes, values, values_avail, first,
                                                   wave_total, m, wave_elem0, n, out, stream_values, lane);
}

// Decoders of the windowed stream.  No scan and no pre-pass: the offset table
// says where a window's bytes are, and a window decodes from its own bytes alone
// (section 5.2: the popcount of a mask gives the offset of the next mask).  A wave
// expands 4 KB of output (a piece, expand_piece) from bytes that are staged in LDS;
// what the kernels differ in is how the masks are found, one after the other -- the
// serial chain the paper's decoder has too:
//   windows of 1, 2 or 4 KB (window_decode_kernel): a piece is 4, 2 or 1 windows and
//     a lane walks each (8..32 masks of 32-bit elements, twice that of 16-bit ones);
//   windows of 8..64 KB (window_split_kernel): a workgroup takes a window and cuts
//     the walk into parts.
// Reads stay inside the aligned 16-byte chunks that [0, stream_bytes) touches and
// inside the staged bytes whatever the table and the masks say; what a damaged
// stream asks for beyond that decodes as zero.
constexpr int kWindowUnitBytes = 1024;  // window sizes are 1 KB << shift
constexpr unsigned kMaxWindowShift = 6; // 64 KB

template <int W>
struct WindowGeometry {
    static constexpr int kPieceGroups = kStageLoads * kWaveSize * 16 / W / 32;   // masks per 4 KB piece: 32 | 64
    static constexpr int kPieceElems = kPieceGroups * 32;
    static constexpr unsigned kGroupBytes = 4 + 32 * W;                // a group with nothing dropped
    static constexpr unsigned kPieceBytes = kPieceGroups * kGroupBytes;
    // window_decode_kernel, a wave's slice: shift < 16, then a piece, then what a walk that is past its end reads
    static constexpr unsigned kSliceBytes = (16 + kPieceBytes + kGroupBytes + 15) / 16 * 16;
};

// The mask at an LDS address that is a multiple of W (or, in a damaged stream, of
// nothing), and its popcount plus `more`.  Two halves for W = 2: an LDS access that is
// not aligned takes the lanes one after the other.
template <int W>
__device__ __forceinline__ unsigned lds_mask(const unsigned char* p) {
    if (W == 4) return *reinterpret_cast<const unsigned*>(p);
    return static_cast<unsigned>(*reinterpret_cast<const unsigned short*>(p)) |
           static_cast<unsigned>(*reinterpret_cast<const unsigned short*>(p + 2)) << 16;
}
template <int W>
__device__ __forceinline__ unsigned lds_mask_bits(const unsigned char* p, unsigned more) {
    if (W == 4) return static_cast<unsigned>(__popc(*reinterpret_cast<const unsigned*>(p))) + more;
    unsigned low = *reinterpret_cast<const unsigned short*>(p), high = *reinterpret_cast<const unsigned short*>(p + 2);
    asm("" : "+v"(low), "+v"(high));      // (or the compiler goes on in 16 bits, with masks of its own)
    return static_cast<unsigned>(__popc(low)) + (static_cast<unsigned>(__popc(high)) + more);
}

// What a mask asks for beyond the bytes that are there decodes as zero, an element
// that is only partly there included: the mask without its bits for elements that are
// not wholly before `limit` (its highest ones).  `at`: LDS offset of the group's first
// stored element.  Only damaged or cut streams enter the loop.
template <int W>
__device__ inline unsigned whole_elements(unsigned mask, unsigned at, unsigned limit) {
    const unsigned room = limit > at ? (limit - at) / W : 0u;
    while (static_cast<unsigned>(__popc(mask)) > room) mask &= ~(0x80000000u >> __clz(mask));
    return mask;
}

// A workgroup takes four pieces, a wave each.  A wave walks its own windows, a lane per
// window, but for 4 KB windows of 16-bit elements, whose one lane would keep the wave for 64
// steps: there one of the waves (not the same one in every workgroup, so that the SIMDs
// share the work) walks for all four, which saves instructions and costs two barriers (51 MB
// bf16: 16.9 us, a wave its own 18.6; but 103 MB fp32 in 4 KB windows 23.5 and 19.6, 51 MB
// bf16 in 2 KB windows 15.1 and 13.6).  The walk was bound by its instructions, and so was
// the rest: 103 MB fp32 from 4 KB windows 23.9 us before, 16-bit 22.5.
template <int W, bool ALIGNED>
__global__ __launch_bounds__(kThreads) void window_decode_kernel(
    const unsigned char* __restrict__ stream, unsigned long long stream_bytes,
    const unsigned long long* __restrict__ offsets, size_t n, size_t num_groups,
    size_t first_window, size_t num_windows, unsigned window_shift, unsigned char* __restrict__ out,
    bool interleave) {
    using G = WindowGeometry<W>;
    constexpr unsigned kSliceBytes = G::kSliceBytes;
    constexpr unsigned kMostWindows = kStageLoads;          // per piece
    static_assert(G::kPieceBytes + 15 <= kFetchSlots * kSlotBytes, "a piece fits the fetch slots");
    __shared__ __align__(16) unsigned char s_stage[16 + kWaves * kSliceBytes];      // (16: see expand_piece)
    __shared__ unsigned s_mask_at[kWaves * G::kPieceGroups];
    __shared__ __align__(8) uint2 s_window[kWaves * kMostWindows];                  // where a window begins, where the piece ends

    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = static_cast<int>(uniform(static_cast<unsigned>(tid / kWaveSize)));
    const bool together = W == 2 && window_shift == 2;
    const unsigned piece_windows = kMostWindows >> window_shift;                    // 4, 2, 1
    const unsigned window_groups = static_cast<unsigned>(G::kPieceGroups) / kMostWindows << window_shift;
    // the wave's piece: dealt out in a row or, as in the planar decoder, interleaved over the XCDs
    const size_t share = interleave ? (static_cast<size_t>(blockIdx.x / 8) * kWaves + wave) * 8 + blockIdx.x % 8
                                    : static_cast<size_t>(blockIdx.x) * kWaves + wave;
    const size_t local = share * piece_windows;             // first of the wave's windows, within the range
    const unsigned windows_here = local >= num_windows ? 0u
                                : num_windows - local < piece_windows ? static_cast<unsigned>(num_windows - local) : piece_windows;
    const size_t window0 = first_window + local;
    const auto clamped = [&](size_t k) {
        const unsigned long long o = offsets[k];
        return o > stream_bytes ? stream_bytes : o;
    };
    const unsigned slice = 16u + wave * kSliceBytes;
    unsigned limit = slice;

    // ---- the piece's bytes, clamped to what can be there, and where its windows begin: a window whose
    //      offset is off reads nothing
    if (windows_here != 0) {
        const unsigned long long lo = clamped(window0), hi = clamped(window0 + windows_here);
        const unsigned bytes = hi <= lo ? 0u : hi - lo > G::kPieceBytes ? G::kPieceBytes : static_cast<unsigned>(hi - lo);
        const unsigned char* src = stream + lo;             // wave-uniform
        const unsigned shift = static_cast<unsigned>(reinterpret_cast<uintptr_t>(src) & 15u);
        limit = slice + shift + bytes;
        wave_stage<false>(s_stage + slice, src - shift, bytes != 0 ? shift + bytes : 0u, lane);
        if (static_cast<unsigned>(lane) < piece_windows) {
            unsigned p = limit;
            if (static_cast<unsigned>(lane) < windows_here) {
                const unsigned long long o = clamped(window0 + lane);
                if (o >= lo && o - lo <= bytes) p = slice + shift + static_cast<unsigned>(o - lo);
            }
            s_window[wave * piece_windows + lane] = make_uint2(p, limit);
        }
        stage_wait();
    } else if (static_cast<unsigned>(lane) < piece_windows) {
        s_window[wave * piece_windows + lane] = make_uint2(limit, limit);
    }
    if (together) lds_barrier();
    else wave_lds_sync();

    // ---- the walks.  Every step waits for the one before: read a mask, add its popcount.  Past the
    //      staged bytes a walk reads whatever lies at their end; those masks are sorted out below.
    const unsigned walkers = together ? kWaves * piece_windows : piece_windows;
    if ((!together || static_cast<unsigned>(wave) == blockIdx.x / 8 % kWaves) && static_cast<unsigned>(lane) < walkers) {
        const unsigned k = together ? lane : wave * piece_windows + lane;
        const uint2 window = s_window[k];
        unsigned* at = s_mask_at + k * window_groups;
        unsigned p = window.x, stop = window.y;
        for (unsigned g0 = 0; g0 < window_groups; g0 += 8) {     // p, stop: less the 4 bytes of every mask since g0
#pragma unroll
            for (unsigned g = 0; g < 8; ++g) {
                at[g0 + g] = p + 4 * g;
                stop -= 4u;
                p = min(p + W * lds_mask_bits<W>(s_stage + p + 4 * g, 0u), stop);
            }
            p += 32u;
            stop += 32u;
        }
    }
    if (together) lds_barrier();
    else wave_lds_sync();
    if (windows_here == 0) return;

    // ---- the piece's masks, a lane each: none where there is no group, or not the whole mask
    const size_t group0 = window0 * window_groups;
    const size_t there = num_groups > group0 ? num_groups - group0 : 0;
    const unsigned groups_here = min(static_cast<unsigned>(min(there, static_cast<size_t>(G::kPieceGroups))),
                                     windows_here * window_groups);
    unsigned mask = 0, value_at = slice;
    if (static_cast<unsigned>(lane) < groups_here) {
        const unsigned at = s_mask_at[wave * G::kPieceGroups + lane];
        value_at = at + 4u;
        if (value_at <= limit) mask = whole_elements<W>(lds_mask<W>(s_stage + at), value_at, limit);
    }
    const unsigned left = static_cast<unsigned>(min(n - min(n, group0 * 32), static_cast<size_t>(groups_here) * 32));
    expand_piece<W, ALIGNED>(s_stage, mask, value_at, left, out + (local << window_shift) * kWindowUnitBytes, lane);
}

// Windows of 8 KB and more: a workgroup of NW = window / 4 KB waves takes one.  A walk
// cannot start in the middle of a window, but where it can come from is limited: a
// group is 1 to 33 words of 32 bits (2 to 34 of 16), so of the walks that cross a given
// byte one enters what follows at one of its first 33 (34) words.  The window's bytes
// are cut into equal parts, and
//   1. every part is walked from all those words at once, a lane each: the (part, word)
//      pairs of the window are laid over the lanes of all waves, kRows per lane (whose
//      chains overlap), so that hardly a lane is idle.  Tables say for each pair where in
//      the next part the walk comes out, where in the part's second half it came out, and
//      how many groups it had passed by then;
//   2. the tables of kPartsPerBlock parts in a row are made one, a wave for each block;
//   3. one or two waves follow the true walk through those, so that they have the first
//      word and the first group of every half of a part, and walk these again from there, a
//      lane each, noting the masks' offsets;
//   4. every wave expands its 4 KB of the window.
// Phase 1 is most of the instructions (6 per step and row) and, like 3, a chain of LDS
// reads: 74 MB bf16 from 64 KB windows of densities 0.1 to 0.9 take 23 us with no walks at
// all, phase 1 adds 5, 3 adds 5, the expansion of real masks 5: 38 us, two workgroups per CU
// (LDS).  Before, every wave walked four parts of its own from 34 of its 64 lanes and
// expanded what it found, 64 us; large numbers of windows went to a wave each, whose one
// lane walked: 822 MB fp32 from 8 KB windows 214 us, now 200; from 64 KB windows 273, now
// 232; 411 MB bf16 145 and 192, now 130 and 168; one or two windows of 64 KB, fp32 and bf16,
// 11.4 and 22.1, now 8.4 and 12.0.  Three or four rows (shorter chains, more of them) are
// slower by 3 to 5 %, walking parts whole in phase 3 by 4 to 9 %, its starts handed over by
// the lanes that walked there (two barriers more) by 6 %.
template <int W, int NW, bool ALIGNED>
__global__ __launch_bounds__(NW * kWaveSize) void window_split_kernel(
    const unsigned char* __restrict__ stream, unsigned long long stream_bytes,
    const unsigned long long* __restrict__ offsets, size_t n, size_t num_groups, size_t first_window,
    unsigned char* __restrict__ out) {
    using G = WindowGeometry<W>;
    constexpr unsigned kWindowGroups = NW * G::kPieceGroups;
    constexpr unsigned kEntries = 32 + 4 / W;               // 33 | 34
    constexpr unsigned kLost = 63;                          // as a word: no walk goes on from here
    constexpr int kRows = 2;
    constexpr unsigned kSubs = 2;                           // a part is walked again in halves
    constexpr unsigned kPairs = NW * kRows * kWaveSize;
    constexpr unsigned kParts = kPairs / kEntries;
    constexpr unsigned kBlocks = NW < 8 ? (NW + 1) / 2 : 8;
    constexpr unsigned kPartsPerBlock = (kParts + kBlocks - 1) / kBlocks;
    constexpr unsigned kMostBytes = kWindowGroups * G::kGroupBytes;
    constexpr unsigned kNoGroup = 0xFFFF;
    static_assert(kBlocks <= NW && kParts * kSubs <= NW * kWaveSize, "a wave per block, a lane per half of a part");
    static_assert(kEntries < kLost && kWindowGroups <= 1024, "a table entry is 6 bits of word, 10 of groups");
    static_assert(kMostBytes / W + 2 * kEntries < kNoGroup, "words in a window are counted in 16 bits");
    static_assert((kMostBytes / kParts + W) / 4 < 1024, "groups of a part in 10");
    // 16: see expand_piece; shift < 16; behind the window what a walk that is past its end reads: from any
    // entry a group further
    constexpr unsigned kStageBytes = (16 + 16 + kMostBytes + W * kEntries + G::kGroupBytes + 4 + 15) / 16 * 16;
    __shared__ __align__(16) unsigned char s_stage[kStageBytes];
    // of every pair, at the end of its part's halves: groups passed << 6 | word that the walk comes out at
    __shared__ unsigned short s_exit[kSubs][kParts * kEntries];
    __shared__ unsigned short s_block[kBlocks][kEntries];   // of every entry into a block of parts: the same at its end
    __shared__ unsigned short s_mask_at[kWindowGroups];     // words from the window's beginning to a group's mask

    const unsigned lane = threadIdx.x & (kWaveSize - 1);
    const unsigned wave = uniform(threadIdx.x / kWaveSize);
    const size_t window = first_window + blockIdx.x;
    const size_t window_group0 = window * kWindowGroups;
    const unsigned groups = num_groups - window_group0 < kWindowGroups ? static_cast<unsigned>(num_groups - window_group0)
                                                                       : kWindowGroups;
    const auto clamped = [&](size_t k) {
        const unsigned long long o = offsets[k];
        return o > stream_bytes ? stream_bytes : o;
    };
    const unsigned long long lo = clamped(window), hi = clamped(window + 1);
    const unsigned long long there = hi > lo ? hi - lo : 0ull;
    const unsigned bytes = there > groups * G::kGroupBytes ? groups * G::kGroupBytes : static_cast<unsigned>(there);

    // ---- the window's bytes: all waves, 1 KB at a time
    const unsigned char* src = stream + lo;
    const unsigned shift = static_cast<unsigned>(reinterpret_cast<uintptr_t>(src) & 15u);
    const unsigned begin = 16u + shift;                     // in s_stage
    const unsigned end = bytes != 0 ? shift + bytes : 0u;
#pragma unroll
    for (unsigned at = 0; at < kMostBytes + 15; at += NW * kSlotBytes) {
        const unsigned slot = at + wave * kSlotBytes;
        if (slot >= end) break;                             // uniform
        stage_slot<false, 0>(s_stage + 16 + slot, src - shift + slot, end - slot, static_cast<int>(lane));
    }
    if (lane < static_cast<unsigned>(G::kPieceGroups)) s_mask_at[wave * G::kPieceGroups + lane] = kNoGroup;
    stage_wait();
    lds_barrier();

    // ---- 1. all walks that can enter a part.  Words are counted from the window's beginning; a walk's state
    //         is its word and, in the upper half, the groups it has passed.  (A finished walk goes on reading
    //         where it stands.)
    const unsigned words = (bytes + W - 1) / W, part = (words + kParts - 1) / kParts, sub = (part + kSubs - 1) / kSubs;
    const unsigned mask_words = bytes >= 4u ? (bytes - 4u) / W + 1u : 0u;   // a mask that begins before this is wholly there
    const auto sub_end = [&](unsigned q, unsigned c) { return min(q * part + min((c + 1) * sub, part), words); };
    const auto step = [&](unsigned state) __attribute__((always_inline)) {
        unsigned at;                                        // begin + W * (the lower half of state)
        asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(at) : "v"(state), "n"(W), "s"(begin));
        return state + lds_mask_bits<W>(s_stage + at, (1u << 16) + 4u / W);
    };
    unsigned state[kRows], q[kRows], entry[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const unsigned i = (wave * kRows + r) * kWaveSize + lane;
        q[r] = i / kEntries;
        entry[r] = i - q[r] * kEntries;
        state[r] = min(q[r] * part, words) + entry[r];
    }
#pragma unroll
    for (unsigned c = 0; c < kSubs; ++c) {
        unsigned stop[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) stop[r] = q[r] < kParts ? min(sub_end(q[r], c), mask_words) : 0u;
        bool going = true;
        while (going) {
            going = false;
#pragma unroll
            for (int twice = 0; twice < 2; ++twice) {
                unsigned next[kRows];
#pragma unroll
                for (int r = 0; r < kRows; ++r) next[r] = step(state[r]);
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    const bool on = static_cast<unsigned short>(state[r]) < static_cast<unsigned short>(stop[r]);
                    state[r] = on ? next[r] : state[r];
                    if (twice == 1) going |= on;
                }
            }
            going = __any(going);
        }
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const unsigned word = state[r] & 0xFFFFu, from = sub_end(q[r], c);
            if (q[r] < kParts)
                s_exit[c][q[r] * kEntries + entry[r]] =
                    static_cast<unsigned short>(state[r] >> 16 << 6 | (word < from ? kLost : word - from));
        }
    }
    lds_barrier();

    // ---- 2. the tables of a block of parts made one; a part's own table then says how a walk gets from the
    //         block's beginning to the part.  (A walk that has passed 1024 groups has passed all there can be.)
    if (wave < kBlocks) {
        unsigned word = lane < kEntries ? lane : kLost, before = 0;
#pragma unroll
        for (unsigned j = 0; j < kPartsPerBlock; ++j) {
            const unsigned part_entry = (wave * kPartsPerBlock + j) * kEntries;
            if (part_entry >= kParts * kEntries) break;     // uniform
            const unsigned v = word != kLost ? s_exit[kSubs - 1][part_entry + word] : kLost;
            if (lane < kEntries)
                s_exit[kSubs - 1][part_entry + lane] = static_cast<unsigned short>(before < kWindowGroups ? before << 6 | word : kLost);
            before += v >> 6;
            word = v & 63u;
        }
        if (lane < kEntries) s_block[wave][lane] = static_cast<unsigned short>(before < kWindowGroups ? before << 6 | word : kLost);
    }
    lds_barrier();

    // ---- 3. the true walk
    const unsigned k = wave * kWaveSize + lane;
    if (k < kParts * kSubs) {
        const unsigned mine = k / kSubs, c = k - mine * kSubs;
        unsigned word = 0, first = 0;
        for (unsigned b = 0; b < mine / kPartsPerBlock && word != kLost; ++b) {
            const unsigned v = s_block[b][word];
            first += v >> 6;
            word = v & 63u;
        }
        if (word != kLost) {
            const unsigned v = s_exit[kSubs - 1][mine * kEntries + word];
            first += v >> 6;
            word = v & 63u;
        }
        if (word != kLost && c != 0) {
            const unsigned v = s_exit[c - 1][mine * kEntries + word];
            first += v >> 6;
            word = v & 63u;
        }
        if (word != kLost && first < groups) {
            unsigned at = (c == 0 ? min(mine * part, words) : sub_end(mine, c - 1)) + word;
            const unsigned last = min(sub_end(mine, c), mask_words);
            while (at < last && first < groups) {
                s_mask_at[first++] = static_cast<unsigned short>(at);
                at += lds_mask_bits<W>(s_stage + begin + W * at, 4u / W);
            }
        }
    }
    lds_barrier();

    // ---- 4. the wave's masks, a lane each (none for groups that a damaged stream has no mask for)
    const size_t elem0 = (window_group0 + wave * G::kPieceGroups) * 32;
    if (elem0 >= n) return;
    unsigned mask = 0, value_at = begin;
    if (lane < static_cast<unsigned>(G::kPieceGroups)) {
        const unsigned at = s_mask_at[wave * G::kPieceGroups + lane];
        if (at != kNoGroup) {
            value_at = begin + W * at + 4u;
            mask = whole_elements<W>(lds_mask<W>(s_stage + value_at - 4), value_at, begin + bytes);
        }
    }
    const unsigned left = static_cast<unsigned>(min(n - elem0, static_cast<size_t>(G::kPieceElems)));
    expand_piece<W, ALIGNED>(s_stage, mask, value_at, left,
                             out + (static_cast<size_t>(blockIdx.x) * NW + wave) * (G::kPieceElems * W), static_cast<int>(lane));
}

// Count-only pass (section 5.4's size, without producing the stream).  One
// workgroup per 32 KB of input, all of a thread's loads in flight together.
// A workgroup adds (1 << 40) + its count to one of 64 accumulators with a single
// atomic: the low 40 bits collect kept elements, the high bits count arrivals.
// The workgroup that completes an accumulator bumps finish_top; the one that
// completes finish_top adds the 64 sums up, reports, and leaves the accumulators
// at zero for the next call.
constexpr int kCountLoads = 8;
constexpr int kCountShift = 40;

// `in` is the 16-byte boundary at or before the tensor, which is elements
// skip .. n - 1 from there (ALIGNED: skip is 0).  Where a load begins makes no
// difference to a count, so every load is a whole aligned one and the elements
// before the tensor are masked out.  (The memory unit splits 16 bytes from an
// odd 16-bit element on: 26 MB took 9.2 us and 300 MB 64.8, now 6.9 and 51.1 as
// from a boundary; from a whole dword both ways are within 3 %.)
template <int W, bool ALIGNED>
__global__ __launch_bounds__(kThreads) void count_kernel(const unsigned char* __restrict__ in,
                                                         unsigned skip, size_t n, WsHeader* hdr,
                                                         unsigned long long* d_bytes,
                                                         size_t num_groups, unsigned num_tiles) {
    constexpr int E = 16 / W;
    __shared__ unsigned long long s_wave[kWaves];
    __shared__ unsigned s_last;
    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = tid / kWaveSize;
    const unsigned tile = blockIdx.x;
    const size_t q0 = static_cast<size_t>(tile) * (kThreads * kCountLoads) + tid;
    uint4 v[kCountLoads];
    if ((q0 - tid + kThreads * kCountLoads) * E <= n) {
#pragma unroll
        for (int j = 0; j < kCountLoads; ++j)
            v[j] = load16_stream(in + (q0 + static_cast<size_t>(j) * kThreads) * 16);
    } else {
#pragma unroll
        for (int j = 0; j < kCountLoads; ++j)
            v[j] = load_chunk<W>(in, (q0 + static_cast<size_t>(j) * kThreads) * E, n);
    }
    unsigned long long count = 0;
#pragma unroll
    for (int j = 0; j < kCountLoads; ++j) {
        unsigned bits = presence_bits<W, false>(v[j]);
        if (!ALIGNED && j == 0 && q0 == 0) bits &= ~0u << skip;
        count += __popc(bits);
    }
    count = wave_sum(count);
    if (lane == 0) s_wave[wave] = count;
    __syncthreads();
    if (tid == 0) {
        unsigned long long block_total = 0;
        for (int k = 0; k < kWaves; ++k) block_total += s_wave[k];
        const unsigned slot = tile % kFinishLanes;
        const unsigned quota = num_tiles / kFinishLanes + (slot < num_tiles % kFinishLanes ? 1u : 0u);
        const unsigned long long old =
            atomicAdd(&hdr->finish[slot].sum, (1ull << kCountShift) + block_total);
        unsigned last = 0;
        if ((old >> kCountShift) == quota - 1) {
            const unsigned slots_used = num_tiles < kFinishLanes ? num_tiles : kFinishLanes;
            last = atomicAdd(&hdr->finish_top.value, 1u) == slots_used - 1 ? 1u : 0u;
        }
        s_last = last;
    }
    __syncthreads();
    if (s_last == 0u || wave != 0) return;
    const unsigned long long part =
        __hip_atomic_load(&hdr->finish[lane].sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
        ((1ull << kCountShift) - 1);
    const unsigned long long total = wave_sum(part);
    hdr->finish[lane].sum = 0ull;
    if (lane == 0) {
        *d_bytes = 4ull * num_groups + static_cast<unsigned long long>(W) * total;
        hdr->finish_top.value = 0u;
    }
}

// Measurement aid, not part of the method: a plain streaming kernel that reads
// read_chunks 16-byte chunks and writes write_chunks of them, split evenly over
// the workgroups (up to 64 KB each way per workgroup, non-temporal accesses, all
// of a thread's loads in flight together, stores that depend on the loads).  It
// shows what this memory system does with the traffic of a codec call when
// nothing else is asked of the kernel.  LOADS 16-byte loads per thread: 64 KB
// per workgroup, or 16 KB for small transfers (more workgroups than CUs).
template <int LOADS>
__global__ __launch_bounds__(kThreads) void reference_stream_kernel(const uint4* __restrict__ in,
                                                                    size_t read_chunks, uint4* __restrict__ out,
                                                                    size_t write_chunks, unsigned read_per_group,
                                                                    unsigned write_per_group) {
    const size_t r0 = static_cast<size_t>(blockIdx.x) * read_per_group;
    const size_t w0 = static_cast<size_t>(blockIdx.x) * write_per_group;
    uint4 v[LOADS];
    unsigned mix = blockIdx.x;
#pragma unroll
    for (int k = 0; k < LOADS; ++k) {
        const unsigned i = threadIdx.x + k * kThreads;
        v[k] = make_uint4(0u, 0u, 0u, 0u);
        if (i < read_per_group && r0 + i < read_chunks) v[k] = load16_stream(in + r0 + i);
    }
#pragma unroll
    for (int k = 0; k < LOADS; ++k) mix ^= v[k].x ^ v[k].y ^ v[k].z ^ v[k].w;
#pragma unroll
    for (int k = 0; k < LOADS; ++k) {
        const unsigned i = threadIdx.x + k * kThreads;
        if (i < write_per_group && w0 + i < write_chunks) {
            uint4 d = v[k];
            d.x ^= mix;
            store16_stream(out + w0 + i, d);
        }
    }
}

// -------------------------------------------------------------- host helpers
// log2(window_bytes / 1 KB) for the window sizes of the windowed stream (a power of
// two from 1 KB to 64 KB), else -1.
inline int window_shift_of(size_t window_bytes) {
    for (unsigned k = 0; k <= kMaxWindowShift; ++k)
        if (window_bytes == static_cast<size_t>(kWindowUnitBytes) << k) return static_cast<int>(k);
    return -1;
}

inline bool aligned_to(const void* p, size_t a) {
    return reinterpret_cast<uintptr_t>(p) % a == 0;
}

inline bool ranges_overlap(const void* a, size_t an, const void* b, size_t bn) {
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return an != 0 && bn != 0 && a0 < b0 + bn && b0 < a0 + an;
}

inline zvc_status hip_ok(hipError_t e) { return e == hipSuccess ? ZVC_OK : ZVC_E_HIP; }

// Kernel launch that reports its own status (hipGetLastError after a <<<>>> launch
// would also report, and clear, an earlier error of the calling thread).
template <typename... Params, size_t... I>
hipError_t launch_impl(void (*kernel)(Params...), dim3 grid, dim3 block, hipStream_t stream,
                       std::tuple<Params...>& values, std::index_sequence<I...>, unsigned lds_bytes) {
    void* pointers[] = {static_cast<void*>(&std::get<I>(values))...};
    return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, pointers, lds_bytes, stream);
}
// lds_bytes: more LDS per workgroup than the kernel declares, for fewer workgroups per CU.
template <typename... Params, typename... Args>
hipError_t launch_padded(void (*kernel)(Params...), unsigned lds_bytes, dim3 grid, dim3 block,
                         hipStream_t stream, Args... args) {
    static_assert(sizeof...(Params) == sizeof...(Args), "one argument per kernel parameter");
    std::tuple<Params...> values{static_cast<Params>(args)...};
    return launch_impl(kernel, grid, block, stream, values, std::index_sequence_for<Params...>{}, lds_bytes);
}
template <typename... Params, typename... Args>
hipError_t launch(void (*kernel)(Params...), dim3 grid, dim3 block, hipStream_t stream, Args... args) {
    return launch_padded(kernel, 0, grid, block, stream, args...);
}

// LDS to add for a workgroup of four waves that declares `declared` bytes, so that seven share a
// CU's 160 KB.  Without it eight do, as many as a CU has wave slots for.
constexpr unsigned kCuLdsBytes = 160u << 10, kSevenLdsBytes = kCuLdsBytes / 8 + 1024;
static_assert(kWaves == 4 && kCuLdsBytes / kSevenLdsBytes == 7, "32 waves and 160 KB per CU");
constexpr unsigned seven_per_cu(unsigned declared) { return kSevenLdsBytes - declared; }

// Zeroes the header and the first state_bytes bytes of scan state.
zvc_status launch_reset(void* d_ws, size_t state_bytes, hipStream_t stream) {
    const size_t words = (kHeaderBytes + state_bytes) / 8;
    const unsigned blocks = static_cast<unsigned>(div_up(words, 256) < 1024 ? div_up(words, 256) : 1024);
    return hip_ok(launch(reset_kernel, dim3(blocks), dim3(256), stream,
                         static_cast<unsigned long long*>(d_ws), words));
}

zvc_status check_workspace(const void* d_ws, size_t ws, size_t n, int w) {
    if (d_ws == nullptr) return ZVC_E_ARG;
    if (!aligned_to(d_ws, 256)) return ZVC_E_ALIGN;
    if (ws < zvc_workspace_bytes(n, w)) return ZVC_E_WORKSPACE;
    return ZVC_OK;
}


// Shape of the encoder's tile: chunks per wave x waves per workgroup.  Each tile
// costs a fixed few nanoseconds of chip-wide time (workgroup launch plus the
// scan's state traffic), so large tensors use larger tiles.  A small tile is
// through its chain of load, test, publish, store sooner, and its straight-line
// code is shorter (a call's first wave on a CU fetches it from memory: one tile
// alone takes 3.7 us with 16 KB, 4.8 with 32 KB, 6.9 with 64 KB).  Measured us with
// 16 | 32 KB tiles, density 0.5 (windowed: 0.1 to 0.9, 12 and 14 MB: 0.1 to 0.7), sizes a few elements
// above a whole number of tiles, three buffers in turn, on both sides of every limit below:
//   fp32      12 MB 7.3 | 8.2   14.1 MB 8.4 | 7.9, density 0.2 8.3 | 7.7, dense 8.7 | 11.2   15.5 MB 8.7 | 8.0, 0.2 8.5 | 7.8,
//             dense 8.8 | 10.2   20 MB 9.6 | 9.4, dense 10.2 | 11.0   32 MB 12.4 | 10.9, dense 13.4 | 13.1   56 MB 20.9 | 17.1
//             (a dense tensor pays for the lower limit: half of its 32 KB tile waits for the scan)
//            103 MB 32.1 | 32.0   150 MB 45.1 | 44.6   170 MB 51.1 | 49.8   300 MB 87.0 | 82.1   (32 | 64 KB)
//   windowed  32 MB 14.1 | 14.3   36 MB 15.4 | 15.6   40 MB 16.6 | 16.4   48 MB 19.4 | 18.2   100 MB 36.5 | 34.1
//             (822 MB: nothing gained from 64 KB)
//   16-bit    32 MB 13.8 | 15.7   44 MB 17.2 | 17.0   47.5 MB 18.0 | 17.6, density 0.5 19.8 | 19.9   49 MB 18.6 | 18.2,
//             0.5 20.4 | 21.0   54 MB 20.0 | 19.0, 0.5 22.1 | 21.9   60 MB 21.9 | 20.8, 0.5 24.3 | 24.4   (0.1 to 0.5;
//             700 MB of buffers in turn 49 MB 19.2 | 18.6; fused ReLU 47.5 MB 18.2 | 17.8, 49 MB 18.6 | 18.3, 54 MB 20.3 | 19.2)
//   windowed  90 MB 38.4 | 39.7  110 MB 45.3 | 45.8  120 MB 49.0 | 48.9  150 MB 59.1 | 57.7  200 MB 77.8 | 73.0
// 16-bit elements are twice the vector work per byte, and the 32 KB tile's eight
// waves per SIMD (against four) hide it better: 64 KB tiles lose up to 9 % there.
// (8 KB tiles, and 8 or 16 waves per tile, were no faster at any size.)
struct TileShape {
    int chunks;   // per wave: 16, 32 or 64
    int waves;    // per workgroup
};
constexpr size_t kLargeTensorBytes = size_t{160} << 20;

constexpr TileShape kMinShape{16, 4};             // 16 KB, the smallest tile (sizes the workspace)
static_assert(kMinShape.chunks * kMinShape.waves * kChunkBytes == kMinLoads * 16 * kThreads, "smallest tile");

// From where on the tile is 32 KB.
constexpr size_t medium_bytes(int w, bool windowed) {
    return w == 4 ? size_t{windowed ? 38u : 14u} << 20 : size_t{windowed ? 120u : 48u} << 20;
}

inline TileShape choose_shape(size_t n, int w, bool windowed) {
    const size_t bytes = n * static_cast<size_t>(w);
    return bytes >= kLargeTensorBytes && w == 4 && !windowed ? TileShape{64, 4}
         : bytes >= medium_bytes(w, windowed) ? TileShape{32, 4} : kMinShape;
}

// The input is read with the streaming hint at every size.  A tensor that is read once, just written or
// from memory, loses without it: its lines push others out of the caches, and where it lies in the caches it is
// served from there with the hint as well.  us with the hint | without, density 0.4; 3 and 12 buffers in turn, each
// just written by a copy; 700 MB of buffers, each just written; 700 MB from memory:
//   fp32   4 MB 6.9 | 6.8  6.0 | 5.8  6.0 | 6.5  6.4 | 7.0   6.4 MB 8.3 | 8.4  6.2 | 6.3  6.3 | 6.9  7.5 | 7.3
//          10 MB 7.7 | 7.7  7.2 | 7.3  7.4 | 8.8  7.7 | 8.3   1 MB 5.0 | 5.1  5.2 | 5.2  5.2 | 5.1  5.3 | 5.0
//   16-bit 6.4 MB 8.8 | 8.8  7.1 | 7.1  7.1 | 7.8  7.2 | 8.0   size pass of 10 MB 5.7 | 5.8  5.2 | 5.3  5.3 | 6.2  5.6 | 6.1
// What gains without it is a tensor that nobody writes and that is compressed again and again: the first call leaves it in the
// caches.  Three such buffers in turn, 1 | 4 | 6.4 | 10 MB fp32: 5.4 | 6.2 | 7.0 | 7.8 with the hint, 4.8 | 5.1 | 5.6 | 6.7 without.

// Which tensors' tiles stage half of their steps before their count is published and half after
// (EARLY; the windowed stream has its own rule).  That pays while the call is a short chain of tiles that
// wait for counts; a large 16-bit tensor's vector units are busy, and the second half's staging is then in the way.
//   fp32, us all | half: 256 KB 4.91 | 4.86, dense 5.66 | 4.86   4 MB dense 5.94 | 5.38   18 MB fused ReLU 9.4 |
//   9.0   32 MB 11.1 | 10.9   49 MB 16.3 | 16.4   56 MB 17.1 | 17.6   64 MB 19.4 | 21.3, dense 24.5 | 27.8   80 MB
//   25.6 | 25.8   (none: 256 KB 5.08; 822 MB, 64 KB tiles, 205.5, all 202.8)
//   16-bit, all | half: 8 MB dense 8.1 | 7.2   12 MB 9.3 | 8.7   15 MB 10.2 | 9.6, dense 9.8 | 9.5   17 MB
//   10.4 | 10.1   20 MB 10.7 | 10.9, dense 10.9 | 10.8   30 MB 13.9 | 14.2, dense 13.2 | 15.5
inline bool choose_early(size_t n, int w) {
    return n * static_cast<size_t>(w) < (size_t{w == 4 ? 48u : 20u} << 20);
}

enum class Encoder { kPlain, kRelu, kWindowed };

template <int W, int CH, bool SPLIT, bool EARLY, bool WINDOWED_TOO = true>
hipError_t launch_compress_as(Encoder mode, hipStream_t stream, const unsigned char* in, size_t n,
                        unsigned* masks, unsigned char* values, WsHeader* hdr,
                        unsigned long long* d_bytes, unsigned long long* h_bytes, unsigned tiles, size_t groups,
                        unsigned long long cap_values, unsigned long long* offsets, unsigned window_shift) {
    const EncoderArgs args{in, n, masks, values, hdr, d_bytes, h_bytes, tiles, groups, cap_values, offsets,
                           window_shift};
    constexpr int WV = 4;
    const dim3 grid(tiles), block(WV * kWaveSize);
    switch (mode) {
        case Encoder::kPlain:
            return launch(compress_kernel<W, CH, WV, false, false, SPLIT, EARLY>, grid, block, stream, args);
        case Encoder::kRelu:
            return launch(compress_kernel<W, CH, WV, true, false, SPLIT, EARLY>, grid, block, stream, args);
        case Encoder::kWindowed:
            if constexpr (WINDOWED_TOO)
                return launch(compress_kernel<W, CH, WV, false, true, SPLIT, false>, grid, block, stream, args);
            else
                return hipErrorInvalidValue;   // choose_shape() gives the windowed stream no such tile
    }
    return hipErrorInvalidValue;
}

// How a tensor is decoded: every workgroup counts the masks before its own (kDirect); one launch with the
// device-wide scan, in workgroups of 4 or 8 waves (kScan4, kScan8); two launches.  kDirect up to 80 KB of masks, with 4 waves
// up to 48 KB: see decompress_direct_kernel.  Beyond, us with kScan4 | kScan8 | two launches.  Up to 32 MB the chip holds all
// waves at once, and fewer workgroups look for fewer counts; above, the larger workgroups' second turn is the longer one.  Then the
// pre-pass is as fast or wins: its expand kernel touches no shared state, and may write in any order.  From 44 MB up on streams from
// memory (dense ones: one launch is ahead up to 60 MB, and in the caches at 0.6 as well), from 56 MB at an odd element, where a
// piece has more to do between its masks and its stores (and from 76 MB with three quarters of the elements stored: there two
// launches were slower, on streams in the caches, than stores that follow the output's alignment, and one is not).
//   density 0.3, fp32    3 MB 4.4 | 4.5 | 6.5   4 MB 4.5 | 4.6 | 6.5   5 MB 5.1 | 4.7 | 6.5   6.1 MB 5.1 | 4.7 | 7.0   8.5 MB 5.8 | 5.6 |
//                        6.8   16 MB 6.8 | 6.2 | 7.9   24 MB 8.3 | 7.8 | 9.4   32 MB 10.0 | 9.9 | 11.3   40 MB 12.2 | 13.5 | 12.9
//                        50 MB 14.6 | 15.8 | 14.6   64 MB 17.4 | 18.7 | 17.5   100 MB 25.1 | 26.8 | 24.7
//                16-bit  4 MB 4.7 | 4.9 | 6.55   6 MB 5.4 | 5.0 | 6.7   12 MB 6.3 | 6.0 | 7.35   19 MB 7.7 | 7.5 | 8.6   30 MB 10.0 | 9.8 |
//                        11.0   40 MB 12.6 | 14.2 | 13.4   51 MB 15.2 | 16.9 | 15.0   64 MB 17.9 | 19.4 | 18.05   100 MB 26.1 | 28.0 | 25.2
//   density 0.9, fp32    24 MB 11.8 | 11.5 | 12.9   50 MB 21.2 | 22.7 | 22.6; 16-bit 64 MB 26.3 | 28.75 | 27.1
//   at an odd element, 0.3: fp32 32 MB 10.7 | 10.8 | 11.9; 16-bit 52 MB 16.5 | 17.75 | 16.2
//   at an odd element, one launch (kScan4) | two: fp32 of 0.1 | 0.3 | 0.6 | 0.9, 36 MB 10.5 | 12.5  12.1 | 13.5  13.7 | 14.9  16.3 | 17.6
//                        46 MB 13.4 | 13.4  14.6 | 14.6  16.0 | 16.7  20.2 | 21.3   55 MB 15.4 | 15.2  16.7 | 16.6  18.6 | 19.1  23.1 | 24.6
//                        (from memory 15.7 | 15.3  16.6 | 16.6  22.4 | 22.3  23.4 | 24.8)   75 MB 19.2 | 18.6  21.3 | 20.5  23.4 | 24.3  30.1 |
//                        31.4 (from memory 19.6 | 18.7  21.2 | 20.5  29.2 | 27.3  31.1 | 31.7); 16-bit 55 MB 16.2 | 16.2  17.2 | 17.2  18.9 |
//                        19.4  23.9 | 25.5   75 MB 20.3 | 20.6  21.8 | 21.8  24.0 | 25.0  31.6 | 32.3 (from memory 20.4 | 20.7  21.8 |
//                        21.8  30.0 | 28.4  31.8 | 32.3)
//   from memory, one launch | two: fp32 of 0.1 | 0.3 | 0.6, 40 MB 11.7 | 12.2  12.4 | 12.9  17.2 | 17.6   46 MB 13.1 | 12.8  13.9 | 13.8
//                        19.2 | 19.7   51 MB 13.9 | 13.7  14.8 | 14.8  20.0 | 20.3; 16-bit 40 MB 12.0 | 12.7  12.6 | 13.5  17.5 | 18.3   46 MB
//                        13.4 | 13.4  14.1 | 14.2  19.4 | 20.2; with zeros in clusters 51 MB of 0.3 16.7 | 16.2; fp32 of 0.9, 46 MB
//                        20.3 | 21.6   60 MB 24.8 | 26.0; in the caches of 0.6 | 0.9, 46 MB 15.5 | 16.5  20.0 | 20.9   60 MB 18.9 | 20.3
//                        24.7 | 25.7 (from memory of 0.6 23.3 | 22.7)
// (Two waves: 4 MB 5.2 for 5.4 with a shorter pause, but they need twice the scan state.)
enum class Decoder { kDirect4, kDirect8, kScan4, kScan8, kTwoLaunches };
inline Decoder choose_decoder(size_t n, int w, const void* out, unsigned long long stored) {
    const size_t bytes = n * static_cast<size_t>(w), masks = 4 * div_up(n, 32);
    if (masks <= (size_t{80} << 10)) return masks <= (size_t{48} << 10) ? Decoder::kDirect4 : Decoder::kDirect8;
    const unsigned one_launch_mb = aligned_to(out, 16) ? 44u : stored >= n / 4 * 3 ? 76u : 56u;
    if (bytes >= (size_t{one_launch_mb} << 20)) return Decoder::kTwoLaunches;
    return bytes >= (size_t{9} << 19) && bytes <= (size_t{32} << 20) ? Decoder::kScan8 : Decoder::kScan4;
}

// Tensors below this size never decode in the interleaved order (no gain there).
inline bool interleaves(size_t n, int w) { return n * static_cast<size_t>(w) >= (size_t{64} << 20); }

template <int W, int LOADS, Output OUTPUT>
hipError_t launch_decompress_as(dim3 grid, hipStream_t stream, const unsigned* masks,
                          const unsigned char* values, unsigned long long avail, size_t n,
                          unsigned char* out, const unsigned* unit_end,
                          const unsigned long long* chunk_prefix, const unsigned* chunk_total,
                          size_t groups) {
    // Dense streams (3/4 of the elements stored, or more) are read with the streaming
    // hint: little of a cache line is then shared between waves, and the hint is worth
    // 5 % there; sparser streams are read through the caches (see load16_stream).
    const bool stream_values = avail >= n / 4 * 3;
    // Order in which the parts of the tensor are dealt out to the workgroups (see the
    // kernel): interleaved where it measures faster, 2-15 % below a twelfth and 2-5 %
    // above a third of the elements stored; in between the plain order is 1 % ahead, but not
    // for the largest tensors (us, plain | interleaved, fp32: 250 MB at density 0.2 50.8 | 51.2, 500 MB
    // 107.1 | 106.2, at 0.1 89.7 | 86.7, at 0.3 116.5 | 113.8; 822 MB at 0.2 168.2 | 163.7, its first pass
    // over new buffers 246 | 220).
    const bool interleave = ((avail < n / 12 || avail > n / 3) && interleaves(n, W)) || n * W >= (size_t{400} << 20);
    // From 64 MB and a quarter of the elements stored up (from 600 MB a sixth), 7 workgroups share a CU instead
    // of the 8 that it has wave slots for: fewer waves write at once and memory takes the writes up to 2 % faster.
    // us, 8 | 7 per CU, 12 streams in turn, fp32 and bf16:
    //   784 MB  0.02 138.4 | 143.8  152.7 | 159.6   0.05 150.2 | 156.8  165.4 | 170.8   0.1 155.9 | 159.2  171.7 | 174.7
    //           0.15 156.5 | 158.6  170.0 | 172.8   0.2  161.4 | 160.6  173.1 | 173.4   0.3 175.1 | 174.3  183.2 | 183.8
    //           0.5  205.9 | 205.2  214.6 | 212.7   1    263.8 | 262.0  269.9 | 268.9
    //   400 MB  0.2  85.3 | 86.4  92.0 | 92.2   0.5 105.8 | 105.4  111.6 | 110.8   80 MB  0.1 18.6 | 19.0  19.8 | 20.4   0.5 27.5 | 27.3
    //           28.5 | 27.8
    // (Sparse streams that stay in the caches, three in turn, gain 1 % with 7: 784 MB fp32 at 0.05 129.8 | 128.5.)  Fewer
    // yet lose where the vector units bind (fp32 at 0.2, 7 | 6 | 5: 163.5 | 166.1 | 177.4), and a tensor of 51 MB, where
    // there are few waves, loses with any (14.9 | 15.0 | 15.9 | 15.5).
    const bool seven = interleaves(n, W) && avail > n / (n * W >= (size_t{600} << 20) ? 6 : 4);
    const unsigned lds_pad = seven ? seven_per_cu(Geometry<W, LOADS>::kDecodeLdsBytes) : 0;
    return launch_padded(decompress_kernel<W, LOADS, OUTPUT>, lds_pad, grid, dim3(kThreads), stream,
                         masks, values, avail, n, out, unit_end, chunk_prefix, chunk_total, groups, stream_values,
                         interleave);
}

// Windows that a workgroup each decodes (window_split_kernel) instead of a lane each: from
// 8 KB on, at every number of windows (in us, lane | workgroup each, densities 0.1 to 0.9:
// 8 KB, 103 MB fp32 30.3 | 27.5, 51 MB bf16 28.1 | 24.0; the lane's chain is a quarter of
// that at 2 KB and the workgroup's three barriers stay).
constexpr int kSplitShift = 3;

// Whether window_decode_kernel deals its windows out in the interleaved order: from the size
// of a range on at which that order is the faster one for a stream of this density.  us,
// plain | interleaved, windows of 1, 2 and 4 KB:
//   fp32  0.02, 130 MB 25.6 | 25.3  25.4 | 24.8  23.2 | 23.4   250 MB 46.5 | 41.8  45.6 | 41.8  39.4 | 39.0
//         0.05, 784 MB 145 | 122  142 | 122  123 | 113   (the plain order writes 16 KB per XCD, and with
//         little to read and to expand the XCDs' writes then hold each other up)
//         0.12, 400 MB 68.6 | 71.0  68.9 | 70.8  71.2 | 74.0   650 MB 125 | 122  126 | 124  133 | 128
//         0.25, 300 MB 65.9 | 66.8  66.0 | 66.5  65.1 | 64.8   400 MB 90.3 | 89.3  89.6 | 89.2  88.7 | 87.0
//         0.4,  175 MB 42.6 | 43.7  42.7 | 43.6  43.4 | 43.6   250 MB 63.7 | 62.3  61.7 | 61.3  62.3 | 60.7
//         0.6,  110 MB 31.0 | 31.9  31.3 | 32.1  32.4 | 32.7   150 MB 44.2 | 42.9  42.4 | 42.2  43.4 | 42.9
//   16-bit  0.04, 400 MB 59.6 | 61.3  72.9 | 73.6  81.5 | 81.2   0.25, 400 MB 96.9 | 91.0  90.4 | 91.0  102 | 102
//         0.4,  250 MB 66.5 | 65.2  62.9 | 62.9  69.7 | 68.2   0.6, 150 MB 43.5 | 43.0  43.7 | 42.9  45.9 | 45.3
// (Three streams in turn, which for sparse tensors stay in the caches.  From memory, 12 in turn, the interleaved order is
// ahead by 0 to 4 % at these sizes, 16-bit 1 KB windows of density 0.2 to 0.4 by 3 to 8 %.  Seven workgroups per CU instead
// of eight: 1 and 2 KB windows of 784 MB fp32 at 0.05 118.8 and 120.1 from the caches, but 4.8 and 1.7 % slower from memory.)
inline bool interleaves_windows(size_t n, int w, int shift, size_t stream_bytes, size_t out_bytes) {
    const size_t tensor = n * static_cast<size_t>(w), masks = 4 * div_up(n, 32);
    const size_t stored = stream_bytes > masks ? stream_bytes - masks : 0;
    const size_t from = stream_bytes / 3 > tensor / 4 ? 64 : stored > tensor / 2 ? 150 : stored > tensor / 3 ? 250
                      : stored > tensor / 5 ? 400 : stored > tensor / (shift == 2 ? 16 : 12) ? 600 : w == 4 ? 150 : 0;
    return from != 0 && out_bytes >= from << 20;
}

template <int W, int NW>
hipError_t launch_window_split_as(bool aligned, hipStream_t stream, const unsigned char* in,
                                  unsigned long long stream_bytes, const unsigned long long* offsets, size_t n,
                                  size_t groups, size_t first_window, size_t num_windows, unsigned char* out) {
    constexpr size_t kWindowBytes = size_t{4096} * NW, kMostWindows = (size_t{1} << 31) / (NW * kWaveSize);
    hipError_t e = hipSuccess;
    for (size_t k = 0; k < num_windows && e == hipSuccess; k += kMostWindows)     // (a launch takes fewer than 2^32 threads)
        e = launch(aligned ? window_split_kernel<W, NW, true> : window_split_kernel<W, NW, false>,
                   dim3(static_cast<unsigned>(num_windows - k < kMostWindows ? num_windows - k : kMostWindows)),
                   dim3(NW * kWaveSize), stream, in, stream_bytes, offsets, n, groups, first_window + k,
                   out + k * kWindowBytes);
    return e;
}
template <int W, typename... Args>
hipError_t launch_window_split(int waves, Args... args) {
    switch (waves) {
        case 2: return launch_window_split_as<W, 2>(args...);
        case 4: return launch_window_split_as<W, 4>(args...);
        case 8: return launch_window_split_as<W, 8>(args...);
        case 16: return launch_window_split_as<W, 16>(args...);
    }
    return hipErrorInvalidValue;   // there is no other window size from kSplitShift on
}

// Picks the instantiation for (w, tile shape, 16-bit elements at an odd half dword, early).  Left
// out are those that choose_shape() and choose_early() never give.
template <int CH, bool EARLY, typename... Args>
hipError_t launch_compress_16bit(bool split, Args... args) {
    return split ? launch_compress_as<2, CH, true, EARLY>(args...) : launch_compress_as<2, CH, false, EARLY>(args...);
}
template <typename... Args>
hipError_t launch_compress(int w, TileShape shape, bool split, bool early, Args... args) {
    switch (shape.waves == 4 ? shape.chunks : 0) {
        case 16:
            return w == 4 ? launch_compress_as<4, 16, false, true>(args...)
                 : early ? launch_compress_16bit<16, true>(split, args...) : launch_compress_16bit<16, false>(split, args...);
        case 32:
            return w == 2 ? launch_compress_16bit<32, false>(split, args...)
                 : early ? launch_compress_as<4, 32, false, true>(args...) : launch_compress_as<4, 32, false, false>(args...);
        case 64:
            if (w == 4) return launch_compress_as<4, 64, false, false, false>(args...);
    }
    return hipErrorInvalidValue;   // choose_shape() returns nothing else
}

// The decoder has one tile size (its waves are independent; one staging step per
// wave measures best at every size).
template <typename... Args>
hipError_t launch_decompress(int w, Output output, Args... args) {
    if (output == Output::kShifted)
        return w == 4 ? launch_decompress_as<4, kMinLoads, Output::kShifted>(args...)
                      : launch_decompress_as<2, kMinLoads, Output::kShifted>(args...);
    return w == 4 ? launch_decompress_as<4, kMinLoads, Output::kAligned>(args...)
                  : launch_decompress_as<2, kMinLoads, Output::kAligned>(args...);
}

// How a planar decoder writes its output (us, as the output lies | shifted, density 0.3 where not stated).
// Two launches: a store that begins in the middle of a line costs 5 to 30 %, but in 64-byte steps only
// the largest fp32 outputs gain, 300 MB 74.0 | 73.1, 784 MB at 0.5 209.7 | 203.9, while 20 MB take 9.7 | 9.9, bf16
// 400 MB 100.4 | 102.8.  16-byte steps: fp32 20 MB at 0.5 10.5 | 9.7, 300 MB 80.7 | 73.0; bf16 20 MB 10.8 | 10.1.
// One launch: from 16-byte steps on as they lie (13 MB fp32 7.23 | 7.34, bf16 7.5 | 7.8), and below 8 MB in any case,
// where the shifted pieces' longer chain counts more (odd elements, fp32 0.25 MB 4.2 | 4.4, 4 MB 5.4 | 5.6, 9 MB
// 7.0 | 6.8, 13 MB 8.3 | 7.5; bf16 0.25 MB 4.4 | 4.7, 4 MB 5.7 | 5.9, 9 MB 7.5 | 7.3, 13 MB 8.8 | 7.8).
inline Output planar_output(const void* out, size_t bytes, int w, bool one_launch) {
    const size_t step = one_launch ? 16 : w == 4 && bytes >= (size_t{256} << 20) ? 128 : 64;
    return aligned_to(out, step) ? Output::kAligned
         : one_launch && bytes < (size_t{8} << 20) ? Output::kLoose : Output::kShifted;
}

// The one-launch decoders for (w, output, eight waves or four, with the streaming hint or not).  The smallest tensors' outputs are written as they lie.
template <int W>
auto direct_decoder_as(Output output, bool eight) {
    return output == Output::kAligned ? (eight ? decompress_direct_kernel<W, Output::kAligned, 8> : decompress_direct_kernel<W, Output::kAligned, 4>)
                                      : (eight ? decompress_direct_kernel<W, Output::kLoose, 8> : decompress_direct_kernel<W, Output::kLoose, 4>);
}
inline auto direct_decoder(int w, Output output, bool eight) {
    return w == 4 ? direct_decoder_as<4>(output, eight) : direct_decoder_as<2>(output, eight);
}
template <int W, bool STREAM>
auto scan_decoder_as(Output output, bool eight) {
    switch (output) {
        case Output::kLoose: return eight ? decompress_scan_kernel<W, Output::kLoose, 8, STREAM> : decompress_scan_kernel<W, Output::kLoose, 4, STREAM>;
        case Output::kShifted: return eight ? decompress_scan_kernel<W, Output::kShifted, 8, STREAM> : decompress_scan_kernel<W, Output::kShifted, 4, STREAM>;
        default: return eight ? decompress_scan_kernel<W, Output::kAligned, 8, STREAM> : decompress_scan_kernel<W, Output::kAligned, 4, STREAM>;
    }
}
inline auto scan_decoder(int w, Output output, bool eight, bool stream_values) {
    if (stream_values) return w == 4 ? scan_decoder_as<4, true>(output, eight) : scan_decoder_as<2, true>(output, eight);
    return w == 4 ? scan_decoder_as<4, false>(output, eight) : scan_decoder_as<2, false>(output, eight);
}

// `bounded`: out_cap may be anything from the size of the mask area up; the
// kernel then writes only runs that end inside it.
// `scan_state_only`: the workspace need only hold the header and the scan state
// of this call's tiles (the library's own scratch array, which no decoder uses).
zvc_status compress_impl(Encoder mode, bool bounded, const void* d_in, size_t n, int w, void* d_out,
                         size_t out_cap, uint64_t* d_bytes, uint64_t* d_offsets, void* d_ws, size_t ws,
                         hipStream_t stream, bool scan_state_only = false, unsigned window_shift = 0,
                         unsigned long long* h_bytes = nullptr) {
    if (w != 2 && w != 4) return ZVC_E_WIDTH;
    if (d_bytes == nullptr || ((d_in == nullptr || d_out == nullptr) && n != 0)) return ZVC_E_ARG;
    if (!aligned_to(d_in, static_cast<size_t>(w)) || !aligned_to(d_out, 4) ||
        !aligned_to(d_bytes, 8))
        return ZVC_E_ALIGN;
    const size_t worst = zvc_max_compressed_bytes(n, w);
    if (out_cap < (bounded ? zvc_mask_bytes(n) : worst)) return ZVC_E_CAPACITY;
    if (ranges_overlap(d_in, n * static_cast<size_t>(w), d_out, out_cap < worst ? out_cap : worst))
        return ZVC_E_ARG;
    if (!scan_state_only)
        if (zvc_status st = check_workspace(d_ws, ws, n, w)) return st;
    unsigned long long* out_bytes = reinterpret_cast<unsigned long long*>(d_bytes);
    if (n == 0) {
        hipError_t e = launch(write_word_kernel, dim3(1), dim3(1), stream, out_bytes, 0ull);
        if (e == hipSuccess && mode == Encoder::kWindowed)
            e = launch(write_word_kernel, dim3(1), dim3(1), stream,
                       reinterpret_cast<unsigned long long*>(d_offsets), 0ull);
        return hip_ok(e);
    }
    const bool split = !aligned_to(d_in, 4);        // 16-bit elements at an odd half dword
    const TileShape shape = choose_shape(n, w, mode == Encoder::kWindowed);
    const size_t tiles = div_up(n * static_cast<size_t>(w), static_cast<size_t>(shape.waves) * shape.chunks * kChunkBytes);
    if (tiles > 0x7FFFFFFFull) return ZVC_E_ARG;
    if (scan_state_only && kHeaderBytes + scan_state_bytes(tiles) > ws) return ZVC_E_WORKSPACE;
    const size_t groups = div_up(n, 32);
    const unsigned char* in = static_cast<const unsigned char*>(d_in);
    unsigned* masks = static_cast<unsigned*>(d_out);
    unsigned char* values = static_cast<unsigned char*>(d_out) + 4 * groups;
    return hip_ok(launch_compress(w, shape, split, choose_early(n, w), mode, stream, in, n, masks,
                    mode == Encoder::kWindowed ? static_cast<unsigned char*>(d_out) : values,
                    static_cast<WsHeader*>(d_ws), out_bytes, h_bytes, static_cast<unsigned>(tiles), groups,
                    !bounded ? ~0ull : out_cap - (mode == Encoder::kWindowed ? 0 : 4 * groups),
                    reinterpret_cast<unsigned long long*>(d_offsets), window_shift));
}

// One event per host thread and GPU for ordering a copy stream after a compute
// stream (or the other way round), created at first use and kept: creating and
// destroying one per call costs several microseconds per tensor.  An ordinary event, which
// releases what lies before it to the whole system: the host reads the size behind one, and
// the documents promise that of no cheaper kind (hipEventDisableSystemFence is for timing,
// 1 to 4 us less a round trip; hipEventReleaseToDevice where that would do: nothing).
hipEvent_t thread_event() {
    thread_local hipEvent_t events[kMaxDevices] = {};
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) return nullptr;
    if (events[device] == nullptr &&
        hipEventCreateWithFlags(&events[device], hipEventDisableTiming) != hipSuccess)
        events[device] = nullptr;
    return events[device];
}

// Where the GPU sees the 8 bytes at `host`, if they are pinned host memory; else null.
unsigned long long* mapped_word(const void* host) {
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, host) != hipSuccess || a.type != hipMemoryTypeHost || !aligned_to(a.devicePointer, 8))
        return nullptr;
    return static_cast<unsigned long long*>(a.devicePointer);
}

// The streams cross the link by hipMemcpyAsync, at every size.  A kernel of this library on
// `copy` starts sooner (a round trip of 1.6 MB on an idle GPU: 48.6 us instead of 57.5),
// but it waits for compute units that the program's own work holds, and keeps them from
// it.  us a layer of one 140 us matrix product and the copy of one tensor beside it (fp32,
// density 0.3), kernel | hipMemcpyAsync: 24.5 MB out 287 | 167, in 233 | 169; 6.1 MB out 174 |
// 160, in 150 | 132; 1.6 MB out 159 | 158, in 134 | 130.
zvc_status offload_impl(Encoder mode, const void* d_in, size_t n, int w, void* d_stage,
                        size_t stage_cap, void* h_pinned, size_t h_cap, uint64_t* h_bytes, void* d_ws,
                        size_t ws, hipStream_t compute, hipStream_t copy) {
    if (w != 2 && w != 4) return ZVC_E_WIDTH;
    if (h_bytes == nullptr || (h_pinned == nullptr && n != 0)) return ZVC_E_ARG;
    if (h_cap < zvc_max_compressed_bytes(n, w)) return ZVC_E_CAPACITY;
    if (zvc_status st = check_workspace(d_ws, ws, n, w)) return st;
    WsHeader* hdr = static_cast<WsHeader*>(d_ws);
    uint64_t* d_size = reinterpret_cast<uint64_t*>(&hdr->size_word);
    // The encoder writes the size to the host itself where it can (a copy of 8 bytes costs 9 us); the
    // size word in the header survives until the next offload on this workspace.
    unsigned long long* const size_to = n != 0 ? mapped_word(h_bytes) : nullptr;
    if (zvc_status st = compress_impl(mode, false, d_in, n, w, d_stage, stage_cap, d_size, nullptr, d_ws,
                                      ws, compute, false, 0, size_to))
        return st;
    if (size_to == nullptr && hipMemcpyAsync(h_bytes, d_size, 8, hipMemcpyDeviceToHost, compute) != hipSuccess)
        return ZVC_E_HIP;
    hipEvent_t ev = thread_event();
    if (ev == nullptr || hipEventRecord(ev, compute) != hipSuccess || hipEventSynchronize(ev) != hipSuccess)
        return ZVC_E_HIP;
    if (*h_bytes > h_cap) return ZVC_E_CAPACITY;
    // (what the event ordered is done and released to the system, so `copy` has nothing to wait for)
    if (*h_bytes == 0) return ZVC_OK;
    return hip_ok(hipMemcpyAsync(h_pinned, d_stage, *h_bytes, hipMemcpyDeviceToHost, copy));
}

// Scratch of zvc_compress_static: header and scan state for tensors of up to
// ZVC_STATIC_MAX_BYTES.  Zero when the code object is loaded, which is the
// state zvc_workspace_init gives a caller's workspace.  Each GPU holds its own copy at its own address.
constexpr size_t kStaticScratchBytes = ZVC_STATIC_SCRATCH_BYTES;
static_assert(kHeaderBytes + 8 * (ZVC_STATIC_MAX_BYTES / (32 << 10)) <= kStaticScratchBytes &&
              kHeaderBytes + 8 * (medium_bytes(2, true) / (16 << 10)) <= kStaticScratchBytes, "scratch holds the scan state of every call");
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];           // device address of `scratch` on each GPU, once looked up

// Device address of the current GPU's copy of `scratch` (looked up once per GPU).
zvc_status static_scratch(void** ptr) {
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) return ZVC_E_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[device] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return ZVC_E_HIP;
        g_scratch_ptr[device] = p;
    }
    *ptr = g_scratch_ptr[device];
    return ZVC_OK;
}

}  // namespace

// ------------------------------------------------------------------ C ABI
extern "C" {

const char* zvc_status_string(int status) {
    switch (status) {
        case ZVC_OK: return "ZVC_OK";
        case ZVC_E_ARG: return "ZVC_E_ARG: invalid argument";
        case ZVC_E_WIDTH: return "ZVC_E_WIDTH: element width must be 2 or 4 bytes";
        case ZVC_E_CAPACITY: return "ZVC_E_CAPACITY: output buffer below the worst-case size";
        case ZVC_E_WORKSPACE: return "ZVC_E_WORKSPACE: workspace too small";
        case ZVC_E_ALIGN: return "ZVC_E_ALIGN: pointer alignment";
        case ZVC_E_HIP: return "ZVC_E_HIP: a HIP runtime call failed";
        case ZVC_E_CORRUPT: return "ZVC_E_CORRUPT: compressed stream inconsistent with its size";
    }
    return "ZVC: unknown status";
}

size_t zvc_mask_bytes(size_t n) { return 4 * div_up(n, 32); }

size_t zvc_max_compressed_bytes(size_t n, int w) {
    if (w != 2 && w != 4) return 0;
    return zvc_mask_bytes(n) + static_cast<size_t>(w) * n;
}

size_t zvc_workspace_bytes(size_t n, int w) {
    if (w != 2 && w != 4) return 0;
    // 4 bytes per smallest tile (and more) and the decoder's arrays, 524 bytes per 131072 elements: together
    // they hold the scan state, 8 bytes per tile
    const size_t tiles = tiles_for(n, w, kMinLoads);
    return kHeaderBytes + 256 * (div_up(tiles, 64) + div_up(tiles, 64 * 128)) +
           decoder_area_bytes(div_up(div_up(n, 32), kChunkMasks));
}

zvc_status zvc_check_stream(const void* h_comp, uint64_t bytes, size_t n, int w) {
    if (w != 2 && w != 4) return ZVC_E_WIDTH;
    if (h_comp == nullptr && bytes != 0) return ZVC_E_ARG;
    const size_t groups = div_up(n, 32);
    if (bytes < 4 * groups) return ZVC_E_CORRUPT;
    const unsigned char* p = static_cast<const unsigned char*>(h_comp);
    uint64_t kept = 0;
    for (size_t g = 0; g < groups; ++g) {
        uint32_t m;
        std::memcpy(&m, p + 4 * g, 4);
        if (g == groups - 1 && n % 32 != 0 && (m >> (n % 32)) != 0) return ZVC_E_CORRUPT;
        kept += static_cast<uint64_t>(__builtin_popcount(m));
    }
    return bytes == 4 * groups + static_cast<uint64_t>(w) * kept ? ZVC_OK : ZVC_E_CORRUPT;
}

zvc_status zvc_window_check_stream(const void* h_stream, uint64_t bytes, const uint64_t* h_offsets,
                                   size_t n, int w, size_t window_bytes) {
    if (w != 2 && w != 4) return ZVC_E_WIDTH;
    if (window_shift_of(window_bytes) < 0) return ZVC_E_ARG;
    if (h_offsets == nullptr || (h_stream == nullptr && bytes != 0)) return ZVC_E_ARG;
    const size_t windows = zvc_window_count(n, w, window_bytes);
    const size_t groups = div_up(n, 32);
    const size_t groups_per_window = window_bytes / static_cast<size_t>(w) / 32;
    const unsigned char* p = static_cast<const unsigned char*>(h_stream);
    if (h_offsets[0] != 0 || h_offsets[windows] != bytes) return ZVC_E_CORRUPT;
    for (size_t k = 0; k < windows; ++k) {
        uint64_t pos = h_offsets[k];
        const uint64_t end = h_offsets[k + 1];
        if (end < pos || end > bytes) return ZVC_E_CORRUPT;
        const size_t g0 = k * groups_per_window;
        const size_t g1 = g0 + groups_per_window < groups ? g0 + groups_per_window : groups;
        for (size_t g = g0; g < g1; ++g) {      // the walk of section 5.2: mask, then its popcount of elements
            if (pos + 4 > end) return ZVC_E_CORRUPT;
            const uint32_t m = static_cast<uint32_t>(p[pos]) | (static_cast<uint32_t>(p[pos + 1]) << 8) |
                               (static_cast<uint32_t>(p[pos + 2]) << 16) |
                               (static_cast<uint32_t>(p[pos + 3]) << 24);
            if (g == groups - 1 && n % 32 != 0 && (m >> (n % 32)) != 0) return ZVC_E_CORRUPT;
            pos += 4 + static_cast<uint64_t>(w) * static_cast<uint64_t>(__builtin_popcount(m));
        }
        if (pos != end) return ZVC_E_CORRUPT;
    }
    return ZVC_OK;
}

zvc_status zvc_workspace_init(void* d_ws, size_t ws, hipStream_t stream) {
    if (d_ws == nullptr) return ZVC_E_ARG;
    if (!aligned_to(d_ws, 256)) return ZVC_E_ALIGN;
    if (ws < kHeaderBytes) return ZVC_E_WORKSPACE;
    return launch_reset(d_ws, (ws - kHeaderBytes) / 8 * 8, stream);
}

zvc_status zvc_workspace_set_lookback_patience(void* d_ws, unsigned polls, hipStream_t stream) {
    if (d_ws == nullptr) return ZVC_E_ARG;
    if (!aligned_to(d_ws, 256)) return ZVC_E_ALIGN;
    WsHeader* hdr = static_cast<WsHeader*>(d_ws);
    return hip_ok(launch(write_word_kernel, dim3(1), dim3(1), stream, &hdr->patience_plus_one,
                         static_cast<unsigned long long>(polls) + 1ull));
}

zvc_status zvc_reference_stream(const void* d_in, size_t read_bytes, void* d_out, size_t write_bytes,
                                hipStream_t stream) {
    if ((d_in == nullptr && read_bytes != 0) || (d_out == nullptr && write_bytes != 0)) return ZVC_E_ARG;
    if (!aligned_to(d_in, 16) || !aligned_to(d_out, 16) || read_bytes % 16 != 0 || write_bytes % 16 != 0)
        return ZVC_E_ALIGN;
    if (ranges_overlap(d_in, read_bytes, d_out, write_bytes)) return ZVC_E_ARG;
    const size_t larger = read_bytes > write_bytes ? read_bytes : write_bytes;
    if (larger == 0) return ZVC_OK;
    const bool small = larger < (size_t{32} << 20);
    const size_t group_bytes = static_cast<size_t>(kThreads) * 16 * (small ? 4 : 16);     // 16 KB | 64 KB
    const size_t groups = div_up(larger, group_bytes);
    if (groups > 0x7FFFFFFFull) return ZVC_E_ARG;
    const size_t read_chunks = read_bytes / 16, write_chunks = write_bytes / 16;
    return hip_ok(launch(small ? reference_stream_kernel<4> : reference_stream_kernel<16>,
                         dim3(static_cast<unsigned>(groups)), dim3(kThreads), stream,
                         static_cast<const uint4*>(d_in), read_chunks, static_cast<uint4*>(d_out), write_chunks,
                         static_cast<unsigned>(div_up(read_chunks, groups)),
                         static_cast<unsigned>(div_up(write_chunks, groups))));
}

zvc_status zvc_workspace_self_help_count(const void* d_ws, uint64_t* h_count) {
    if (d_ws == nullptr || h_count == nullptr) return ZVC_E_ARG;
    const WsHeader* hdr = static_cast<const WsHeader*>(d_ws);
    return hip_ok(hipMemcpy(h_count, &hdr->helped, 8, hipMemcpyDeviceToHost));
}

zvc_status zvc_compressed_size(const void* d_in, size_t n, int w, uint64_t* d_bytes, void* d_ws,
                               size_t ws, hipStream_t stream) {
    if (w != 2 && w != 4) return ZVC_E_WIDTH;
    if (d_bytes == nullptr || (d_in == nullptr && n != 0)) return ZVC_E_ARG;
    if (!aligned_to(d_in, static_cast<size_t>(w)) || !aligned_to(d_bytes, 8)) return ZVC_E_ALIGN;
    if (zvc_status st = check_workspace(d_ws, ws, n, w)) return st;
    unsigned long long* out = reinterpret_cast<unsigned long long*>(d_bytes);
    if (n == 0) {
        return hip_ok(launch(write_word_kernel, dim3(1), dim3(1), stream, out, 0ull));
    }
    WsHeader* hdr = static_cast<WsHeader*>(d_ws);   // accumulators are zero between calls
    const unsigned char* in = static_cast<const unsigned char*>(d_in);
    const size_t groups = div_up(n, 32);
    const unsigned before = static_cast<unsigned>(reinterpret_cast<uintptr_t>(d_in) % 16);   // bytes
    const size_t tiles = div_up(before + n * static_cast<size_t>(w), static_cast<size_t>(kThreads) * 16 * kCountLoads);
    if (tiles > 0x7FFFFFFFull) return ZVC_E_ARG;
    const dim3 grid(static_cast<unsigned>(tiles)), block(kThreads);
    const unsigned nt = static_cast<unsigned>(tiles), skip = before / static_cast<unsigned>(w);
    const bool al = skip == 0;
    const auto kernel = w == 4 ? (al ? count_kernel<4, true> : count_kernel<4, false>)
                               : (al ? count_kernel<2, true> : count_kernel<2, false>);
    return hip_ok(launch(kernel, grid, block, stream, in - before, skip, n + skip, hdr, out, groups, nt));
}

zvc_status zvc_compress(const void* d_in, size_t n, int w, void* d_out, size_t out_cap,
                        uint64_t* d_bytes, void* d_ws, size_t ws, hipStream_t stream) {
    return compress_impl(Encoder::kPlain, false, d_in, n, w, d_out, out_cap, d_bytes, nullptr, d_ws, ws,
                         stream);
}

zvc_status zvc_compress_static(const void* d_in, size_t n, int w, void* d_out, size_t out_cap,
                               uint64_t* d_bytes, hipStream_t stream) {
    if (w != 2 && w != 4) return ZVC_E_WIDTH;
    if (n > ZVC_STATIC_MAX_BYTES / static_cast<size_t>(w)) return ZVC_E_WORKSPACE;
    void* ws = nullptr;
    if (zvc_status st = static_scratch(&ws)) return st;
    return compress_impl(Encoder::kPlain, false, d_in, n, w, d_out, out_cap, d_bytes, nullptr, ws,
                         kStaticScratchBytes, stream, true);
}

zvc_status zvc_relu_compress(const void* d_in, size_t n, int w, void* d_out, size_t out_cap,
                             uint64_t* d_bytes, void* d_ws, size_t ws, hipStream_t stream) {
    return compress_impl(Encoder::kRelu, false, d_in, n, w, d_out, out_cap, d_bytes, nullptr, d_ws, ws,
                         stream);
}

zvc_status zvc_compress_bounded(const void* d_in, size_t n, int w, int relu, void* d_out, size_t out_cap,
                                uint64_t* d_bytes, void* d_ws, size_t ws, hipStream_t stream) {
    if (relu != 0 && relu != 1) return ZVC_E_ARG;
    return compress_impl(relu ? Encoder::kRelu : Encoder::kPlain, true, d_in, n, w, d_out, out_cap,
                         d_bytes, nullptr, d_ws, ws, stream);
}

size_t zvc_window_elements(int w, size_t window_bytes) {
    if ((w != 2 && w != 4) || window_shift_of(window_bytes) < 0) return 0;
    return window_bytes / static_cast<size_t>(w);
}

size_t zvc_window_count(size_t n, int w, size_t window_bytes) {
    if ((w != 2 && w != 4) || window_shift_of(window_bytes) < 0) return 0;
    return div_up(n * static_cast<size_t>(w), window_bytes);
}

zvc_status zvc_window_compress(const void* d_in, size_t n, int w, size_t window_bytes, void* d_out,
                               size_t out_cap, uint64_t* d_offsets, uint64_t* d_bytes, void* d_ws,
                               size_t ws, hipStream_t stream) {
    if (d_offsets == nullptr) return ZVC_E_ARG;
    if (!aligned_to(d_offsets, 8)) return ZVC_E_ALIGN;
    const int shift = window_shift_of(window_bytes);
    if (shift < 0) return ZVC_E_ARG;
    if (w == 2 || w == 4) {
        const size_t table = 8 * (zvc_window_count(n, w, window_bytes) + 1);
        if (ranges_overlap(d_offsets, table, d_out, zvc_max_compressed_bytes(n, w)) ||
            ranges_overlap(d_offsets, table, d_in, n * static_cast<size_t>(w)))
            return ZVC_E_ARG;
    }
    return compress_impl(Encoder::kWindowed, false, d_in, n, w, d_out, out_cap, d_bytes, d_offsets, d_ws, ws,
                         stream, false, static_cast<unsigned>(shift));
}

zvc_status zvc_window_decompress(const void* d_stream, size_t stream_bytes, const uint64_t* d_offsets,
                                 size_t n, int w, size_t window_bytes, size_t first_window,
                                 size_t num_windows, void* d_out, hipStream_t stream) {
    if (w != 2 && w != 4) return ZVC_E_WIDTH;
    const int shift = window_shift_of(window_bytes);
    if (shift < 0) return ZVC_E_ARG;
    const size_t windows = zvc_window_count(n, w, window_bytes);
    if (first_window > windows || num_windows > windows - first_window) return ZVC_E_ARG;
    if (num_windows == 0) return ZVC_OK;
    if (d_stream == nullptr || d_offsets == nullptr || d_out == nullptr) return ZVC_E_ARG;
    if (!aligned_to(d_out, static_cast<size_t>(w)) || !aligned_to(d_stream, static_cast<size_t>(w)) ||
        !aligned_to(d_offsets, 8))
        return ZVC_E_ALIGN;
    const size_t elems_per_window = window_bytes / static_cast<size_t>(w);
    const size_t last_elem = (first_window + num_windows) * elems_per_window < n
                                 ? (first_window + num_windows) * elems_per_window : n;
    const size_t out_bytes = (last_elem - first_window * elems_per_window) * static_cast<size_t>(w);
    if (ranges_overlap(d_stream, stream_bytes, d_out, out_bytes)) return ZVC_E_ARG;
    const unsigned char* in = static_cast<const unsigned char*>(d_stream);
    const unsigned long long* offs = reinterpret_cast<const unsigned long long*>(d_offsets);
    unsigned char* out = static_cast<unsigned char*>(d_out);
    const size_t groups = div_up(n, 32);
    const bool al = aligned_to(d_out, 16);
    if (shift >= kSplitShift) {
        return hip_ok(w == 4 ? launch_window_split<4>(1 << (shift - 2), al, stream, in, stream_bytes, offs, n, groups,
                                                      first_window, num_windows, out)
                             : launch_window_split<2>(1 << (shift - 2), al, stream, in, stream_bytes, offs, n, groups,
                                                      first_window, num_windows, out));
    }
    // a wave takes 4 KB of output
    const size_t wave_windows = static_cast<size_t>(kStageLoads >> shift);
    // (a multiple of 8 workgroups for the interleaved order)
    const size_t blocks = div_up(div_up(num_windows, static_cast<size_t>(kWaves) * wave_windows), 8) * 8;
    if (blocks > 0x7FFFFFFFull) return ZVC_E_ARG;
    const dim3 grid(static_cast<unsigned>(blocks)), block(kThreads);
    const bool interleave = interleaves_windows(n, w, shift, stream_bytes, out_bytes);
    const auto kernel = w == 4 ? (al ? window_decode_kernel<4, true> : window_decode_kernel<4, false>)
                               : (al ? window_decode_kernel<2, true> : window_decode_kernel<2, false>);
    return hip_ok(launch(kernel, grid, block, stream, in, static_cast<unsigned long long>(stream_bytes), offs, n,
                         groups, first_window, num_windows, static_cast<unsigned>(shift), out, interleave));
}

zvc_status zvc_decompress(const void* d_comp, size_t comp_bytes, size_t n, int w, void* d_out,
                          void* d_ws, size_t ws, hipStream_t stream) {
    if (w != 2 && w != 4) return ZVC_E_WIDTH;
    if ((d_comp == nullptr || d_out == nullptr) && n != 0) return ZVC_E_ARG;
    if (!aligned_to(d_out, static_cast<size_t>(w)) || !aligned_to(d_comp, 4)) return ZVC_E_ALIGN;
    if (comp_bytes < zvc_mask_bytes(n)) return ZVC_E_CAPACITY;
    if (ranges_overlap(d_comp, comp_bytes, d_out, n * static_cast<size_t>(w))) return ZVC_E_ARG;
    if (zvc_status st = check_workspace(d_ws, ws, n, w)) return st;
    if (n == 0) return ZVC_OK;
    // a multiple of 8 workgroups: the interleaved order deals the parts out in rounds of 8
    const size_t tiles = div_up(tiles_for(n, w, kMinLoads), 8) * 8;
    if (tiles > 0x7FFFFFFFull) return ZVC_E_ARG;
    const size_t groups = div_up(n, 32);
    const unsigned char* stream_values_at = static_cast<const unsigned char*>(d_comp) + 4 * groups;
    const unsigned long long stored_avail = (comp_bytes - 4 * groups) / static_cast<size_t>(w);
    const Decoder decoder = choose_decoder(n, w, d_out, stored_avail);
    const Output output = planar_output(d_out, n * static_cast<size_t>(w), w, decoder != Decoder::kTwoLaunches);
    if (decoder != Decoder::kTwoLaunches) {
        const bool eight = decoder == Decoder::kScan8 || decoder == Decoder::kDirect8;
        const unsigned waves = eight ? 8u : 4u, one_tiles = static_cast<unsigned>(
            div_up(n * static_cast<size_t>(w), size_t{kStageLoads * kSlotBytes} * waves));
        const dim3 grid(one_tiles), block(waves * kWaveSize);
        const unsigned* masks = static_cast<const unsigned*>(d_comp);
        unsigned char* out = static_cast<unsigned char*>(d_out);
        const bool stream_values = stored_avail >= n / 4 * 3;
        if (decoder == Decoder::kDirect4 || decoder == Decoder::kDirect8)
            return hip_ok(launch(direct_decoder(w, output, eight), grid, block, stream, masks, stream_values_at, stored_avail,
                                 n, out, groups, stream_values));
        // the workgroups find their offsets with the encoder's scan (its state is at the front of the workspace)
        return hip_ok(launch(scan_decoder(w, output, eight, stream_values), grid, block, stream, masks, stream_values_at, stored_avail, n,
                             out, static_cast<WsHeader*>(d_ws), one_tiles, groups));
    }
    const size_t chunks = div_up(groups, kChunkMasks);
    if (chunks > 0xFFFFFFFFull) return ZVC_E_ARG;
    // The pre-pass arrays need no reset, and what they leave behind is no count of a later call's (see there).
    unsigned char* area = static_cast<unsigned char*>(d_ws) + (ws - decoder_area_bytes(chunks)) / 256 * 256;
    unsigned long long* chunk_prefix =
        chunks <= kFewChunks ? nullptr : reinterpret_cast<unsigned long long*>(area);
    unsigned* chunk_total = reinterpret_cast<unsigned*>(area + pad256(8 * chunks));
    unsigned* unit_end = reinterpret_cast<unsigned*>(area + pad256(8 * chunks) + pad256(4 * chunks));
    const unsigned* masks = static_cast<const unsigned*>(d_comp);
    if (launch(mask_prefix_kernel, dim3(static_cast<unsigned>(chunks)), dim3(kThreads), stream, masks,
               groups, static_cast<unsigned>(n % 32), unit_end, chunk_total, chunk_prefix,
               static_cast<WsHeader*>(d_ws), static_cast<unsigned>(chunks)) != hipSuccess)
        return ZVC_E_HIP;
    const unsigned char* values = static_cast<const unsigned char*>(d_comp) + 4 * groups;
    const unsigned long long avail = (comp_bytes - 4 * groups) / static_cast<size_t>(w);
    return hip_ok(launch_decompress(w, output, dim3(static_cast<unsigned>(tiles)), stream, masks, values, avail, n,
                                    static_cast<unsigned char*>(d_out), unit_end, chunk_prefix, chunk_total,
                                    groups));
}

zvc_status zvc_offload(const void* d_in, size_t n, int w, void* d_stage, size_t stage_cap,
                       void* h_pinned, size_t h_cap, uint64_t* h_bytes, void* d_ws, size_t ws,
                       hipStream_t compute, hipStream_t copy) {
    return offload_impl(Encoder::kPlain, d_in, n, w, d_stage, stage_cap, h_pinned, h_cap, h_bytes, d_ws,
                        ws, compute, copy);
}

zvc_status zvc_relu_offload(const void* d_in, size_t n, int w, void* d_stage, size_t stage_cap,
                            void* h_pinned, size_t h_cap, uint64_t* h_bytes, void* d_ws, size_t ws,
                            hipStream_t compute, hipStream_t copy) {
    return offload_impl(Encoder::kRelu, d_in, n, w, d_stage, stage_cap, h_pinned, h_cap, h_bytes, d_ws,
                        ws, compute, copy);
}

zvc_status zvc_prefetch(const void* h_pinned, uint64_t bytes, size_t n, int w, void* d_stage,
                        size_t stage_cap, void* d_out, void* d_ws, size_t ws, hipStream_t copy,
                        hipStream_t compute) {
    if (w != 2 && w != 4) return ZVC_E_WIDTH;
    if ((h_pinned == nullptr || d_stage == nullptr) && bytes != 0) return ZVC_E_ARG;
    if (bytes < zvc_mask_bytes(n) || bytes > zvc_max_compressed_bytes(n, w)) return ZVC_E_CORRUPT;
    if (stage_cap < bytes) return ZVC_E_CAPACITY;
    if ((d_out == nullptr && n != 0)) return ZVC_E_ARG;
    if (!aligned_to(d_out, static_cast<size_t>(w)) || !aligned_to(d_stage, 4)) return ZVC_E_ALIGN;
    if (zvc_status st = check_workspace(d_ws, ws, n, w)) return st;
    if (n == 0) return ZVC_OK;
    if (hipMemcpyAsync(d_stage, h_pinned, bytes, hipMemcpyHostToDevice, copy) != hipSuccess) return ZVC_E_HIP;
    if (copy != compute) {
        hipEvent_t ev = thread_event();
        if (ev == nullptr || hipEventRecord(ev, copy) != hipSuccess ||
            hipStreamWaitEvent(compute, ev, 0) != hipSuccess)
            return ZVC_E_HIP;
    }
    return zvc_decompress(d_stage, bytes, n, w, d_out, d_ws, ws, compute);
}

}  // extern "C"
