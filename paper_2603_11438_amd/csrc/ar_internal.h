// Internal declarations shared by the host runtime and the HIP kernels of
// libar.  Not part of the C ABI (see include/ar.h).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "ar.h"

namespace ar {

// Flag memory layout: every connection (channel c, wave w, sender rank r,
// i.e. the link r -> r+1 of one wave's ring) owns two 128-byte lines, so no
// two counters written by different waves share a cache line.
//   tail: messages the sender has published on the link (sender writes)
//   head: messages the receiver has consumed on the link (receiver writes)
// The sender's tail line also holds, at u64 offset kEpochU64, that wave's
// message epoch: the absolute index of its next run's first message.
constexpr int kFlagLineU64 = 16;                 // 128 bytes
constexpr int kConnFlagU64 = 2 * kFlagLineU64;   // tail line + head line
constexpr int kEpochU64 = 8;                     // epoch: byte 64 of the tail line
constexpr int kCtlU32 = 64;                      // control block: 256 bytes
constexpr int kCtlAbort = 0;                     // nonzero: every wave must leave
constexpr int kCtlStatus = 32;                   // sticky AR_ERR_* bit set
// Line-check counters of AR_DEBUG_CHECK_LINES, 64-bit, at these u32 indices
// (bytes 64..87, a line of their own).
constexpr int kCtlLinesChecked = 16;             // LL / LL128 lines accepted and checked
constexpr int kCtlLinesFirst = 18;               // of those, accepted on the first load
constexpr int kCtlLinesBad = 20;                 // of those, data not matching the flag
// A step record of AR_DEBUG_TRACE: this many 64-bit fields.
constexpr int kTraceFields = 8;

// Status bits written by the kernel into ctl[kCtlStatus].
constexpr uint32_t kStatusTimeout = 1u;

// Everything a ring kernel launch needs; passed by value as the kernel
// argument.  Counts are in elements of the plan's dtype.
struct RingArgs {
    const char *src[AR_MAX_RANKS];   // rank inputs
    char *dst[AR_MAX_RANKS];         // rank outputs (== src for in place)
    char *fifo;                      // all FIFO slots
    uint64_t *flags;                 // per-connection head/tail lines
    uint32_t *ctl;                   // abort word + status word
    uint64_t count;                  // elements of the segmented buffer (AllReduce: count;
                                     // ReduceScatter / AllGather: N blocks of count)
    uint64_t seg;                    // segment length (ReduceScatter / AllGather: one block)
    uint64_t cs;                     // per-channel sub-range of a segment
    uint64_t chunk;                  // per-(segment, channel) ring step
    uint64_t kw;                     // one wave's share of a chunk step
    uint64_t part;                   // elements of segment full_segs (0 .. seg-1)
    uint64_t slot_bytes;             // bytes of one FIFO slot
    uint64_t timeout_ticks;          // watchdog, in 100 MHz real-time ticks
    uint32_t nranks, nchannels, nwaves, depth, nchunks, placement, debug;
    uint32_t ll128_ordered;          // AR_PLAN_LL128_ORDERED: lines only from loads after their flags
    uint32_t coll;                   // AR_COLL_*: which steps of the ring run
    uint32_t full_segs;              // segments 0 .. full_segs-1 hold seg elements; segment
                                     // full_segs holds part, any later one none
    uint64_t *trace;                 // AR_DEBUG_TRACE: step records, rank r's at
                                     // [r * trace_per_rank, (r + 1) * trace_per_rank)
    uint32_t trace_per_rank;         // records per rank (0: none kept)
};

// Resolved plan geometry.  Computed on the host only.
int resolve_geometry(const ar_plan_desc *desc, int max_channels, ar_plan_info *out);

// Protocol defaults.
int default_nwaves(int proto);
int default_depth(int proto);
size_t default_chunk_bytes(int proto);

// Kernel launchers (ar_kernels.hip; launch_ring_lds: ring_lds.hip,
// launch_direct: direct.hip).
int launch_direct(const ar_plan_info &info, const RingArgs &args, void *stream);
int launch_ring_lds(const ar_plan_info &info, const RingArgs &args, void *stream);
int launch_ring(const ar_plan_info &info, const RingArgs &args, void *stream);
int launch_fill_u32(uint32_t *p, size_t n, uint32_t value, void *stream);
int launch_copy(const void *src, void *dst, size_t bytes, void *stream);
int ring_occupancy(int proto, int dtype, int block, int *blocks_per_cu);
int launch_bf16_round(const float *in, uint16_t *out, size_t n, void *stream);

// Workgroups of the direct algorithm have at most kMaxDirectWaves waves: a
// plan's workgroup of more is launched as direct_split workgroups of
// direct_threads threads.
constexpr int kMaxDirectWaves = 8;
constexpr uint32_t direct_split(int nwaves) { return ((uint32_t)nwaves + kMaxDirectWaves - 1) / kMaxDirectWaves; }
constexpr uint32_t direct_threads(int nwaves)
{
    return 64 * (((uint32_t)nwaves + direct_split(nwaves) - 1) / direct_split(nwaves));
}
// The most workgroups per segment that one launch can hold: fewer than 2^32
// threads in all, with one workgroup left for the partial unit.
constexpr uint64_t direct_max_parts(int nranks, int nwaves)
{
    return (0xFFFFFFFFull / direct_threads(nwaves) - 1) / (direct_split(nwaves) * (uint64_t)nranks);
}

// Workgroups (rings) of a ring plan with its links in LDS, for segments of
// seg_b bytes in pieces of piece_b.
//
// The plan's C * N workgroups of W waves become C * N * W / 2 rings of N
// waves, or 4 * C * W where those are more (below eight ranks), so that few
// ranks get as many waves as eight.  Simple default, 16 channels of 4 waves:
// 8 ranks, bf16, 9 MiB 37.9 us with C * N rings, 30.2 with C * N * W / 2; 2
// ranks, fp32, 4 MiB 14.5 us with 64 rings, 6.3 with 256, 32 MiB 97 and 34
// us; 4 ranks, 32 MiB, 128 and 256 rings 76 and 51 us.  The channel and wave
// counts a caller names are thus a limit on the rings, of N waves each, not
// on the waves themselves.
//
// Not more than fill the compute units twice (512 workgroups, more of few
// ranks); where the inputs together exceed half of the 256 MiB last-level
// cache, once: more only widen the stretch of memory that is open at a time (8
// ranks, fp32, 256 against 512 workgroups: 128 MiB 385 and 400 us, 32 MiB 101
// and 104 us), while a message that the cache holds gains from the second
// workgroup per compute unit (8 MiB 24.8 and 23.9 us, 4 MiB 13.1 and 12.1 us).
// Beyond 256 down to a multiple of 256, as many on each compute unit (bf16, 5
// ranks, 16 MiB, 255 / 320 / 380 / 510 workgroups: 31.8 / 41.0 / 33.9 / 31.5
// us; 7 ranks, 48 MiB, 252 and 292: 164 and 204 us); that takes 504 to 511,
// which a table row of 32 channels comes to at 9 and 11 to 15 ranks, to 256
// as well.  At last, not more than there are pieces, whatever that leaves.
inline uint64_t ring_lds_workgroups(const ar_plan_info &g, uint64_t seg_b, uint64_t piece_b)
{
    const uint64_t n = (uint64_t)g.nranks, c = (uint64_t)g.nchannels, w = (uint64_t)g.nwaves;
    const uint64_t pieces = (seg_b + piece_b - 1) / piece_b;
    const uint64_t in_b = seg_b * n * (g.coll == AR_COLL_ALLGATHER ? 1 : n);
    const uint64_t once = n == 2 ? 1024 : n < 5 ? 512 : 256, most = in_b > (128ull << 20) ? once : 2 * once;
    uint64_t grid = c * n * ((w + 1) / 2);
    if (grid < 4 * c * w) grid = 4 * c * w;
    if (grid > most) grid = most;
    if (grid > 256) grid -= grid % 256;
    return grid > pieces ? pieces : grid;
}

// How the outputs of a run in LDS or of the direct algorithm are stored.  All
// ranks' outputs together up to half of the 256 MiB last-level cache: written
// through the L2 to the memory side (sc1), where that cache takes them, and
// where the program that reads them next finds them.  Stores with the
// non-temporal hint would go on to HBM, and what they leave in the L2 is
// written back at the end of the kernel while everything waits (8 ranks,
// AllReduce, device time, non-temporal against sc1: 256 KiB fp32 3.0 and 2.2
// us, 1 MiB bf16 4.2 and 3.3 us, 8 MiB fp32 24.8 and 21.9 us; AllGather of
// 12 MiB 20.8 and 17.4 us; ReduceScatter of 64 MiB bf16 104.7 and 97.1 us).
// More: the hint, which keeps them from driving each other and the inputs out
// (20 MiB bf16 58.4 and 61.8 us, 32 MiB 92.8 and 97 us, 64 MiB fp32 186 and
// 196 us).
//
// What sc1 gains depends on what the cache still holds.  Its time over the
// hint's, direct algorithm, fp32, by the outputs of all ranks: the same
// buffers over and over / three sets in turn / buffers that the cache has lost:
//   AllReduce, 8 ranks      4 MiB .94 / .91 / 1.00    12 MiB .77 / 1.17 / 1.22
//                          24 MiB 1.08 / 1.12 / 1.10  48 MiB .93 / .92 / 1.04
//   ReduceScatter, 8 ranks  2 MiB .94 / 1.11 / 1.09   64 MiB .97 / .95 / .96
//   AllGather, 8 ranks     16 MiB .94 / .95 / 1.05    64 MiB .93 / .89 / 1.09
//   AllGather, 5 ranks     30 MiB .76 / .74 / 1.49    80 MiB .66 / .69 / 1.14
// It costs most where outputs start off the memory side's lines (5 ranks'
// blocks) and the cache has to fetch what a partial line lacks; the direct
// algorithm's iterations therefore start on lines (direct.hip; without that
// the figures above).
inline bool outputs_fit_cache(const ar_plan_info &g)
{
    const uint64_t rank = g.count * (g.dtype == AR_FLOAT32 ? 4 : 2) *
                          (g.coll == AR_COLL_ALLGATHER ? (uint64_t)g.nranks : 1);
    return rank * (uint64_t)g.nranks <= (128ull << 20);
}

// Run-time helpers of ar_runtime.cpp.
// Where a ring plan's links are.  In LDS, unless the plan asks for links in
// memory: FIFO-only plans, and plans with debug flags, whose hooks (skipped
// posts, jitter, the line checker, the step trace) belong to lines and
// counters in memory.
inline bool links_in_lds(const ar_plan_info &g, const ar_plan_desc &d)
{
    return g.algo == AR_ALGO_RING && g.peer_direct && d.debug_flags == 0;
}
constexpr uint32_t kDefaultTimeoutUs = 2000000;  // 2 s per flag wait
constexpr uint64_t kTicksPerUs = 100;            // 100 MHz real-time counter
// Bytes of each rank's send and recv buffer for a collective's geometry.
void buffer_bytes(const ar_plan_info &g, size_t *send_b, size_t *recv_b);
// Rank buffers non-NULL, 16-byte aligned, receive buffers overlapping
// nothing but their own rank's in-place layout: AR_OK or AR_ERR_ARG.
int check_buffers(const ar_plan_info &g, const void *const *send, void *const *recv);
// Workgroups of a ring launch that fit on the current device, per rank.
int device_channel_capacity(int proto, int dtype, int nranks, int nwaves, int *cap);
// Kernel arguments of one run.
void fill_args(const ar_plan_info &g, const ar_plan_desc &d, uint64_t timeout_ticks, const void *const *send,
               void *const *recv, char *fifo, uint64_t *flags, uint32_t *ctl, RingArgs *out);
// The tuner's and defaults' geometry for a description on the current device.
int resolve_for_device(const ar_plan_desc *desc, ar_plan_desc *d_out, ar_plan_info *info_out, int *dev_out);
// Ring memory layout: total bytes, with the flag lines and FIFO offsets.
size_t workspace_layout(const ar_plan_info &info, size_t *flags_off, size_t *fifo_off);

// Thread-local last error.
void set_last_error(int code);

}  // namespace ar
