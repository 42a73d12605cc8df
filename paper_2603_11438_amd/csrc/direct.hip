// The direct (two-shot) algorithm (gfx950), with no links and no waits.
//
// Workgroup b works on segment s = b mod N (part b / N of its parts): a
// thread loads one 16-byte unit of segment s from every rank (ranks s, s+1,
// ..., s+N-1 in that order), sums them in that chain order -- the same
// additions, in the same order, as the ring's reduce-scatter -- and stores
// the result to every rank.  Every element is read once per rank and written
// once per rank: the compulsory 2 N S bytes.  In place is safe: each element
// is read and then written by the same thread.
//
// The same kernel runs the other collectives: ReduceScatter sums block s
// along the chain that starts at rank s+1 (the ring's order for a block that
// ends at rank s) and writes it to rank s only; AllGather copies rank s's
// block to block s of every rank.
//
// What bounds it.  Small messages: launch and the way to the first load, so
// the rank count and the collective are template arguments (no divisions, no
// tests of either, one round of scalar loads: 8 ranks, 4 KiB fp32, 3.0 us as
// one kernel for all collectives and up to 8 ranks, 2.1 us so), and the
// partial unit at the end of the data has a workgroup of its own (100003 bf16
// elements: 8.0 -> 3.1 us).  Large messages: HBM; see units_per_unroll and
// the loop below for what keeps enough of it in flight.
#include "ar_device.h"

namespace ar {
namespace dev {

// What the kernel reads from the kernel argument; sizes in bytes.
struct DirectArgs {
    const char *src[AR_MAX_RANKS];
    char *dst[AR_MAX_RANKS];
    uint64_t seg;        // a whole segment
    uint64_t part;       // the whole units of segment full_segs
    uint32_t full_segs;
    uint32_t rem;        // elements of the partial unit after them (0: none)
    uint32_t parts;      // workgroups per segment
};

// LINE: the units of an iteration start on a line of the memory side.  A
// segment that starts inside a line (5 ranks, say, whose segments are a
// multiple of 16 bytes and no more) would have every wave's 1 KiB of stores
// end in two partial ones, and a line that the last-level cache does not hold
// is fetched for the rest.  So the first iteration begins that much earlier,
// at the line's start, where its first lanes have nothing to do (cold buffers,
// fp32: AllGather, 5 ranks, 8 MiB 15.9 -> 11.1 us; AllReduce, 5 ranks, 8 MiB
// 20.5 -> 17.3, 128 MiB 271 -> 246).  A build of its own, since its few scalar
// operations more cost segments that do start on lines up to 5 %.
constexpr uint32_t kLineBytes = 128;

// Units per thread and iteration for each that the plan asks for (its
// direct_unroll, 1 or 2): eight ranks have eight loads per unit in flight,
// fewer ranks and AllGather, which reads one rank per unit, correspondingly
// less, so they take more units (2 ranks, 48 MiB, bf16, the table's geometry:
// 72 us with one and two, 35 us with two and four).
constexpr int units_per_unroll(int n, int coll) { return coll == AR_COLL_ALLGATHER ? 4 : n <= 4 ? 2 : 1; }

// KEEP: the outputs fit the last-level cache (outputs_fit_cache).
// LOOP: a thread has more than one iteration.  Without it the kernel is
// straight-line code (8 ranks, 4 KiB and 256 KiB, fp32: 2.1 and 2.6 us
// against 2.2 and 2.75 us).
// kMaxDirectWaves: 256 registers per lane hold a thread's loads and the next
// ones' without spills.
template <int DT, int N, int COLL, int U, bool LOOP, bool KEEP, bool LINE>
__global__ __launch_bounds__(64 * kMaxDirectWaves) void direct_kernel(DirectArgs a)
{
    constexpr uint32_t E = Elem<DT>::E, A = Elem<DT>::A;
    constexpr int kOut = KEEP ? kKeepPol : kOutPol;
    constexpr int NSRC = COLL == AR_COLL_ALLGATHER ? 1 : N;      // chain length
    constexpr int NDST = COLL == AR_COLL_REDUCESCATTER ? 1 : N;  // ranks written
    const uint32_t s = blockIdx.x % N;
    const uint32_t nth = blockDim.x, tid = threadIdx.x;
    const bool tail = COLL == AR_COLL_ALLREDUCE && blockIdx.x == a.parts * N;  // see below
    const uint32_t seg = tail ? a.full_segs : s;
    // Rank j of the chain, and the place of the segment in its buffers.
    // AllGather reads, and ReduceScatter writes, one block-sized buffer.
    const uint32_t first = COLL == AR_COLL_REDUCESCATTER ? s + 1 : seg;
    auto src_of = [&](int j) {
        const uint32_t r = first + j;
        return a.src[r >= N ? r - N : r] + (COLL == AR_COLL_ALLGATHER ? 0 : seg * a.seg);
    };
    auto dst_of = [&](int j) {
        return a.dst[COLL == AR_COLL_REDUCESCATTER ? s : j] + (COLL == AR_COLL_REDUCESCATTER ? 0 : seg * a.seg);
    };

    if (tail) {
        // The partial unit at the end of the data: a workgroup of its own,
        // one lane per element, so that no thread does it on top of its
        // units, one round trip to memory later.
        const bool ok = tid < a.rem;
        float x[N];
#pragma unroll
        for (int j = 0; j < NSRC; ++j) {
            const Rsrc w = make_rsrc(src_of(j) + a.part, (uint64_t)a.rem * E);
            x[j] = as_f32(E == 4 ? ld32<kInPol>(w, in_range(ok, tid * E)) : ld16<kInPol>(w, in_range(ok, tid * E)) << 16);
        }
        float acc = x[0];
#pragma unroll
        for (int j = 1; j < NSRC; ++j) acc += x[j];
        const uint32_t y = E == 4 ? as_u32(acc) : bf16_rne(acc);
#pragma unroll
        for (int j = 0; j < NDST; ++j) {
            const Rsrc w = make_rsrc(dst_of(j) + a.part, (uint64_t)a.rem * E);
            if (E == 4) st32<kOut>(w, in_range(ok, tid * E), y);
            else st16<kOut>(w, in_range(ok, tid * E), y);
        }
        return;
    }

    const uint64_t n = s < a.full_segs ? a.seg : s == a.full_segs ? a.part : 0;
    const uint32_t span = nth * U * 16;
    const uint64_t step = (uint64_t)a.parts * span;
    // An iteration's bytes of the segment start at off; those of the first one
    // of all lack the `skip` bytes between the line's start and the segment's.
    const uint32_t lead = LINE ? (uint32_t)(uintptr_t)dst_of(0) & (kLineBytes - 1) : 0;
    uint64_t off = (uint64_t)(blockIdx.x / N) * span;
    uint32_t skip = LINE && off == 0 ? lead : 0;
    if (LINE && off != 0) off -= lead;
    if (off >= n) return;
    u32x4 v[U][NSRC];
    // Descriptors cover this iteration's bytes; their range check drops the
    // lanes past the end, and those before the segment use an offset outside.
    auto span_bytes = [&](uint64_t o, uint32_t skip) {
        return o >= n ? 0u : n - o < span - skip ? (uint32_t)(n - o) : span - skip;
    };
    auto lane_off = [&](int t, uint32_t skip) {
        return LINE && t == 0 ? in_range(tid * 16 >= skip, tid * 16 - skip) : (t * nth + tid) * 16 - skip;
    };
    auto load = [&](uint64_t o, uint32_t skip) {
        const uint32_t b = span_bytes(o, skip);
#pragma unroll
        for (int j = 0; j < NSRC; ++j) {
            const Rsrc w = make_rsrc(src_of(j) + o, b);
#pragma unroll
            for (int t = 0; t < U; ++t) v[t][j] = ld128<kInPol>(w, lane_off(t, skip));
        }
    };
    auto arrive = [&]() {
#pragma unroll
        for (int t = 0; t < U; ++t)
#pragma unroll
            for (int j = 0; j < NSRC; ++j) asm volatile("" : "+v"(v[t][j]));
    };
    load(off, skip);
    if (LOOP) arrive();
    while (true) {
        u32x4 y[U];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            if (COLL == AR_COLL_ALLGATHER) {
                y[t] = v[t][0];  // a copy keeps every bit, NaN payloads included
            } else if (E == 4) {
                y[t] = v[t][0];
#pragma unroll
                for (int j = 1; j < NSRC; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) y[t][i] = as_u32(as_f32(y[t][i]) + as_f32(v[t][j][i]));
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float lo = bf16_lo(v[t][0][i]), hi = bf16_hi(v[t][0][i]);
#pragma unroll
                    for (int j = 1; j < NSRC; ++j) {
                        lo = lo + bf16_lo(v[t][j][i]);
                        hi = hi + bf16_hi(v[t][j][i]);
                    }
                    y[t][i] = pack_bf16(lo, hi);
                }
            }
        }
        const uint32_t b = span_bytes(off, skip);
        const uint64_t next = off + step - skip;
        const bool more = LOOP && next < n;
        // The next units' loads go out before these units' stores: loads
        // and stores retire in order, so loads issued after the stores could
        // only be waited for together with them.  That is what eight ranks'
        // pairs of fp32 units are better with once the outputs are streamed
        // to HBM: sixteen loads, then sixteen stores (AllReduce, 32 workgroups
        // of two waves per segment, mean of three buffer layouts, repeated and
        // cold, loads first and stores first: 32 MiB 93.8 and 92.5 us, 64 MiB
        // 185.8 and 183.2, 128 MiB 389 and 381; but bf16, 64 workgroups of one
        // wave, 96 MiB 286 and 296).
        constexpr bool kLoadsFirst = !(DT == AR_FLOAT32 && N == 8 && U == 2 && COLL == AR_COLL_ALLREDUCE && !KEEP);
        if (kLoadsFirst && more) load(next, 0);
#pragma unroll
        for (int j = 0; j < NDST; ++j) {
            const Rsrc w = make_rsrc(dst_of(j) + off, b);
#pragma unroll
            for (int t = 0; t < U; ++t) st128<kOut>(w, lane_off(t, skip), y[t]);
        }
        if (!more) return;
        if (!kLoadsFirst) load(next, 0);
        arrive();
        off = next;
        skip = 0;
    }
}

typedef void (*DirectFn)(DirectArgs);

// Units per thread and iteration for a plan's direct_unroll, where a thread of
// the plan's workgroups has per_thread 16-byte units of a segment.  Where half
// of a plan's units per iteration already hold an AllReduce's of three or four
// ranks, half: with more, half of the workgroups would have nothing to do
// (AllReduce, 4 ranks, fp32, 64 workgroups of 8 waves per segment, cold
// buffers: 3 MiB 8.8 us with four units, 6.4 with two; 4 MiB 8.9 and 7.2).
// Elsewhere fewer workgroups with more loads each are as fast or faster (2
// ranks, 4 MiB bf16: 3.5 us with four units, 4.5 with two; 8 ranks, 1.5 MiB
// fp32: 5.5 and 5.8; ReduceScatter, 2 ranks, 4 MiB: 2.5 and 2.8).
constexpr int direct_units(int n, int coll, int unroll, uint64_t per_thread)
{
    const int u = units_per_unroll(n, coll);
    if (n > 8 || unroll != 2) return u;
    return coll == AR_COLL_ALLREDUCE && (n == 3 || n == 4) && per_thread <= (uint64_t)u ? u : 2 * u;
}

template <int DT, int COLL, bool KEEP, bool LINE, int N = AR_MAX_RANKS>
__host__ DirectFn direct_fn(int nranks, int units, bool loop)
{
    if constexpr (N >= 2) {
        if (nranks != N) return direct_fn<DT, COLL, KEEP, LINE, N - 1>(nranks, units, loop);
        constexpr int U = units_per_unroll(N, COLL);
        if constexpr (N <= 8) {
            if (units == 2 * U)
                return loop ? direct_kernel<DT, N, COLL, 2 * U, true, KEEP, LINE>
                            : direct_kernel<DT, N, COLL, 2 * U, false, KEEP, LINE>;
        }
        return loop ? direct_kernel<DT, N, COLL, U, true, KEEP, LINE> : direct_kernel<DT, N, COLL, U, false, KEEP, LINE>;
    }
    return nullptr;
}

template <int DT, bool KEEP, bool LINE>
__host__ DirectFn direct_fn_of(int coll, int nranks, int units, bool loop)
{
    switch (coll) {
    case AR_COLL_REDUCESCATTER: return direct_fn<DT, AR_COLL_REDUCESCATTER, KEEP, LINE>(nranks, units, loop);
    case AR_COLL_ALLGATHER: return direct_fn<DT, AR_COLL_ALLGATHER, KEEP, LINE>(nranks, units, loop);
    default: return direct_fn<DT, AR_COLL_ALLREDUCE, KEEP, LINE>(nranks, units, loop);
    }
}

template <int DT>
__host__ DirectFn direct_fn_for(int coll, int nranks, int units, bool loop, bool keep, bool line)
{
    if (line) return keep ? direct_fn_of<DT, true, true>(coll, nranks, units, loop) : direct_fn_of<DT, false, true>(coll, nranks, units, loop);
    return keep ? direct_fn_of<DT, true, false>(coll, nranks, units, loop) : direct_fn_of<DT, false, false>(coll, nranks, units, loop);
}

}  // namespace dev

// Whether a run's iterations are to start on lines: segments that do not,
// outputs of 12 MiB in all (with less the shift gains nothing), and no
// iteration more than without the shift, which also holds where the kernel
// has no loop.  one: units of one iteration of a segment's workgroups.
static bool start_on_lines(const ar_plan_info &info, const RingArgs &args, uint64_t one)
{
    constexpr uint64_t line = dev::kLineBytes;
    const uint64_t e = info.dtype == AR_FLOAT32 ? 4 : 2, seg_b = args.seg * e, units = seg_b / 16;
    bool off_line = info.coll != AR_COLL_REDUCESCATTER && seg_b % line != 0;
    for (int r = 0; r < info.nranks; ++r) off_line |= (uintptr_t)args.dst[r] % line != 0;
    const uint64_t out_b = seg_b * (uint64_t)info.nranks * (info.coll == AR_COLL_REDUCESCATTER ? 1 : (uint64_t)info.nranks);
    return off_line && out_b >= (12ull << 20) && (units + line / 16 - 1 + one - 1) / one == (units + one - 1) / one;
}

int launch_direct(const ar_plan_info &info, const RingArgs &args, void *stream)
{
    const bool f32 = info.dtype == AR_FLOAT32;
    const uint64_t e = f32 ? 4 : 2;
    // The plan's geometry is at most direct_max_parts per segment, so that
    // these counts and the grid below fit 32 bits.
    const uint32_t threads = direct_threads(info.nwaves);
    const uint32_t parts = (uint32_t)info.nchannels * direct_split(info.nwaves);
    const uint64_t all = (uint64_t)parts * threads, seg_units = args.seg * e / 16;
    const uint64_t per_thread = (seg_units + all - 1) / all;
    const int units = dev::direct_units(info.nranks, info.coll, info.direct_unroll, per_thread);
    const dev::DirectFn fn = (f32 ? dev::direct_fn_for<AR_FLOAT32> : dev::direct_fn_for<AR_BFLOAT16>)(
        info.coll, info.nranks, units, per_thread > (uint64_t)units, outputs_fit_cache(info),
        start_on_lines(info, args, all * units));
    if (!fn) return AR_ERR_UNSUPPORTED;
    dev::DirectArgs a;
    for (int r = 0; r < AR_MAX_RANKS; ++r) {
        a.src[r] = args.src[r];
        a.dst[r] = args.dst[r];
    }
    a.seg = args.seg * e;
    a.part = args.part * e / 16 * 16;
    a.full_segs = args.full_segs;
    a.rem = (uint32_t)(args.part % (16 / e));
    a.parts = parts;
    void *kargs[] = {&a};
    return hipLaunchKernel((const void *)fn, dim3(parts * (unsigned)info.nranks + (a.rem ? 1u : 0u)),
                           dim3(threads), kargs, 0, (hipStream_t)stream) == hipSuccess ? AR_OK : AR_ERR_HIP;
}

}  // namespace ar
