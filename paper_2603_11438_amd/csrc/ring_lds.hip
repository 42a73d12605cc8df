// The ring with its links in LDS (gfx950).
//
// One workgroup holds one whole ring: wave r is rank r, and the link
// r -> r+1 is a pair of slots in the workgroup's LDS.  A plan's C * N
// workgroups of W waves become up to C * N * W / 2 such rings, R of them; ring
// q takes the pieces q, q + R, ... of every segment, so that neighbouring
// workgroups touch neighbouring memory.  The schedule is the ring's of
// ar_kernels.hip (segment s is summed along the chain x_s + x_{s+1} + ... +
// x_{s+N-1} while it travels round the reduce-scatter, the last rank of the
// chain finishes it, and it travels round once more), with the same
// additions in the same order, so the bits are those of every other path.
//
// A reduce-scatter step writes its message to the own outgoing slot and reads
// the next one's from the incoming link.  One workgroup barrier per step
// stands for what the protocols' flags and counters do for links in memory:
// it publishes the step's messages, and, since a link alternates between two
// slots, it frees the slots of the step before.  No wave waits for another
// workgroup, so nothing has to be resident together, and a run keeps no
// state: no epochs, no FIFOs, no watchdog.
//
// What bounds it.  Large messages: HBM.  Partials and forwarded values stay
// in LDS, so each input is read once and each output written once, the
// 2 N S bytes no AllReduce can do without, where the Simple ring through
// memory moves 34 S and LL128 44 S (8 ranks, fp32).  As soon as a step has
// used its input, the load for the same step of the next piece goes out into
// the same registers, so HBM latency passes during the steps.  Small
// messages: launch, one load, N LDS hops, one store.
#include "ar_device.h"

namespace ar {
namespace dev {

// Order this wave's LDS accesses around a workgroup barrier without waiting
// for its global loads and stores: the fences name the local address space
// alone, so loads for the next piece and stores of the last one stay in
// flight across the steps.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// N ranks.  A lane moves U units of 16 bytes per segment and piece.  One unit
// is the fastest from 3 ranks up: two halve the number of pieces, and a small
// message then keeps fewer compute units busy (8 ranks, fp32, device time:
// 4 KiB 3.7 against 4.8 us, 1 MiB 5.5 against 7.4 us, 128 MiB 382 against
// 393-414 us).  With two ranks a wave would have only 2 KiB of loads in
// flight (48 MiB, bf16: 37 us with two units, 2.8 us at 64 KiB).  AllGather
// reads one segment per piece and takes twice as many (8 ranks, 12 MiB per
// rank, fp32: 20.3 us with two units, 21.9 with one).
template <int N, int COLL>
struct LdsShape {
    static constexpr int U = (N == 2 ? 2 : 1) * (COLL == AR_COLL_ALLGATHER ? 2 : 1);
    // Beyond 12 ranks the waves of a workgroup have 128 registers each, too
    // few to hold the next piece's inputs across the gather: spilling them
    // took 16 ranks from 11 to 13 us at 64 KiB.
    static constexpr bool kPrefetch = N <= 12 || COLL == AR_COLL_ALLGATHER;
    static constexpr uint32_t kPieceBytes = 64 * U * 16;
};

// KEEP: the outputs fit the last-level cache (outputs_fit_cache).
template <int DT, int N, int COLL, bool KEEP>
__global__ __launch_bounds__(64 * N) void lds_ring_kernel(RingArgs a)
{
    constexpr int U = LdsShape<N, COLL>::U;
    constexpr uint32_t PB = LdsShape<N, COLL>::kPieceBytes;
    constexpr uint32_t E = Elem<DT>::E, A = Elem<DT>::A;
    constexpr int kOut = KEEP ? kKeepPol : kOutPol;
    constexpr bool kReduce = COLL != AR_COLL_ALLGATHER;
    constexpr int IN = kReduce ? N : 1;            // segments read per piece
    constexpr int PV = kReduce ? (int)A / 4 : 1;   // 16-byte vectors of a unit on the link
    __shared__ u32x4 slots[2][N][PV * U * 64];

    const uint32_t rank = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane = lane_id();
    const uint32_t prev = rank == 0 ? N - 1 : rank - 1;
    const char *const src = a.src[rank];
    char *const dst = a.dst[rank];
    // Bytes of a whole segment, and of the whole units of the partial one.
    const uint64_t full_b = a.seg * E, part_b = a.part / A * 16;
    const uint32_t rem = (uint32_t)(a.part % A);  // elements of the partial unit (0: none)

    // Segment of chain step k, and of all-gather step i: the owner of segment
    // s is rank s - 1.  `r` is the rank as a value the compiler cannot hoist
    // from: the addresses and sizes of 2 N segments held across the loop
    // would not fit the scalar registers.
    uint32_t r = rank;
    auto back = [&](uint32_t k) { return r >= k ? r - k : r + N - k; };  // k <= N
    auto chain_seg = [&](uint32_t k) {
        return COLL == AR_COLL_REDUCESCATTER ? back(k + 1) : COLL == AR_COLL_ALLREDUCE ? back(k) : r;
    };
    auto gather_seg = [&](uint32_t i) {
        const uint32_t s = back(i) + (COLL == AR_COLL_ALLREDUCE ? 1 : 0);
        return s >= N ? s - N : s;
    };
    // Bytes of the piece at `off` that exist in a segment of n bytes; and a
    // descriptor of segment s's piece (full / part: those bytes for a whole
    // and for the partial segment), whose range check drops the rest.
    auto piece_bytes = [&](uint64_t n, uint64_t off) { return off >= n ? 0u : n - off < PB ? (uint32_t)(n - off) : PB; };
    auto window = [&](const char *base, uint32_t s, uint32_t full, uint32_t part) {
        return make_rsrc(base, s < a.full_segs ? full : s == a.full_segs ? part : 0u);
    };
    auto load = [&](u32x4 (&in)[U], int k, uint64_t off, uint32_t full, uint32_t part) {
        const uint32_t s = chain_seg(k);  // AllGather reads one block-sized buffer
        const Rsrc w = window(src + off + (COLL == AR_COLL_ALLGATHER ? 0 : s * full_b), s, full, part);
#pragma unroll
        for (int t = 0; t < U; ++t) in[t] = ld128<kInPol>(w, (64 * t + lane) * 16);
    };
    auto store = [&](const u32x4 (&y)[U], uint32_t s, uint64_t off, uint32_t full, uint32_t part) {
        // ReduceScatter writes one block-sized buffer.
        const Rsrc w = window(dst + off + (COLL == AR_COLL_REDUCESCATTER ? 0 : s * full_b), s, full, part);
#pragma unroll
        for (int t = 0; t < U; ++t) st128<kOut>(w, (64 * t + lane) * 16, y[t]);
    };
    // Inputs are waited for in one place, where only stores have been issued
    // after them: loads and stores retire in order, so the compiler, which
    // has one count for all ways to reach an instruction, would elsewhere
    // make the steps wait for the last piece's stores too.
    auto arrive = [&](u32x4 (&in)[IN][U]) {
#pragma unroll
        for (int k = 0; k < IN; ++k)
#pragma unroll
            for (int t = 0; t < U; ++t) asm volatile("" : "+v"(in[k][t]));
    };
    uint32_t slot = 0;  // slot of the next message, on every link
    auto widen = [&](const u32x4 &x, u32x4 *f) {  // a unit in the data type -> PV vectors of fp32
        if (E == 4) {
            f[0] = x;
        } else {
            f[0] = u32x4{x[0] << 16, x[0] & 0xFFFF0000u, x[1] << 16, x[1] & 0xFFFF0000u};
            f[PV - 1] = u32x4{x[2] << 16, x[2] & 0xFFFF0000u, x[3] << 16, x[3] & 0xFFFF0000u};
        }
    };

    // The partial unit at the end of the data (AllReduce only): its piece,
    // and its place in that piece.
    const uint64_t rem_off = part_b / PB * PB;
    const uint32_t rem_t = (uint32_t)(part_b - rem_off) / 1024, rem_lane = (uint32_t)(part_b - rem_off) / 16 & 63u;

    const uint64_t step = (uint64_t)gridDim.x * PB;
    uint64_t off = (uint64_t)blockIdx.x * PB;
    uint32_t full = piece_bytes(full_b, off), part = piece_bytes(part_b, off);
    u32x4 in[IN][U];
    constexpr bool kPrefetch = LdsShape<N, COLL>::kPrefetch;
    if (kPrefetch) {
#pragma unroll
        for (int k = 0; k < IN; ++k) load(in[k], k, off, full, part);
        arrive(in);
    }
    while (off < full_b) {
        asm volatile("" : "+s"(r));
        if (!kPrefetch) {
#pragma unroll
            for (int k = 0; k < IN; ++k) load(in[k], k, off, full, part);
        }
        const uint64_t off2 = off + step;  // the next piece
        const uint32_t full2 = piece_bytes(full_b, off2), part2 = piece_bytes(part_b, off2);
        const bool has_rem = COLL == AR_COLL_ALLREDUCE && rem != 0 && off == rem_off;
        u32x4 rem_y = {0, 0, 0, 0};
        if (has_rem) {
            // The rank's elements of the partial unit, into their lane.
            const Rsrc w = make_rsrc(src + a.full_segs * full_b + part_b, (uint64_t)rem * E);
            u32x4 v = {0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < (int)A; ++i) {
                const uint32_t o = in_range((uint32_t)i < rem, i * E);
                if (E == 4) v[i] = ld32<kInPol>(w, o);
                else v[i >> 1] |= ld16<kInPol>(w, o) << ((i & 1) * 16);
            }
#pragma unroll
            for (int k = 0; k < IN; ++k)
#pragma unroll
                for (int t = 0; t < U; ++t)
                    if (chain_seg(k) == a.full_segs && (uint32_t)t == rem_t && lane == rem_lane) in[k][t] = v;
        }

        u32x4 y[U];
        if constexpr (kReduce) {
            // A message: PV vectors per unit, vector v of every unit before
            // vector v + 1 of any, so that each LDS instruction covers
            // contiguous bytes.
            u32x4 m[PV * U];
#pragma unroll
            for (int k = 0; k < N; ++k) {
                if (k > 0) {
#pragma unroll
                    for (int i = 0; i < PV * U; ++i) m[i] = slots[slot ^ 1][prev][64 * i + lane];
                }
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    u32x4 f[PV];
                    widen(in[k][t], f);
#pragma unroll
                    for (int v = 0; v < PV; ++v)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            m[v * U + t][i] = k == 0 ? f[v][i] : as_u32(as_f32(m[v * U + t][i]) + as_f32(f[v][i]));
                }
                if (kPrefetch) load(in[k], k, off2, full2, part2);
                if (k < N - 1) {
#pragma unroll
                    for (int i = 0; i < PV * U; ++i) slots[slot][rank][64 * i + lane] = m[i];
                    lds_barrier();
                    slot ^= 1;
                }
            }
            // The end of the chain: rounded once.
#pragma unroll
            for (int t = 0; t < U; ++t) {
                if (E == 4) {
                    y[t] = m[t];
                } else {
                    const u32x4 &lo = m[t], &hi = m[(PV - 1) * U + t];
                    y[t] = u32x4{pack_bf16(as_f32(lo[0]), as_f32(lo[1])), pack_bf16(as_f32(lo[2]), as_f32(lo[3])),
                                 pack_bf16(as_f32(hi[0]), as_f32(hi[1])), pack_bf16(as_f32(hi[2]), as_f32(hi[3]))};
                }
            }
        } else {
#pragma unroll
            for (int t = 0; t < U; ++t) y[t] = in[0][t];
            load(in[0], 0, off2, full2, part2);
        }
        if constexpr (COLL == AR_COLL_REDUCESCATTER) {
            store(y, r, off, full, part);
        } else {
            // The all-gather forwards without copying: a finished message
            // stays in the slot its first rank wrote, and step i reads it
            // there, i ranks further on.
#pragma unroll
            for (int t = 0; t < U; ++t) slots[slot][rank][64 * t + lane] = y[t];
            lds_barrier();
            slot ^= 1;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if (i > 0) {
                    const uint32_t q = back(i);
#pragma unroll
                    for (int t = 0; t < U; ++t) y[t] = slots[slot ^ 1][q][64 * t + lane];
                }
                // With many ranks, four steps' slots at a time: all of them
                // read ahead would not fit the registers.
                if (N > 8 && i % 4 == 0) __builtin_amdgcn_sched_barrier(0);
                const uint32_t s = gather_seg(i);
                store(y, s, off, full, part);
                if (has_rem && s == a.full_segs) {
#pragma unroll
                    for (int t = 0; t < U; ++t)
                        if ((uint32_t)t == rem_t) rem_y = y[t];
                }
            }
        }
        if (has_rem) {
            const Rsrc w = make_rsrc(dst + a.full_segs * full_b + part_b, (uint64_t)rem * E);
#pragma unroll
            for (int i = 0; i < (int)A; ++i) {
                const uint32_t o = in_range((uint32_t)i < rem && lane == rem_lane, i * E);
                if (E == 4) st32<kOut>(w, o, rem_y[i]);
                else st16<kOut>(w, o, (rem_y[i >> 1] >> ((i & 1) * 16)) & 0xFFFFu);
            }
        }
        if (kPrefetch) arrive(in);
        off = off2;
        full = full2;
        part = part2;
    }
}

typedef void (*RingFn)(RingArgs);

template <int DT, int COLL, bool KEEP, int N = AR_MAX_RANKS>
__host__ RingFn lds_fn(int nranks, uint32_t *piece)
{
    if constexpr (N >= 2) {
        if (nranks != N) return lds_fn<DT, COLL, KEEP, N - 1>(nranks, piece);
        *piece = LdsShape<N, COLL>::kPieceBytes;
        return lds_ring_kernel<DT, N, COLL, KEEP>;
    }
    return nullptr;
}

template <int DT, bool KEEP>
__host__ RingFn lds_fn_of(int coll, int nranks, uint32_t *piece)
{
    switch (coll) {
    case AR_COLL_REDUCESCATTER: return lds_fn<DT, AR_COLL_REDUCESCATTER, KEEP>(nranks, piece);
    case AR_COLL_ALLGATHER: return lds_fn<DT, AR_COLL_ALLGATHER, KEEP>(nranks, piece);
    default: return lds_fn<DT, AR_COLL_ALLREDUCE, KEEP>(nranks, piece);
    }
}

}  // namespace dev

int launch_ring_lds(const ar_plan_info &info, const RingArgs &args, void *stream)
{
    uint32_t piece = 0;
    const bool f32 = info.dtype == AR_FLOAT32, keep = outputs_fit_cache(info);
    const auto pick = f32 ? (keep ? dev::lds_fn_of<AR_FLOAT32, true> : dev::lds_fn_of<AR_FLOAT32, false>)
                          : (keep ? dev::lds_fn_of<AR_BFLOAT16, true> : dev::lds_fn_of<AR_BFLOAT16, false>);
    const dev::RingFn fn = pick(info.coll, info.nranks, &piece);
    if (!fn) return AR_ERR_UNSUPPORTED;
    const uint64_t grid = ring_lds_workgroups(info, args.seg * (f32 ? 4 : 2), piece);
    RingArgs a = args;
    void *kargs[] = {&a};
    return hipLaunchKernel((const void *)fn, dim3((unsigned)grid), dim3(64u * (unsigned)info.nranks), kargs, 0,
                           (hipStream_t)stream) == hipSuccess ? AR_OK : AR_ERR_HIP;
}

}  // namespace ar
