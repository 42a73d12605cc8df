// Device helpers shared by the kernels of libar (gfx950): buffer accesses with
// a cache policy, wave-uniform values, and the fp32 / bf16 conversions.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ar_internal.h"

namespace ar {
namespace dev {

typedef uint32_t u32x4 __attribute__((__vector_size__(16)));
typedef uint32_t u32x2 __attribute__((__vector_size__(8)));
typedef __amdgpu_buffer_rsrc_t Rsrc;

// Cache-policy operand of gfx950 buffer instructions.
enum : int { kPolPlain = 0, kPolSc0 = 1, kPolNt = 2, kPolSc1 = 16 };
// The policies are fixed, not build options.  A FIFO line (or, in the
// peer-direct mode, an output element) is written on one XCD and read on
// another, behind a different L2; without the device-scope bit on both the
// write and the read, a reader can be served a stale copy and the ring
// returns wrong sums or waits until the watchdog fires.
constexpr int kFifoLd = kPolSc1;  // device-coherent FIFO reads
constexpr int kFifoSt = kPolSc1;  // device-coherent FIFO writes
constexpr int kInPol = kPolNt;    // rank inputs: read once, streamed
constexpr int kOutPol = kPolNt;   // rank outputs: written once, streamed
constexpr int kKeepPol = kPolSc1; // rank outputs that the last-level cache holds (outputs_fit_cache)
static_assert((kFifoLd & kPolSc1) != 0 && (kFifoSt & kPolSc1) != 0, "FIFO accesses must be device-coherent");

template <int DT> struct Elem;
template <> struct Elem<AR_FLOAT32> { static constexpr uint32_t E = 4, A = 4; };
template <> struct Elem<AR_BFLOAT16> { static constexpr uint32_t E = 2, A = 8; };

__device__ __forceinline__ Rsrc make_rsrc(const void *p, uint64_t bytes)
{
    // Word 3 = 0x00020000: raw 32-bit dword format, as on the rest of CDNA.
    uint32_t n = bytes > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)n, 0x00020000);
}

template <int POL> __device__ __forceinline__ u32x4 ld128(Rsrc r, uint32_t off)
{
    return __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, POL);
}
template <int POL> __device__ __forceinline__ u32x2 ld64(Rsrc r, uint32_t off)
{
    return __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, POL);
}
template <int POL> __device__ __forceinline__ uint32_t ld32(Rsrc r, uint32_t off)
{
    return __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, POL);
}
template <int POL> __device__ __forceinline__ uint32_t ld16(Rsrc r, uint32_t off)
{
    return (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, POL);
}
template <int POL> __device__ __forceinline__ void st128(Rsrc r, uint32_t off, u32x4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)off, 0, POL);
}
template <int POL> __device__ __forceinline__ void st64(Rsrc r, uint32_t off, u32x2 v)
{
    __builtin_amdgcn_raw_buffer_store_b64(v, r, (int)off, 0, POL);
}
template <int POL> __device__ __forceinline__ void st32(Rsrc r, uint32_t off, uint32_t v)
{
    __builtin_amdgcn_raw_buffer_store_b32(v, r, (int)off, 0, POL);
}
template <int POL> __device__ __forceinline__ void st16(Rsrc r, uint32_t off, uint32_t v)
{
    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)v, r, (int)off, 0, POL);
}

// A buffer offset outside every resource built by the ring steps (each covers
// at most one step's data or one FIFO slot, far below 2^31 bytes): a load
// there returns zeros and a store there is dropped, by the hardware's range
// check.  Lanes past the end of a message use it instead of a branch, which
// keeps a batch of accesses straight-line code; the compiler can then wait
// for exactly the loads an instruction needs instead of for every
// outstanding access (a branch around each access makes it wait for all of
// them, earlier stores included, before each store).
constexpr uint32_t kOobOff = 0x80000000u;
__device__ __forceinline__ uint32_t in_range(bool ok, uint32_t off) { return ok ? off : kOobOff; }

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63u; }

// True on every lane when p holds on any active lane; the result is a
// wave-uniform value the compiler knows to be uniform.
//
// Uniformity matters throughout the ring steps: a branch on the lane (such as
// "lane 0 stores the flag") whose join merges any value makes the compiler
// treat everything that depends on it as per-lane.  The step loop then runs
// under an execution mask, loop-carried counters and pointers move into
// vector registers, and every buffer access is wrapped in a loop that reads
// its descriptor lane by lane.  So flags are stored by every lane (the same
// value to the same address: one write), and partial units and groups use
// out-of-range offsets instead of lane branches.
__device__ __forceinline__ bool any_lane(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }

// The lane index as a value the compiler may not hoist out of the step loop:
// a step's per-lane offsets are then recomputed each step (a few ALU ops)
// instead of being held in registers across every step of the kernel.
__device__ __forceinline__ uint32_t step_lane()
{
    uint32_t l = lane_id();
    asm volatile("" : "+v"(l));
    return l;
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// ---- fp32 / bf16 ------------------------------------------------------------

__device__ __forceinline__ float as_f32(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint32_t as_u32(float f) { return __builtin_bit_cast(uint32_t, f); }

// bf16 -> fp32 is exact: the bf16 bits are the top half of the fp32 word.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return as_f32(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return as_f32(w & 0xFFFF0000u); }

// fp32 -> bf16, round to nearest even; NaN -> quiet NaN 0x7FC0.
__device__ __forceinline__ uint32_t bf16_rne(float f)
{
    uint32_t u = as_u32(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    return bf16_rne(lo) | (bf16_rne(hi) << 16);
}

}  // namespace dev
}  // namespace ar
