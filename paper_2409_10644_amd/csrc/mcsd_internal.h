// Internal declarations shared by the library's translation units (not part of the public ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include "mcsd.h"

struct mcsd_mask {
    int32_t gamma_max;
    int32_t n_nodes_max;
    int32_t words_per_row;
    int32_t device;
    int32_t branching[MCSD_MAX_LEVELS];
    int32_t level_off[MCSD_MAX_LEVELS + 1];
    uint64_t *bits_host;
    int32_t *parent_host;
    int32_t *level_host;
    void *dev_block;       // one device allocation: bits, then parent
    uint64_t *bits_dev;
    int32_t *parent_dev;
};

// Tree shape passed to kernels by value.
struct McsdTreeDesc {
    int32_t gamma;
    int32_t b[MCSD_MAX_LEVELS];
    int32_t off[MCSD_MAX_LEVELS + 1];
};

static inline int mcsd_hip_status(hipError_t e) { return e == hipSuccess ? MCSD_OK : MCSD_EHIP; }

// Accelerator dies (each with its own L2) of `device` when the hardware deals workgroup i of a launch to die
// i % dies, as established by a probe launch in mcsd_build_mask; 0 when unknown or not so.  Defined in mask.cpp.
int mcsd_xcc_count(int device);

// One-shot profiling events per kernel (see mcsd_profile_next); defined in mask.cpp.  Arming stores `stop` and then
// `start`; a launch takes `start` with an atomic exchange, so exactly one launch consumes an armed pair even when
// several host threads launch the same kernel at once.
#include <atomic>
struct McsdProfileSlot { std::atomic<hipEvent_t> start, stop; };
extern McsdProfileSlot g_mcsd_profile[6];

// Launch `kernel` on `st`; if a profiling pair is armed for `which`, bracket the launch with it and disarm.
template <typename... Args, typename... Actual>
inline void mcsd_launch(int which, void (*kernel)(Args...), dim3 grid, dim3 block, hipStream_t st, Actual... args)
{
    McsdProfileSlot &slot = g_mcsd_profile[which];
    hipEvent_t start = slot.start.load(std::memory_order_relaxed);
    if (start) start = slot.start.exchange(nullptr, std::memory_order_acquire);
    if (start) {
        hipEvent_t stop = slot.stop.exchange(nullptr, std::memory_order_relaxed);
        hipExtLaunchKernelGGL(kernel, grid, block, 0, st, start, stop, 0, args...);
    } else {
        hipLaunchKernelGGL(kernel, grid, block, 0, st, args...);
    }
}

// 16 bytes per lane from global memory straight into LDS: lane l reads gbase + voff and lands at lds_base + 16*l
// (gbase and lds_base uniform).  Written as assembly on purpose: the compiler knows nothing about where such a
// load writes in LDS unless alias information happens to survive inlining, and otherwise makes the next LDS
// read wait for it (vmcnt(0)), which serialises the stream with the compute.  Here it is just an opaque
// instruction; the kernel waits for it itself (MCSD_WAIT_VMCNT + barrier) before anyone reads the stage.
// An untracked load can only make compiler-placed vmcnt waits longer, never shorter (loads retire in order).
// M0 carries the LDS address; nothing else in these kernels uses M0 (the toolchain rejects it as a clobber).
// NT marks the load non-temporal, for prefix K/V that exactly one workgroup reads: keeping a read-once stream out
// of the caches' retained set is worth 5-12 % of the sweep (measured; the coherence-scope bits make no
// difference).  Where several workgroups share a stream (grouped-query heads cut into several query chunks) the
// second reader needs the lines in L2 and the plain load is the faster one.
template <bool NT>
static __device__ inline void load_to_lds16(const void *gbase, uint32_t voff, void *lds_base)
{
    const uint32_t lds_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds_base;
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     :
                     : "s"(lds_addr), "v"(voff), "s"(gbase)
                     : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(lds_addr), "v"(voff), "s"(gbase)
                     : "memory");
}

// The same with an address of its own for every lane.
static __device__ inline void load_to_lds16_at(const void *src, void *lds_base)
{
    const uint32_t lds_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds_base;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_addr), "v"(src) : "memory");
}

// 4 bytes per lane, at an address of its own: lane l lands at lds_base + 4*l.
static __device__ inline void load_to_lds4_at(const void *src, void *lds_base)
{
    const uint32_t lds_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds_base;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" : : "s"(lds_addr), "v"(src) : "memory");
}

// s_waitcnt vmcnt(N) only (expcnt / lgkmcnt left at their maxima)
#define MCSD_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(((N) & 15) | (7 << 4) | (15 << 8) | (((N) >> 4) << 14))
