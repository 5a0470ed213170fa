// fq_kernels.hpp -- the merge, spawn and resident kernel templates of the FCIQMC step.
//
// Their instantiations (address words W, model variant, workgroup size,
// compression style) are compiled in separate translation units, one per
// (W, model variant) pair (fq_inst.hip built with FQ_INST_W and
// FQ_INST_MODEL), so that they build in parallel; the host runtime declares
// them with FQ_EXTERN_STEP_KERNELS and launches them through their handles.
#pragma once
#include "fq_resident.hpp"
#include "fq_step.hpp"

// The step kernels run over a set of instances: one, or a batch.  `insts` is
// a device array of instance descriptors.  A merge or spawn workgroup finds
// its instance and bucket through `map` (entry = instance << 15 | bucket);
// without a map there is one instance and workgroup b takes bucket b.

__device__ __forceinline__ const fq::Inst &locate(const fq::Inst *const *insts, const fq::u32 *map, int &b)
{
    if (map) {
        const fq::u32 m = map[blockIdx.x];
        b = (int)(m & 0x7fffu);
        return fq::const_inst(insts[m >> 15]);
    }
    b = (int)blockIdx.x;
    return fq::const_inst(insts[0]);
}

// EARLY: early compression (separate kernels, so the late-compression
// kernels carry none of its code and registers)
template <int W, int MODEL, int BS, bool EARLY>
__global__ __launch_bounds__(BS) void k_merge(const fq::Inst *const *insts, const fq::u32 *map)
{
    extern __shared__ __align__(16) char smem[];
    int b;
    const fq::Inst &I = locate(insts, map, b);
    fq::merge_bucket<W, MODEL, BS, EARLY>(I, b, smem);
}

// waves per SIMD the spawn kernel's register budget must allow (1: no
// constraint beyond the workgroup size)
#ifndef FQ_SPAWN_WAVES
#define FQ_SPAWN_WAVES 1
#endif
template <int W, int MODEL, int BS, bool EARLY>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(FQ_SPAWN_WAVES))) void k_spawn(const fq::Inst *const *insts, const fq::u32 *map, int mode)
{
    extern __shared__ __align__(16) char smem[];
    int b;
    const fq::Inst &I = locate(insts, map, b);
    fq::spawn_bucket<W, MODEL, BS, EARLY>(I, b, mode, smem);
}

// Resident steps, 2^lg_grid workgroups of the grid for
// each.  Up to 32 (the CUs of an XCD) they are placed on XCD i mod 8 for
// instance i: workgroup 8 ((i / 8) 2^lg_grid + g) + i mod 8 of the grid is
// its workgroup g.  Above, workgroup i 2^lg_grid + g is.  An instance takes
// as many of them as it has buckets, and enough that none owns more than
// RES_MAXK.  stop[i]: the step at which instance i ends this launch.
struct ResStops {
    fq::i64 step[fq::RES_MAXG];
};
__host__ __device__ __forceinline__ int res_log2_groups(int lg, int log2B)
{
    const int least = log2B - 6;  // RES_MAXK = 2^6
    return lg < least ? least : lg > log2B ? log2B : lg;
}
template <int W, int MODEL, bool EARLY>
__global__ __launch_bounds__(fq::RES_BS) void k_resident(const fq::Inst *const *insts, int n, int lg, int lg_grid,
                                                         fq::i64 max_items, fq::u64 patience, ResStops stops)
{
    extern __shared__ __align__(16) char smem[];
    const int x = (int)blockIdx.x, y = lg_grid <= 5 ? x >> 3 : x;
    const int g = y & ((1 << lg_grid) - 1), i = lg_grid <= 5 ? ((y >> lg_grid) << 3) | (x & 7) : y >> lg_grid;
    if (i >= n) return;
    const fq::Inst &I = fq::const_inst(insts[i]);
    const int own = res_log2_groups(lg, I.log2B);
    if (g >> own) return;
    fq::resident_steps<W, MODEL, EARLY, 0>(I, g, own, stops.step[i], max_items << own, patience, fq::Overlap{}, 0, nullptr,
                                           smem);
}

// The same for replicas and their overlaps (KIND 1), or two runs for excited
// states (KIND 2), with late compression: instance r of O.rep is stepped by the workgroups from r 2^lg on of those that blockIdx counts in
// steps of `spread`: 8 puts all of them on one XCD.
template <int W, int MODEL, int KIND>
__global__ __launch_bounds__(fq::RES_BS) void k_resident_joint(fq::Overlap O, fq::Fx3 *norms, int spread, int lg,
                                                               fq::i64 max_items, fq::u64 patience, fq::i64 stop)
{
    extern __shared__ __align__(16) char smem[];
    if ((int)blockIdx.x % spread) return;
    const int y = (int)blockIdx.x / spread, me = y >> lg;
    fq::resident_steps<W, MODEL, false, KIND>(fq::const_inst(O.rep[me]), y & ((1 << lg) - 1), lg, stop, max_items << lg,
                                              patience, O, me, norms, smem);
}

// explicit instantiations (EXT = extern: declaration only) of the merge,
// spawn and resident kernels of one (W, model variant) pair, all workgroup
// sizes and both compression styles (variant 1 is for one word only)
#define FQ_STEP_KERNEL_SET(EXT, W_, M_)                                                       \
    EXT template __global__ void k_merge<W_, M_, 256, false>(const fq::Inst *const *, const fq::u32 *); \
    EXT template __global__ void k_merge<W_, M_, 512, false>(const fq::Inst *const *, const fq::u32 *); \
    EXT template __global__ void k_merge<W_, M_, 1024, false>(const fq::Inst *const *, const fq::u32 *); \
    EXT template __global__ void k_merge<W_, M_, 256, true>(const fq::Inst *const *, const fq::u32 *); \
    EXT template __global__ void k_merge<W_, M_, 512, true>(const fq::Inst *const *, const fq::u32 *); \
    EXT template __global__ void k_merge<W_, M_, 1024, true>(const fq::Inst *const *, const fq::u32 *); \
    EXT template __global__ void k_spawn<W_, M_, 256, false>(const fq::Inst *const *, const fq::u32 *, int); \
    EXT template __global__ void k_spawn<W_, M_, 512, false>(const fq::Inst *const *, const fq::u32 *, int); \
    EXT template __global__ void k_spawn<W_, M_, 1024, false>(const fq::Inst *const *, const fq::u32 *, int); \
    EXT template __global__ void k_spawn<W_, M_, 256, true>(const fq::Inst *const *, const fq::u32 *, int); \
    EXT template __global__ void k_spawn<W_, M_, 512, true>(const fq::Inst *const *, const fq::u32 *, int); \
    EXT template __global__ void k_spawn<W_, M_, 1024, true>(const fq::Inst *const *, const fq::u32 *, int); \
    EXT template __global__ void k_resident<W_, M_, false>(const fq::Inst *const *, int, int, int, fq::i64, fq::u64, ResStops); \
    EXT template __global__ void k_resident<W_, M_, true>(const fq::Inst *const *, int, int, int, fq::i64, fq::u64, ResStops); \
    EXT template __global__ void k_resident_joint<W_, M_, 1>(fq::Overlap, fq::Fx3 *, int, int, fq::i64, fq::u64, fq::i64); \
    EXT template __global__ void k_resident_joint<W_, M_, 2>(fq::Overlap, fq::Fx3 *, int, int, fq::i64, fq::u64, fq::i64);

#define FQ_EXTERN_STEP_KERNELS                                                                \
    FQ_STEP_KERNEL_SET(extern, 1, 0) FQ_STEP_KERNEL_SET(extern, 1, 1) FQ_STEP_KERNEL_SET(extern, 1, 2)        \
    FQ_STEP_KERNEL_SET(extern, 1, 3) FQ_STEP_KERNEL_SET(extern, 2, 0) FQ_STEP_KERNEL_SET(extern, 2, 2)        \
    FQ_STEP_KERNEL_SET(extern, 2, 3)
