// fq_resident.hpp -- many FCIQMC steps of an instance in one launch.
//
// A step of a few thousand entries takes a few microseconds of work, but as
// four launches it took 32 to 45 us: every kernel starts with cold
// instruction and data caches, reads its descriptor, counts and data in
// dependent round trips of about 1 us each, and fills its LDS tables anew.
// Here G = 2^lg workgroups stay on the GPU and run step after step.
// Workgroup g owns B/G consecutive hash buckets of the instance.  A step is:
//   merge the own buckets in one LDS hash (the rules of merge_bucket), write
//   the survivors to table[1-p] and keep them in LDS, spawn from there into
//   the bucket slabs of every workgroup (slab[1-p]); then one barrier of the
//   G workgroups, after which each of them sums the G partial norms and
//   computes the same shift.
// Tables, slabs, counts and statistics in device memory are after every step
// what the step kernels would have left, up to the order of entries in a
// bucket, so either path continues the other's state.
//
// The barrier needs all G workgroups on the GPU at once.  A gate ensures
// that before anything is written: every workgroup counts itself in and
// waits for the last one, which opens the gate; a workgroup that has waited
// too long closes it instead (one compare-and-swap decides).  Behind a
// closed gate every workgroup returns, the instance has made no step, and the
// host steps it with the step kernels.  Behind an open gate every workgroup
// is running, so each later barrier ends.
//
// A small step is bound by its chain of dependent latencies (a dozen
// workgroup barriers of 60 ns, LDS and L2 round trips, Philox blocks, two
// logarithms, the barrier of the workgroups) and by the VALU issue of 16 waves
// on 4 SIMDs: 10.9 us a step at 1e3 walkers of the 6/6 ring.  The code is kept
// small (loops are rolled, every building block is inlined once; 30 KB); 67 KB
// of unrolled code were no faster.
//
// Exchange.  What another workgroup reads (records, counts, partial sums) is
// read with agent-scope loads.  An instance of up to 32 workgroups is placed
// on one XCD (workgroups go round robin to the 8 XCDs); when the gate finds
// all of them on one, their common L2 is the meeting point, and a barrier
// needs no cache maintenance.  Otherwise the last workgroup to arrive on each
// XCD writes its L2 back (agent release) for all of them, waits until that is
// done, and the XCDs meet.
// Measured per step with 1024 records of 12 bytes from every workgroup to all
// others: 1.4 to 1.6 us on one XCD at 2 to 16 workgroups, 2.2 at 32; on all
// XCDs 2.7 to 3.6 us up to 32, 4.0 at 64, 4.6 at 128 and 6.0 at 256 (4096
// records each: 12.0).  With a write back by every workgroup instead of one an
// XCD it was 6.1, 10.4 and 17.3 us at 64, 128 and 256 (4096 records: 34).
//
// Larger steps.  The same kernel is the faster one up to several million
// entries and records: the four kernels of a step each pay their cold start
// per bucket, some 14 us for the buckets that fit the chip at once.  A
// workgroup of a large step merges its buckets in one hash as long as their
// distinct addresses fit it, and reserves slab places for four rounds of
// attempts with one atomic per pair of buckets, in order of the buckets (23
// times the rate of single atomics, which cap a step at 10 records per ns).
// us a step, step kernels and resident: 16/16 in momentum space with the
// initiator rule at 1.4e6 items and 2048 buckets 99 and 57, the 16/16 ring at
// 1.8e6 items 135 and 64, 48 rings of 5e4 items 640 and 130.
#pragma once
#include "fq_overlap.hpp"
#include "fq_step.hpp"

namespace fq {

constexpr int RES_BS = 1024;      // threads of a workgroup: one workgroup per CU
// slots of its LDS hash, by address words
template <int W> struct ResSlots { static constexpr int N = W == 2 ? 2048 : 4096; };
constexpr int RES_MAXG = 256;     // workgroups of all instances of a launch: the CUs
constexpr int RES_MAXB = 8192;    // buckets of an instance: LDS counters of the spawn records
constexpr int RES_GROUP = 4;      // rounds of spawn attempts that reserve slab places together
constexpr int RES_MAXR = 8;       // replicas
constexpr int RES_XCCS = 16;      // values of the XCC_ID register
constexpr int RES_MAXK = 64;      // buckets of a workgroup: one wave scans their counts

// Partial sums of one workgroup for one step, and what it knows of the next.
// Every workgroup reads the first four words of all parts, workgroup 0 the
// rest as well.
struct ResPart {
    u64 norm[2];
    u64 items;    // entries from bit 40; records of the spawn pass for the next step below
    u64 state;    // bit 0: some sum was rounded first, bit 1: the step failed, bit 2: the hash did
                  // not hold the whole vector; from bit 8 the most distinct addresses in a
                  // bucket; from bit 32 exact parents of the spawn pass
    u64 hproj[2], vproj[2];
};
static_assert(sizeof(ResPart) == 64, "two to a cache line");

// Exchange area of one instance, counters zero before the launch.  The parts are
// double buffered by step parity: a workgroup can be at most one barrier
// ahead of the slowest reader.
struct ResSync {
    u32 arrived, gate, xccs, abort[2], pad0[11], on[RES_XCCS];  // XCDs the workgroups run on (mask), how many on each
    u32 count, pad1[31];
    u32 here[RES_XCCS][32];  // barrier arrivals by XCD, a line each
    ResPart part[2][RES_MAXG];
    u64 parents[2][RES_MAXG];  // excited states: survivors after the projection
};

// LDS: the hash; slot indices of its occupied slots (before them the marks
// of the initiator rule) and of the survivors; attempt offsets of the
// survivors; counters of the spawn records; then small tables.
template <int W> struct ResLds {
    static constexpr int N = ResSlots<W>::N;
    static constexpr int LIST = N * (W == 2 ? 36 : 24), LIVE = LIST + 2 * N, OFF = LIVE + 2 * N, CNT = OFF + 4 * N,
                         TABLES = CNT + 2 * RES_MAXB;
    // places of the spawn records by bucket: in the high words of the hash,
    // which hold nothing once compressed, if they are enough
    static constexpr bool IN_HASH = RES_MAXB <= 2 * N;
    static constexpr int BASE = IN_HASH ? 8 * N * (W + 1) : TABLES, MISC = TABLES + (IN_HASH ? 0 : 4 * RES_MAXB),
                         LUT = MISC + 64 * 8, TRI = LUT + 2048, RED = TRI + 2 * TRI_N, WORDS = RED + 8 * 20,
                         BYTES = WORDS + 7 * 4 * RES_MAXK;
    static_assert(BYTES + 512 <= 160 * 1024, "the LDS of one CU, with the kernel's own words");
};

template <class X> __device__ __forceinline__ X res_load(const X *p)
{
    return __hip_atomic_load(gmem(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// a spawn record that another workgroup wrote
template <int W> __device__ __forceinline__ void res_load_rec(int rec, const char *base, i64 i, u64 &a0, u64 &a1, double &v)
{
    a1 = 0;
    if (W == 2) {
        const u64 *r = (const u64 *)base + 3 * i;
        a0 = res_load(r);
        a1 = res_load(r + 1);
        v = bitsd(res_load(r + 2));
    } else if (rec == 12) {
        const u32 *r = (const u32 *)base + 3 * i;
        a0 = res_load(r);
        v = bitsd(((u64)res_load(r + 2) << 32) | res_load(r + 1));
    } else {
        const u64 *r = (const u64 *)base + 2 * i;
        a0 = res_load(r);
        v = bitsd(res_load(r + 1));
    }
}

// Whether every workgroup of the instance is on the GPU, or else the instance
// is not stepped here: the same answer in every workgroup.  where: the own
// XCD, its workgroups, and the number of XCDs.
__device__ __forceinline__ bool res_gate(ResSync *Y, int G, u64 patience, u32 *where)
{
    const u32 xcc = __builtin_amdgcn_s_getreg(20 | (3 << 11));  // hardware register 20 (XCC_ID), bits 0 .. 3
    u32 zero = 0;
    __hip_atomic_fetch_or(&Y->xccs, 1u << xcc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(&Y->on[xcc], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__hip_atomic_fetch_add(&Y->arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (u32)G - 1)
        __hip_atomic_compare_exchange_strong(&Y->gate, &zero, 1u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
    const u64 t0 = wall_clock64();
    u32 s;
    while ((s = __hip_atomic_load(&Y->gate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) {
        if (wall_clock64() - t0 > patience) {
            zero = 0;
            __hip_atomic_compare_exchange_strong(&Y->gate, &zero, 2u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_s_sleep(1);
    }
    where[0] = xcc;
    where[1] = __hip_atomic_load(&Y->on[xcc], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    where[2] = __popc(__hip_atomic_load(&Y->xccs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    return s == 1;
}

// Barrier number `round` (from 1) of the G workgroups of an instance: what
// any of them stored before it, all of them read behind it with agent-scope
// loads.  On several XCDs the last workgroup to arrive on each writes its L2
// back, once for all of them, and counts the XCD in.
__device__ __forceinline__ void res_barrier(ResSync *Y, int G, u32 round, const u32 *where)
{
    if (G == 1) {
        __syncthreads();
        return;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's stores have reached the L2
    __syncthreads();
    if (threadIdx.x == 0) {
        const u32 xcc = where[0], n = where[1], xccs = where[2];
        u32 all = (u32)G;
        bool count = true;
        if (xccs > 1) {
            all = xccs;
            count = __hip_atomic_fetch_add(&Y->here[xcc][0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                    n * round - 1u;
            if (count) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                // The count must not overtake the write back.  The compiler
                // leaves the fence's own wait out: it does not count the
                // write back among the operations in flight, and knows of no other.
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
        }
        if (count) __hip_atomic_fetch_add(&Y->count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        while (__hip_atomic_load(&Y->count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < all * round) {}
    }
    __syncthreads();
}

// Replicas (Sec. 4.3) are stepped together, with one gate and one barrier for
// the workgroups of all of them (in the exchange area of the first), because
// the overlaps of a step need all vectors of that step.  Workgroup g of
// replica A still has its part of the vector in the hash when the barrier
// behind the step opens, and the other replicas' tables hold the same buckets
// of theirs: they are streamed against the hash before it is cleared.  What
// the workgroups add up is published at the next barrier, in O.part (twice,
// by parity of the round; hence at most half as many workgroups as buckets),
// and the row written behind it.  Two replicas of the 8/8 ring in momentum
// space at 1e3 walkers take 15.7 us a step so, 43.8 with the step and overlap
// kernels.
__device__ __forceinline__ void wave_scan_fx3(Fx3 &x)  // sum in lane 63
{
    fx3_add(x, Fx3{dpp0<0x111, 0xf>(x.w0), dpp0<0x111, 0xf>(x.w1), dpp0<0x111, 0xf>(x.w2)});
    fx3_add(x, Fx3{dpp0<0x112, 0xf>(x.w0), dpp0<0x112, 0xf>(x.w1), dpp0<0x112, 0xf>(x.w2)});
    fx3_add(x, Fx3{dpp0<0x114, 0xf>(x.w0), dpp0<0x114, 0xf>(x.w1), dpp0<0x114, 0xf>(x.w2)});
    fx3_add(x, Fx3{dpp0<0x118, 0xf>(x.w0), dpp0<0x118, 0xf>(x.w1), dpp0<0x118, 0xf>(x.w2)});
    fx3_add(x, Fx3{dpp0<0x142, 0xa>(x.w0), dpp0<0x142, 0xa>(x.w1), dpp0<0x142, 0xa>(x.w2)});
    fx3_add(x, Fx3{dpp0<0x143, 0xc>(x.w0), dpp0<0x143, 0xc>(x.w1), dpp0<0x143, 0xc>(x.w2)});
}

// Entries [0, words[K]) of the buckets [bA, bA + K) of a table: f(a0, a1, v).
template <int W, class F>
__device__ __forceinline__ void resident_stream(const Inst &IJ, const int pj, const int bA, const int K,
                                                const int *words, F f)
{
#pragma unroll 1
    for (int i = threadIdx.x; i < words[K]; i += RES_BS) {
        int k = 0;
        for (int hi = K; hi - k > 1;) {
            const int mid = (k + hi) >> 1;
            if (words[mid] <= i) k = mid;
            else hi = mid;
        }
        const i64 e = (i64)(bA + k) * IJ.cap_t + (i - words[k]);
        f(res_load(&IJ.tab_a[pj][0][e]), W == 2 ? res_load(&IJ.tab_a[pj][1][e]) : (u64)0,
          bitsd(res_load((const u64 *)IJ.tab_v[pj] + e)));
    }
}
// words[0 .. K]: where the entries of the buckets start
__device__ __forceinline__ void resident_stream_words(const Inst &IJ, const int pj, const int bA, const int K, int *words)
{
    const int lane = threadIdx.x & 63;
    if (threadIdx.x >= 64) return;
    int n = lane < K ? res_load(&IJ.tab_n[pj][bA + lane]) : 0;
    n = (int)wave_scan((u64)min((i64)n, IJ.cap_t));
    if (lane < K) words[lane + 1] = n;
    if (lane == 0) words[0] = 0;
}

// Overlaps of replica A with every later replica on the buckets [bA, bA + K):
// its amplitudes are in the hash (low word; 0 where compressed away).
// words: LDS, K + 1 ints and from word 2 RES_MAXK 16 Fx3; to[pair].
template <int W>
__device__ __forceinline__ void resident_overlap(const Overlap &O, const Lds &L, const int A, const int *parity,
                                                 const int bA, const int K, int *words, Fx3 *to)
{
    constexpr int BS = RES_BS;
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    Fx3 *tmp = (Fx3 *)(words + 2 * RES_MAXK);
    int inexact = 0, ovf = 0;
#pragma unroll 1
    for (int B = A + 1; B < O.R; B++) {
        const Inst &IB = const_inst(O.rep[B]);
        const int pB = parity[B];
        resident_stream_words(IB, pB, bA, K, words);
        __syncthreads();
        Fx3 acc = fx3_zero();
        resident_stream<W>(IB, pB, bA, K, words, [&](u64 a0, u64 a1, double v) {
            const int s = lds_find<W>(L, a0, a1, slot_hash(a0, a1));
            const double c = s >= 0 ? bitsd(L.lo[s]) : 0.0;
            if (c != 0.0) fx3_add(acc, to_fx3(c * v, inexact, ovf));
        });
        if (__any((acc.w0 | acc.w1 | acc.w2) != 0)) wave_scan_fx3(acc);
        if (lane == 63) tmp[wid] = acc;
        __syncthreads();
        if (wid == 0) {
            acc = lane < BS / 64 ? tmp[lane] : fx3_zero();
            wave_scan_fx3(acc);
            if (lane == 63) to[pair_index(A, B, O.R)] = acc;
        }
    }
    if (inexact) atomicOr(&O.flags[1], 1);
    if (ovf) atomicOr(&O.flags[2], 1);
    __syncthreads();
}

// Excited states (Sec. 2.2): two runs, the second orthogonalised against the
// first between merge and spawn, step together in the same way, with three
// barriers a step.  At the first the new table of run 0 is complete; a step in
// which a hash did not hold its vector or a merge failed ends there, undone
// (only the tables that the next step overwrites have been written), and the
// step kernels make it.  Then the workgroups of run 1 stream their buckets of
// run 0 against their hash for c_0 . c_1 and c_0 . c_0, counting the addresses
// of run 0 that it does not hold, meet, and stream them once more to
// subtract.  The second barrier undoes the step in the same way when some
// hash does not hold the addresses of both runs: its vote has a word of its
// own, because the votes of the first barrier are still being read then.  A
// step of two runs of the 12/12 ring at 1e5 walkers takes 46 us so, 92 with
// the step and projection kernels.
//
// This workgroup's c_0 . c_1 and c_0 . c_0 (to[0], to[1]); words: as above,
// the sums of the waves behind them.  addresses (LDS): those of the hash,
// plus in the end those of run 0 beyond them.
template <int W>
__device__ __forceinline__ void resident_dot(const Inst &I, const Lds &L, const Inst &IJ, const int pj, const int bA,
                                             const int K, int *words, int *flags, Fx3 *to, int *addresses)
{
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Fx3 *tmp = (Fx3 *)(words + 2 * RES_MAXK);
    resident_stream_words(IJ, pj, bA, K, words);
    __syncthreads();
    int inexact = 0, ovf = 0;
    Fx3 dot = fx3_zero(), sq = fx3_zero();
    int fresh = 0;
    resident_stream<W>(IJ, pj, bA, K, words, [&](u64 a0, u64 a1, double v) {
        fx3_add(sq, to_fx3(v * v, inexact, ovf));
        const int s = lds_find<W>(L, a0, a1, slot_hash(a0, a1));
        fresh += s < 0;
        const double c = s >= 0 ? bitsd(L.lo[s]) : 0.0;
        if (c != 0.0) fx3_add(dot, to_fx3(v * c, inexact, ovf));
    });
    wave_scan_fx3(dot);
    wave_scan_fx3(sq);
    fresh = (int)wave_scan((u64)fresh);
    if (lane == 63 && fresh) atomicAdd(addresses, fresh);
    if (lane == 63) {
        tmp[wid] = dot;
        tmp[RES_BS / 64 + wid] = sq;
    }
    if (inexact) atomicOr(flags, 1);
    if (ovf) fail(I, L, FQE_DIVERGED, bA);
    __syncthreads();
    if (wid < 2) {
        Fx3 x = lane < RES_BS / 64 ? tmp[wid * (RES_BS / 64) + lane] : fx3_zero();
        wave_scan_fx3(x);
        if (lane == 63) to[wid] = x;
    }
}

// c_1 <- c_1 - alpha c_0 in the hash, which has room for the addresses of
// both, unless the step is undone (*undone, LDS, read behind a barrier);
// sums: the workgroups' resident_dot
template <int W>
__device__ __forceinline__ void resident_project(const Inst &I, const Lds &L, const Inst &IJ, const int pj, const int bA,
                                                 const int K, const int G, const int *words, const Fx3 *sums,
                                                 double *s_alpha, const int *undone)
{
    const int lane = threadIdx.x & 63;
    if (threadIdx.x < 64) {
        Fx3 d = fx3_zero(), q = fx3_zero();
#pragma unroll 1
        for (int w = lane; w < G; w += 64) {
            const Fx3 *x = sums + 2 * w;
            fx3_add(d, Fx3{res_load(&x[0].w0), res_load(&x[0].w1), res_load(&x[0].w2)});
            fx3_add(q, Fx3{res_load(&x[1].w0), res_load(&x[1].w1), res_load(&x[1].w2)});
        }
        wave_scan_fx3(d);
        wave_scan_fx3(q);
        if (lane == 63) {
            const double nq = from_fx3(q);
            *s_alpha = nq > 0.0 ? from_fx3(d) / nq : 0.0;
        }
    }
    __syncthreads();
    if (*undone) return;
    const double alpha = *s_alpha;
    int np = 0;  // (probes, not reported from here)
    resident_stream<W>(IJ, pj, bA, K, words, [&](u64 a0, u64 a1, double v) {
        const int s = lds_slot<W>(L, a0, a1, slot_hash(a0, a1), np);
        if (s < 0) {
            fail(I, L, FQE_CAP_LDS, bA);
        } else {
            const double p = alpha * v;
            L.lo[s] = dbits(bitsd(L.lo[s]) - p);
        }
    });
}

// Exclusive scan of x over the workgroup; tmp: 16 words.  One barrier.
__device__ __forceinline__ u64 res_scan(u64 x, u64 *tmp, u64 &total)
{
    static_assert(RES_BS / 64 == 16, "one lane of a row per wave");
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u64 in = wave_scan(x);
    if (lane == 63) tmp[wid] = in;
    __syncthreads();
    const u64 w = row_scan(tmp[lane & 15]);
    total = lane_value(w, 15);
    return in - x + (wid ? lane_value(w, wid - 1) : 0);
}

// The A attempts of the nS survivors (hash slots list[i], attempts before
// survivor i in off[i]) for step spawn_step, straight into the bucket slabs
// of parity out_par.  The step kernel cuts the attempts of a bucket into
// units of four of one parent, to save instructions; here a few hundred
// attempts meet 1024 threads, and the length of the chain counts: the
// attempts of all parents, exact and stochastic, are enumerated flat, one per
// thread and round, each with its own parent search (four ways at a time)
// and Philox block.  A thread keeps the records of RES_GROUP rounds in
// registers until their places are known.  cnt, base: records of these rounds
// by bucket (16 bits each, from 0) and their place in its slab, from own (all
// records so far) when this workgroup is alone, else from one global atomic
// for two buckets; the workgroups start at different ones (bucket `first`).
// misc[60] counts the records of early compression.
template <int W, int MODEL, bool EARLY>
__device__ __forceinline__ void resident_spawn(const Inst &I, const Lds &L, const int out_par, const int first,
                                               const bool alone,
                                               const u32 spawn_step, const int nS, const i64 A,
                                               const unsigned short *list, const u32 *off, u32 *cnt, int *base,
                                               int *own, const unsigned char *lut, const unsigned short *tri)
{
    typedef typename AddrOf<W>::T T;
    constexpr int BS = RES_BS, R = RES_GROUP;
    const int tid = threadIdx.x;
    const bool narrow = MODEL == 1 || (W == 1 && I.mc.nb <= 32);
    int top = 1;
    while (4 * top < nS) top *= 4;
    static_assert(RES_MAXB <= 1 << 13, "bucket and rank in one word");
#pragma unroll 1
    for (i64 from = 0; from < A; from += R * BS) {
        // records of the last R rounds; at = bucket + (rank among the group's records of the bucket) << 13
        T d[R];
        double v[R];
        int at[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            d[r] = AddrOf<W>::make(0, 0);
            v[r] = 0.0;
            at[r] = -1;
        }
#pragma unroll 1
        for (int r = 0; r < R && from + r * BS < A; r++) {
#pragma unroll
            for (int e = R - 1; e > 0; e--) {
                d[e] = d[e - 1];
                v[e] = v[e - 1];
                at[e] = at[e - 1];
            }
            at[0] = -1;
            // (wave 0 takes the last attempts: it has the row to write)
            const i64 x = from + r * BS + ((tid + BS - 64) & (BS - 1));
            if (x >= A) continue;
            // the last survivor whose first attempt is at or before x
            int w = 0;
#pragma unroll 1
            for (int stp = top; stp > 0; stp >>= 2) {
                const int i1 = w + stp, i2 = i1 + stp, i3 = i2 + stp;
                const u32 o1 = off[min(i1, nS - 1)], o2 = off[min(i2, nS - 1)], o3 = off[min(i3, nS - 1)];
                w = i3 < nS && o3 <= (u32)x ? i3 : i2 < nS && o2 <= (u32)x ? i2 : i1 < nS && o1 <= (u32)x ? i1 : w;
            }
            const u32 k = (u32)x - off[w], n = (w + 1 < nS ? off[w + 1] : (u32)A) - off[w];
            const int s = list[w];
            const u64 a0 = L.k0[s], a1 = W == 2 ? L.k1[s] : 0;
            const double c = bitsd(L.lo[s]);
            const T a = AddrOf<W>::make(a0, a1);
            double h;
            if constexpr (MODEL == 0 || MODEL == 3) {
                const int m = (MODEL == 0 ? 2 : I.mc.ndir) * (narrow ? popc(run_starts((u32)a0)) : popc(run_starts(a)));
                const bool exact = fabs(c) >= I.t_rel * (double)m;
                int e = (int)k;
                if (!exact) e = (int)pick(rword(draw(I.seed, a0, a1, spawn_step, 0u, k >> 2), (int)(k & 3u)), (u32)m);
                // in 32-bit words when the address fits them
                auto entry = [&](auto y) {
                    const auto st = run_starts(y);
                    if constexpr (MODEL == 0) {
                        return real_entry(I.mc, y, st, popc(st), e, h);
                    } else {
                        int kd;
                        const auto z = lat_entry(I.mc, y, st, popc(st), e, h, kd, lut);
                        h = h * gmem(I.mc.gz)[I.mc.N + kd];
                        return z;
                    }
                };
                if (narrow) d[0] = AddrOf<W>::make((u64)entry((u32)a0), 0);
                else d[0] = entry(a);
                v[0] = (-(I.dtau * h)) * c;
                if (!exact) v[0] = v[0] * ((double)m / (double)n);
            } else {
                const i64 m = narrow ? mom_col_size<u32>(I.mc, (u32)a0) : mom_col_size(I.mc, a);
                if (fabs(c) >= I.t_rel * (double)m) {
                    if (narrow) d[0] = AddrOf<W>::make((u64)mom_column_entry<u32>(I.mc, (u32)a0, (int)k, h, lut), 0);
                    else d[0] = mom_column_entry(I.mc, a, (int)k, h, lut);
                    v[0] = (-(I.dtau * h)) * c;
                } else {
                    const R4 rr = draw(I.seed, a0, a1, spawn_step, 0u, k >> 1);
                    const u32 x0 = (k & 1u) ? rr.z : rr.x, x1 = (k & 1u) ? rr.w : rr.y;
                    int R, P;
                    if constexpr (MODEL == 1 && W == 1) {
                        const MomCtx32 y = mom_ctx32(I.mc, (u32)a0);
                        P = y.P;
                        d[0] = AddrOf<W>::make((u64)mom_draw31(I.mc, y, x0, x1, h, R, lut, tri), 0);
                    } else {
                        const MomCtx<T> y = mom_ctx<T>(I.mc, a);
                        P = y.P;
                        d[0] = mom_draw<T>(I.mc, y, x0, x1, h, R, lut);
                    }
                    v[0] = ((-(I.dtau * h)) * c) * ((double)((i64)P * R) / (double)n);
                }
            }
            const u64 fl = !(fabs(c) > I.n_a) ? I.iflag : 0ull;
            if (EARLY && fabs(v[0]) < I.theta)
                v[0] = compress1(v[0], I.theta, draw(I.seed, a0, a1, spawn_step, 4u + (k >> 28), k & 0x0fffffffu).x);
            if (!EARLY || v[0] != 0.0) {
                const int t = (int)bucket_index(d[0], I.log2B, I.mc.nb <= 32), up = 16 * (t & 1);
                at[0] = t | (((atomicAdd(&cnt[t >> 1], 1u << up) >> up) & 0xffff) << 13);
            }
            d[0] = AddrOf<W>::make(W == 1 ? word0(d[0]) | fl : word0(d[0]), W == 2 ? word1(d[0]) | fl : 0ull);
        }
        __syncthreads();
        if (*L.failed) break;  // a slab is full: counts stay near its size
        for (int i = tid; 2 * i < I.B; i += BS) {
            const int w = (i + first / 2) & (I.B / 2 - 1);  // the workgroups start at different buckets
            const u32 c = cnt[w];
            if (c) {
                const int c0 = (int)(c & 0xffff), c1 = (int)(c >> 16);
                if (alone) {
                    base[2 * w] = own[2 * w];
                    own[2 * w] += c0;
                    if (c1) {
                        base[2 * w + 1] = own[2 * w + 1];
                        own[2 * w + 1] += c1;
                    }
                } else {
                    // (two counts that stay below 2^31 in one word)
                    const u64 x = gatomic_add((u64 *)&I.slab_n[out_par][2 * w], ((u64)(u32)c1 << 32) | (u32)c0);
                    base[2 * w] = (int)(u32)x;
                    base[2 * w + 1] = (int)(x >> 32);
                }
                cnt[w] = 0;
                if (EARLY) atomicAdd((unsigned long long *)&L.misc[60], (unsigned long long)(c0 + c1));
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (at[r] < 0) continue;
            const int t = at[r] & ((1 << 13) - 1);
            const i64 pos = (i64)base[t] + (at[r] >> 13);
            if (pos < I.cap_s) store_rec<W>(I.rec, I.slab[out_par], (i64)t * I.cap_s + pos, d[r], v[r]);
            else fail(I, L, FQE_CAP_SLAB, t);
        }
    }
}

// Steps of instance I up to last_step by workgroup g of G = 2^lg (every
// workgroup of the instance makes the same number).  Stops early at the
// instance's stop step, at an error, and after a step that leaves more than
// max_items entries and records to merge.  An instance whose buckets may hold
// more addresses than the hash is not begun when one of them might now; later
// the number of items, half the hash a bucket, keeps them from it, and a
// bucket that nevertheless fills three quarters of it (a state may have all
// its entries in one bucket) ends the launch.
// KIND 1: the instance is replica `me` of O, whose replicas start at one step
// and stop together: all of them decide from the same sums and flags.  O.ring
// receives the overlaps of all steps but the last, whose tables the launch
// leaves.  KIND 2: run `me` of two for excited states, together likewise;
// O.part takes the dot products (two a workgroup), norms the projected norms,
// O.flags[0] whether one was rounded.
template <int W, int MODEL, bool EARLY, int KIND>
__device__ __forceinline__ void resident_steps(const Inst &I, const int g, const int lg, const i64 last_step,
                                               const i64 max_items, const u64 patience, const Overlap &O, const int me,
                                               Fx3 *norms, char *smem)
{
    typedef typename AddrOf<W>::T T;
    typedef ResLds<W> M;
    constexpr int BS = RES_BS, SLOTS = ResSlots<W>::N;
    constexpr bool OV = KIND == 1, GS = KIND == 2, JOINT = KIND != 0;
    const bool second = GS && me == 1;
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = 1 << lg;
    const int K = I.B >> lg;   // buckets of this workgroup, at most RES_MAXK
    const int bA = g * K;
    Ctrl *ctrl = I.ctrl;
    // the workgroups that meet at the barrier, and where
    const int meet = JOINT ? O.R << lg : G;
    ResSync *Y = JOINT ? const_inst(O.rep[0]).res : I.res;

    __shared__ int s_go, s_fail, s_full, s_len, s_load, s_inx, s_list, s_ex;
    __shared__ u32 s_where[3];
    __shared__ double s_state[2];  // shift and norm after the step
    __shared__ i64 s_sp;
    __shared__ int s_par[JOINT ? RES_MAXR : 1];  // parity of each replica's state
    __shared__ int s_live, s_abort;                // excited states: survivors after the projection; the step is undone
    __shared__ double s_alpha, s_projected;
    Lds L;
    L.k0 = (u64 *)smem;
    L.k1 = L.k0 + SLOTS;
    L.lo = L.k0 + SLOTS * W;
    L.hi = L.lo + SLOTS;
    L.state = (u32 *)(L.hi + SLOTS);
    L.misc = (i64 *)(smem + M::MISC);
    L.occ = (unsigned char *)(smem + M::LIST);
    L.failed = &s_fail;
    L.full = &s_full;
    unsigned short *list = (unsigned short *)(smem + M::LIST), *live = (unsigned short *)(smem + M::LIVE);
    u32 *off = (u32 *)(smem + M::OFF);
    u32 *cnt = (u32 *)(smem + M::CNT);
    int *base = (int *)(smem + M::BASE);
    unsigned char *lut = (unsigned char *)(smem + M::LUT);
    unsigned short *tri = (unsigned short *)(smem + M::TRI);
    // 128-bit sums of the workgroup, ||c||_1, y.Hc, y.c, as 32-bit limbs in
    // 64-bit words (adds without a carry); from word 12 the sums of a row
    u64 *red = (u64 *)(smem + M::RED);
    int *pt = (int *)(smem + M::WORDS), *ps = pt + 2 * RES_MAXK;  // own buckets: prefix sums of the entries, the records
    int *keep = ps + 2 * RES_MAXK, *used = keep + RES_MAXK;  // survivors, distinct addresses
    int *own = used + RES_MAXK;                   // G = 1: records written, per bucket (B <= RES_MAXK then)
    const bool init = I.iflag != 0;
    const bool narrow = MODEL == 1 || (W == 1 && I.mc.nb <= 32);

    // the state before this launch, read before the gate: no workgroup
    // changes it until all of them have passed
    i64 n = ctrl->step;
    int p = ctrl->parity;
    double S = ctrl->shift, N0 = ctrl->norm;
    const i64 stop = min(ctrl->stop_step, last_step);
    const bool large = I.slots > SLOTS;
    const i64 item_limit = large ? min(max_items, (i64)I.B * (SLOTS / 2)) : max_items;
    const i64 ring_base = ctrl->ring_base;
    if (tid == 0) s_go = !halted(ctrl);
    __syncthreads();
    if (JOINT) {
        // none is stepped when one of them cannot be: the same answer in every workgroup
        if (tid < O.R) {
            Ctrl *c = const_inst(O.rep[tid]).ctrl;
            s_par[tid] = c->parity;
            if (halted(c) || c->step != n || c->stop_step != ctrl->stop_step) s_go = 0;
        }
        __syncthreads();
    }
    if (!s_go) return;
    if (large) {
        __syncthreads();
        if (tid < K && (i64)I.tab_n[p][bA + tid] + I.slab_n[p][bA + tid] > SLOTS) s_go = 0;
        __syncthreads();
        if (!s_go) {
            // not here, and not by the other workgroups
            u32 zero = 0;
            if (tid == 0 && meet > 1)
                __hip_atomic_compare_exchange_strong(&Y->gate, &zero, 2u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
    }
    if (meet > 1) {
        __syncthreads();
        if (tid == 0) s_go = res_gate(Y, meet, patience, s_where);
        __syncthreads();
        if (!s_go) return;
    }
    if (n >= stop) return;
    for (int i = tid; i < 2048; i += BS) lut[i] = select_lut_entry(i);
    if (MODEL == 1 || MODEL == 2) tri_fill(tri, tid, BS);
    for (int t = tid; 2 * t < I.B; t += BS) cnt[t] = 0;
    // the reference entries of the own buckets, one per thread from the last
    // thread down, if there are no more than threads
    const int ref0 = I.ref_off[bA], nref = I.ref_off[bA + K] - ref0;
    const bool ref_held = nref <= BS;
    u64 f0 = 0, f1 = 0;
    double fh = 0.0;
    if (ref_held && BS - 1 - tid < nref) {
        f0 = gmem(I.ref_a[0])[ref0 + BS - 1 - tid];
        if (W == 2) f1 = gmem(I.ref_a[1])[ref0 + BS - 1 - tid];
        fh = gmem(I.ref_h)[ref0 + BS - 1 - tid];
    }
    // workgroup 0 writes the rows: counts of the spawn pass before the first step
    i64 row_ex = 0, row_st = 0, row_sp = 0;
    u32 row_inx = 0;
    i64 first_inx = 0;
    int max_load = 0;
    if (g == 0 && wid == 0) {
        for (int b = lane; b < I.B; b += 64) {
            const SpawnPart x = I.spart[(n + 1) & 1][b];
            row_ex += x.exact;
            row_st += x.inexact;
            row_sp += x.spawns;
        }
        row_ex = (i64)lane_value(wave_scan((u64)row_ex), 63);
        row_st = (i64)lane_value(wave_scan((u64)row_st), 63);
        row_sp = (i64)lane_value(wave_scan((u64)row_sp), 63);
        row_inx = ctrl->inexact_in;
        first_inx = ctrl->first_inexact;
    }

    u32 round = 0, met = 0;  // steps begun and barriers passed in this launch
    double Nrow = N0;        // norm of the row to be written
    int slots = 0;           // of the hash: from the distinct addresses of the step before
    bool few = false;        // those fill no more than 5/8 of the whole hash
    bool concluded = true;   // no step waits for its shift
    bool held = false;       // the survivors are in registers, at most one per thread: hc = 0 or (h0, h1), hc
    u64 h0 = 0, h1 = 0;
    double hc = 0.0;
    bool row_due = false;    // wave 0 of workgroup 0: the row of step n is to be written
    bool whole = true;       // the hash holds the whole vector of the step
    bool dead = false;       // OV: this replica has diverged and waits for the others to hear of it
    // OV, replica 0: the step whose overlaps have been published and are to be written, and from which half of O.part
    i64 ov_step = -1;
    Fx3 *const sums = OV ? O.part + (i64)g * O.P : nullptr;  // this workgroup's overlaps, first half
    auto write_overlaps = [&]() {
        const i64 row = ov_step - ring_base;
#pragma unroll 1
        for (int k = 0; k < O.P; k++) {
            Fx3 x = fx3_zero();
#pragma unroll 1
            for (int w = lane; w < G; w += 64) {
                const Fx3 *y = O.part + ((i64)((round & 1) ^ 1) * G + w) * O.P + k;
                fx3_add(x, Fx3{res_load(&y->w0), res_load(&y->w1), res_load(&y->w2)});
            }
            wave_scan_fx3(x);
            if (lane == 63 && row >= 0 && row < O.ring_cap) O.ring[row * O.P + k] = from_fx3(x);
        }
        ov_step = -1;
    };
    auto write_row = [&]() {
        const bool flagged = red[18] || row_inx;
        // one conversion: y.Hc in lane 0, y.c in the others
        const double e = from_fixed(red[lane == 0 ? 12 : 14], red[lane == 0 ? 13 : 15]);
        const double hp = lane_value(e, 0), vp = lane_value(e, 1);
        const i64 len = (i64)(red[17] >> 40), row = n - ring_base;
        if (lane == 0 && row >= 0 && row < I.ring_cap) {
            StepStats &R = I.ring[row];
            R.step = n;
            R.len = len;
            R.exact_steps = row_ex;
            R.inexact_steps = row_st;
            R.spawns = row_sp;
            R.shift = S;
            R.norm = GS ? Nrow : N0;
            R.hproj = hp;
            R.vproj = vp;
            R.flags = flagged ? ROW_INEXACT : 0;
        }
        row_inx = 0;
        if (flagged && first_inx == 0) first_inx = n;
        row_ex = (i64)red[16];
        row_st = (GS ? (i64)red[19] : len) - row_ex;
        row_sp = (i64)(red[17] & (((u64)1 << 40) - 1));
        row_due = false;
    };
    s_go = 2;
    if (GS && tid == 0) s_abort = 0;
    for (;;) {
        // ------------------------------------------------ 0. what the other workgroups left
        // wave 0: the parts of the step that waits for its shift, summed over
        // the workgroups lane, lane + 64, ..
        u64 nl = 0, nh = 0, both = 0, state = 0;
        bool full = false;  // a bucket of any instance that meets here comes close to the hash
        auto load_of = [](u64 st) { return (int)((st >> 8) & 0xffffff); };
        const bool split = !concluded;
        const ResPart *part = I.res->part[round & 1];
        if (OV && split && !dead && me < O.R - 1)
            resident_overlap<W>(O, L, me, s_par, bA, K, (int *)off, sums + (i64)(round & 1) * G * O.P);
        if (split && wid == 0) {
#pragma unroll 1
            for (int k = lane; k < G; k += 64) {
                const u64 x0 = res_load(&part[k].norm[0]), x1 = res_load(&part[k].norm[1]),
                          x2 = res_load(&part[k].items), x3 = res_load(&part[k].state);
                add128(nl, nh, x0, x1);
                both += x2;
                full = full || (large && load_of(x3) > 3 * SLOTS / 4);
                // flags joined, largest load, sum of exact parents
                state = (state & 7) | (x3 & 7) | (max(state & 0xffffff00u, x3 & 0xffffff00u)) |
                        (((state >> 32) + (x3 >> 32)) << 32);
            }
        }
        u64 others = 0;  // OV: flags of the other replicas; their entries and records from bit 8
        if (JOINT && split && wid == 0) {
#pragma unroll 1
            for (int w = lane; w < meet; w += 64) {
                const int r = w >> lg;
                if (r == me) continue;
                const ResPart *x = &const_inst(O.rep[r]).res->part[round & 1][w & (G - 1)];
                const u64 it = res_load(&x->items), st = res_load(&x->state);
                others |= st & 6;
                full = full || (large && load_of(st) > 3 * SLOTS / 4);
                others += ((it >> 40) + (it & (((u64)1 << 40) - 1))) << 8;
            }
        }
        // wave 1: the counts of the own buckets
        const int p1 = concluded ? p : 1 - p;  // parity of the state to advance
        if (wid == 1) {
            int x = 0, y = 0;
            if (lane < K) {
                x = res_load(&I.tab_n[p1][bA + lane]);
                y = min(res_load(&I.slab_n[p1][bA + lane]), (int)I.cap_s);
            }
            const u64 xy = wave_scan(((u64)x << 32) | (u32)y);
            if (lane < K) {
                pt[lane + 1] = (int)(xy >> 32);
                ps[lane + 1] = (int)(u32)xy;
                keep[lane] = used[lane] = own[lane] = 0;
            }
            if (lane < 12) red[lane] = 0;
            if (lane == 0) {
                pt[0] = ps[0] = 0;
                s_fail = s_full = 0;
                s_len = s_load = s_inx = s_ex = 0;
                s_sp = 0;
                if (GS) s_live = 0;
            }
        }
        int inx = 0, distinct = 0;
        int np = 0;  // (probes, not reported from here)
        // Batches of consecutive buckets whose entries and records together
        // fit the hash; a bucket larger than that is a batch alone (its
        // distinct addresses usually fit).  The first batch is cleared for
        // while the counts arrive, and merged again if it does not fit.
        for (int k0 = 0, k1 = 0, redo = 0, most = JOINT ? 1 << 30 : few ? 8 * SLOTS : SLOTS; k0 < K;) {
            const bool all = k0 > 0 || redo;
            if (all || slots == 0 || second) slots = SLOTS;
            if (all || wid > 1) {
#pragma unroll 1
                for (int s = all ? tid : tid - 128; s < slots; s += all ? BS : BS - 128) {
                    L.k0[s] = EMPTY;
                    if (W == 2) { L.k1[s] = EMPTY; L.state[s] = 0u; }
                    L.lo[s] = 0;
                    L.hi[s] = 0;
                }
            }
            if (tid == 64) s_list = s_full = 0;
            __syncthreads();
            k1 = K;
            if (pt[K] - pt[k0] + ps[K] - ps[k0] > most) {
                k1 = k0 + 1;
                while (k1 < K && pt[k1 + 1] - pt[k0] + ps[k1 + 1] - ps[k0] <= most) k1++;
            }
            L.mask = slots - 1;
            // ------------------------------------------------ 1. merge
            // The records first; meanwhile wave 0, which takes no items,
            // concludes the step before, whose shift scales the survivors:
            // s_go = 0 that step failed, 1 it was the last, 2 go on, 3 it
            // failed and the other replicas do not know.  With
            // the initiator rule the survivors come first.
            const bool waits = split && !concluded;
            if (waits && wid == 0) {
                const int last = G <= 16 ? 15 : 63;
                if (G > 1) {
                    row_scan128(nl, nh);
                    both = row_scan(both);
                    if (G > 16) {
                        add128(nl, nh, dpp0<0x142, 0xa>(nl), dpp0<0x142, 0xa>(nh));
                        add128(nl, nh, dpp0<0x143, 0xc>(nl), dpp0<0x143, 0xc>(nh));
                        both += dpp0<0x142, 0xa>(both);
                        both += dpp0<0x143, 0xc>(both);
                    }
                }
                const int from = G > 1 ? last : 0;
                nl = lane_value(nl, from);
                nh = lane_value(nh, from);
                both = lane_value(both, from);
                const double N1 = from_fixed(nl, nh);
                // lanes 0 and 1 take one logarithm each
                const double ln = N1 > 0.0 ? det_log(N1 / (lane == 0 ? N0 : I.target)) : 0.0;
                const double l0 = lane_value(ln, 0), l1 = lane_value(ln, 1);
                double S1 = S;
                if (N1 > 0.0) S1 = (S - I.zeta / I.dtau * l0) - I.xi / I.dtau * l1;
                const bool error = __any(state & 2), diverged = !(N1 < 17592186044416.0) || !(S1 == S1);
                i64 items = (i64)(both >> 40) + (i64)(both & (((u64)1 << 40) - 1));
                bool end = n + 1 >= stop || __any(full);
                if (JOINT) {
                    // the same answer in every replica: after each step all go on or none
                    items += (i64)lane_value(wave_scan(others >> 8), 63);
                    end = end || items > item_limit * O.R || __any(((others | state) & 6) != 0);
                } else {
                    end = end || items > item_limit;
                }
                if (lane == 0) {
                    // (a replica that has diverged takes part in one more step, for the others to read its flag)
                    s_go = error ? 0 : diverged ? (JOINT && !end ? 3 : 0) : end ? 1 : 2;
                    s_state[0] = S1;
                    s_state[1] = N1;
                    if (g == 0 && !error && diverged) set_error(ctrl, FQE_DIVERGED, -1);
                }
                if (second) {
                    Fx3 x = fx3_zero();
#pragma unroll 1
                    for (int w = lane; w < G; w += 64)
                        fx3_add(x, Fx3{res_load(&norms[w].w0), res_load(&norms[w].w1), res_load(&norms[w].w2)});
                    wave_scan_fx3(x);
                    if (lane == 63) s_projected = from_fx3(x);
                }
            }
#pragma unroll 1
            for (int ph = 0; ph < 3; ph++) {
                // 0: records, 1: table, 2: records with the initiator rule
                if (ph == 1) {
                    if (waits) {
                        __syncthreads();
                        concluded = true;
                        dead = JOINT && s_go == 3;
                        if (s_go == 1 || s_go == 2) {
                            n++;
                            p = p1;
                            S = lane_value(s_state[0], 0);
                            N0 = lane_value(s_state[1], 0);
                            if (GS) Nrow = N0;
                            if (second) N0 = lane_value(s_projected, 0);
                        }
                        if ((s_go == 1 || s_go == 2) && g == 0 && wid == 0) {
                            // the sums of its row, written further down
                            u64 hl = 0, hh = 0, vl = 0, vh = 0, parents = 0;
#pragma unroll 1
                            for (int k = lane; k < G; k += 64) {
                                if (GS) parents += res_load(&I.res->parents[round & 1][k]);
                                const u64 x0 = res_load(&part[k].hproj[0]), x1 = res_load(&part[k].hproj[1]),
                                          x2 = res_load(&part[k].vproj[0]), x3 = res_load(&part[k].vproj[1]);
                                add128(hl, hh, x0, x1);
                                add128(vl, vh, x2, x3);
                            }
                            wave_scan128(hl, hh);
                            wave_scan128(vl, vh);
                            const u64 x = wave_scan(state >> 32);
                            if (GS) parents = wave_scan(parents);
                            const bool flagged = __any(state & 1);
                            if (lane == 63) {
                                red[12] = hl; red[13] = hh; red[14] = vl; red[15] = vh;
                                red[16] = x; red[17] = both; red[18] = flagged;
                                if (GS) red[19] = parents;
                            }
                            max_load = max(max_load, load_of(state));
                            row_due = true;
                        }
                        if (s_go != 2) break;
                    }
                } else {
                    if (init != (ph == 2)) continue;
                    if (init) {
                        __syncthreads();
                        for (int s = tid; s < slots; s += BS)
                            L.occ[s] = (W == 1 ? L.k0[s] != EMPTY : L.state[s] == 2u) ? 1 : 0;
                        __syncthreads();
                    }
                }
                // the registers hold the survivors of all buckets: not for a
                // batch of some of them, which reads its own from the table
                const bool table = ph == 1, regs = table && held && k0 == 0 && k1 == K;
                if (wid == 0) continue;
                const int *pre = table ? pt : ps;
                const int end = pre[k1];
                int i = pre[k0] + tid - 64;
                bool have = regs ? hc != 0.0 : i < end;
#pragma unroll 1
                while (have) {
                    u64 a0, a1 = 0;
                    double v;
                    bool ok = true, ni = false;
                    int k = k0;
                    if (regs) {
                        a0 = h0;
                        if (W == 2) a1 = h1;
                        v = hc;
                    } else {
                        for (int hi = k1; hi - k > 1;) {
                            const int mid = (k + hi) >> 1;
                            if (pre[mid] <= i) k = mid;
                            else hi = mid;
                        }
                        const int j = i - pre[k];
                        const i64 b = bA + k;
                        if (table) {
                            const i64 e = b * I.cap_t + j;
                            a0 = gmem(I.tab_a[p][0])[e];
                            if (W == 2) a1 = gmem(I.tab_a[p][1])[e];
                            v = gmem(I.tab_v[p])[e];
                        } else {
                            res_load_rec<W>(I.rec, I.slab[p1] + b * I.cap_s * (i64)I.rec, j, a0, a1, v);
                            ni = ((W == 1 ? a0 : a1) & I.iflag) != 0;
                            ok = !ni;
                            if (W == 1) a0 &= ~I.iflag;
                            else a1 &= ~I.iflag;
                        }
                    }
                    if (table) {
                        const T a = AddrOf<W>::make(a0, a1);
                        double hii;
                        if (MODEL == 0 || MODEL == 3)
                            hii = narrow ? real_diag_runs<u32>(I.mc, (u32)a0) : real_diag_runs(I.mc, a);
                        else hii = narrow ? mom_diag_modes<u32>(I.mc, (u32)a0) : mom_diag_modes(I.mc, a);
                        const double gd = 1.0 + I.dtau * (S - hii);
                        v = v * gd;
                        if (EARLY && fabs(v) < I.theta)
                            v = compress1(v, I.theta, draw(I.seed, a0, a1, (u32)(n + 1), 2u, 0u).x);
                        ok = v != 0.0 || init;
                    }
                    lds_add_n<W, 1>(L, I, &a0, &a1, &v, &ok, bA + k, np, inx);
                    if (init && ph == 2) lds_add_occupied<W, 1>(L, I, &a0, &a1, &v, &ni, bA + k, inx);
                    i += BS - 64;
                    have = !regs && i < end;
                }
            }
            if (s_go != 2) {
                if (OV && ov_step >= 0) write_overlaps();
                break;
            }
            __syncthreads();
            if (s_full && (slots < SLOTS || (!GS && most > SLOTS && k1 - k0 > 1))) {
                // more addresses than expected: again with the whole hash,
                // then with fewer buckets
                if (slots == SLOTS) most = SLOTS;
                redo = 1;
                __syncthreads();
                continue;
            }
            redo = 0;
            if (s_full && tid == 0) fail(I, L, FQE_CAP_LDS, bA + k0);
            // (the second run of two comes back here after its projection)
            int nS = 0;
            i64 A = 0;
            const u32 step1 = (u32)(n + 1);
#pragma unroll 1
            for (int pass = 0;; pass++) {
                const bool final = !second || pass == 1;
                // ------------------------------------------------ 2. occupied slots
                // an index of them, so that the sums, draws and conversions run
                // on full waves
#pragma unroll 1
                for (int s = tid; s < slots; s += BS) {
                    const bool occ = W == 1 ? L.k0[s] != EMPTY : L.state[s] == 2u;
                    const u64 m = __ballot(occ);
                    int at = 0;
                    if (lane == 0 && m) at = atomicAdd(&s_list, __popcll(m));
                    at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1));
                    if (occ) list[at] = (unsigned short)s;
                }
                __syncthreads();
                // ------------------------------------------------ 3. compress, survivors and their attempts
                const int nU = s_list, kb = k1 - k0;
                distinct += nU;
                Fx3 pn = fx3_zero();  // norm after the projection
                int pinx = 0, povf = 0;
                whole = k0 == 0 && k1 == K;
                held = whole && nU <= BS - 64;
                u64 sum = 0;  // survivors from bit 48, attempts below
                u64 nlo = 0, nhi = 0;
                int odd = 0;
                hc = 0.0;
#pragma unroll 1
                for (int j0 = -64; j0 + 64 < nU; j0 += BS - 64, odd ^= 16) {
                    const bool occ = wid > 0 && j0 + tid < nU;
                    int s = 0, bl = 0, pos = 0;
                    u64 a0 = 0, a1 = 0;
                    double c = 0.0;
                    u32 att = 0;
                    if (occ) {
                        s = list[j0 + tid];
                        a0 = L.k0[s];
                        if (W == 2) a1 = L.k1[s];
                        c = GS && pass == 1 ? bitsd(L.lo[s]) : from_fixed(L.lo[s], L.hi[s]);
                        if (!EARLY && !(GS && pass == 1) && c != 0.0 && fabs(c) < I.theta)
                            c = compress1(c, I.theta, draw(I.seed, a0, a1, step1, 1u, 0u).x);
                        L.lo[s] = dbits(c);
                        if (kb > 1) bl = (int)bucket_index(AddrOf<W>::make(a0, a1), I.log2B, I.mc.nb <= 32) - (bA + k0);
                    }
                    const bool alive = c != 0.0;
                    bool exact = false;
                    if (alive) {
                        int bad = 0;
                        if (final) spawn_info<W, MODEL>(I, AddrOf<W>::make(a0, a1), c, att, exact, bad);
                        if (bad) fail(I, L, FQE_ATTEMPTS, bA + k0 + bl);
                        if (GS && pass == 1) {
                            fx3_add(pn, to_fx3(fabs(c), pinx, povf));
                        } else {
                            u64 lo, hi;
                            int ovf = 0;
                            to_fixed(fabs(c), lo, hi, ovf, inx);
                            add128(nlo, nhi, lo, hi);
                        }
                    }
                    {
                        const u64 em = __ballot(exact);
                        if (lane == 0 && em) atomicAdd(&s_ex, __popcll(em));
                    }
                    // rank inside the bucket: one LDS atomic per wave for a few
                    // buckets, else one per lane
                    if (kb <= 4) {
#pragma unroll 1
                        for (int b = 0; b < kb; b++) {
                            const u64 um = __ballot(occ && bl == b), lm = __ballot(alive && bl == b);
                            int at = 0;
                            if (lane == 0) {
                                if (um && pass == 0) atomicAdd(&used[k0 + b], __popcll(um));
                                if (lm) at = atomicAdd(&keep[k0 + b], __popcll(lm));
                            }
                            at = __builtin_amdgcn_readfirstlane(at);
                            if (alive && bl == b) pos = at + __popcll(lm & ((1ull << lane) - 1));
                        }
                    } else {
                        if (occ && pass == 0) atomicAdd(&used[k0 + bl], 1);
                        if (alive) pos = atomicAdd(&keep[k0 + bl], 1);
                    }
                    if (alive && final && pos < I.cap_t) {
                        const i64 e = (i64)(bA + k0 + bl) * I.cap_t + pos;
                        gmem(I.tab_a[1 - p][0])[e] = a0;
                        if (W == 2) gmem(I.tab_a[1 - p][1])[e] = a1;
                        gmem(I.tab_v[1 - p])[e] = c;
                    }
                    u64 total;
                    const u64 at = sum + res_scan(alive ? ((u64)1 << 48) + att : 0, (u64 *)L.misc + odd, total);
                    sum += total;
                    if (alive) {
                        live[at >> 48] = (unsigned short)s;
                        off[at >> 48] = (u32)at;
                    }
                    h0 = a0;
                    h1 = a1;
                    hc = c;
                }
                if (tid == 0) L.misc[60] = 0;
                __syncthreads();
                nS = (int)(sum >> 48);
                A = (i64)(sum & (((u64)1 << 48) - 1));
                // ------------------------------------------------ 4. projected energy
                u64 hlo = 0, hhi = 0, vlo = 0, vhi = 0;
                if (pass == 0) {
                    const int e0 = I.ref_off[bA + k0], e1 = I.ref_off[bA + k1];
#pragma unroll 1
                    for (int e = ref_held ? ref0 + BS - 1 - tid : e0 + tid; e < e1; e += BS) {
                        if (e >= e0) {
                            const u64 a0 = ref_held ? f0 : gmem(I.ref_a[0])[e];
                            const u64 a1 = W == 1 ? 0 : ref_held ? f1 : gmem(I.ref_a[1])[e];
                            const double rh = ref_held ? fh : gmem(I.ref_h)[e];
                            const int s = lds_find<W>(L, a0, a1, slot_hash(a0, a1));
                            const double cv = s >= 0 ? bitsd(L.lo[s]) : 0.0;
#pragma unroll 1
                            for (int r = 0; r < (e == I.ref_self ? 2 : 1); r++) {
                                u64 lo, hi;
                                int ovf = 0;
                                to_fixed(r ? I.yref * cv : I.yref * (rh * cv), lo, hi, ovf, inx);
                                if (r) add128(vlo, vhi, lo, hi);
                                else add128(hlo, hhi, lo, hi);
                            }
                        }
                        if (ref_held) break;
                    }
                }
                // the wave's sums, limb by limb
                auto limbs = [&](u64 *w, u64 &lo, u64 &hi) {
                    wave_scan128(lo, hi);
                    if (lane == 63) {
                        atomicAdd(&w[0], lo & 0xffffffffull);
                        atomicAdd(&w[1], lo >> 32);
                        atomicAdd(&w[2], hi & 0xffffffffull);
                        atomicAdd(&w[3], hi >> 32);
                    }
                };
                if (__any((nlo | nhi) != 0)) limbs(red, nlo, nhi);
                if (__any((hlo | hhi | vlo | vhi) != 0)) {
                    limbs(red + 4, hlo, hhi);
                    limbs(red + 8, vlo, vhi);
                }
                // capacities as the step kernels hold them
                if (tid >= k0 && tid < k1) {
                    const int u = used[tid];
                    if (keep[tid] > I.cap_t) fail(I, L, FQE_CAP_TABLE, bA + tid);
                    if (u > I.slots) fail(I, L, FQE_CAP_LDS, bA + tid);
                    atomicMax(&s_load, u);
                    if (final) I.tab_n[1 - p][bA + tid] = keep[tid];
                }
                if (!GS) break;
                // ------------------------------------------------ projection
                if (pass == 1) {
                    if (pinx) atomicOr(&O.flags[0], 1);
                    if (povf) fail(I, L, FQE_DIVERGED, bA);
                    Fx3 *tmp = (Fx3 *)L.misc;
                    static_assert(sizeof(Fx3) * (BS / 64) <= 60 * 8, "beside misc[60]");
                    wave_scan_fx3(pn);
                    __syncthreads();
                    if (lane == 63) tmp[wid] = pn;
                    __syncthreads();
                    if (wid == 0) {
                        pn = lane < BS / 64 ? tmp[lane] : fx3_zero();
                        wave_scan_fx3(pn);
                        if (lane == 63) norms[g] = pn;
                    }
                    break;
                }
                if (tid == 0) s_len = nS;
                __syncthreads();
                if (tid == 0 && (s_full || s_fail))
                    __hip_atomic_store(&Y->abort[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                res_barrier(Y, meet, ++met, s_where);
                if (tid == 0) s_abort = (int)res_load(&Y->abort[0]);
                __syncthreads();
                if (s_abort) break;
                const Inst &IJ = const_inst(O.rep[0]);
                if (second) {
                    // (s_list: the addresses of the hash)
                    resident_dot<W>(I, L, IJ, 1 - s_par[0], bA, K, (int *)off, O.flags, O.part + 2 * g, &s_list);
                    if (tid == 0 && s_list > SLOTS)
                        __hip_atomic_store(&Y->abort[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                res_barrier(Y, meet, ++met, s_where);
                // (wave 1: resident_project sums the dot products in wave 0)
                if (tid == 64) s_abort = (int)res_load(&Y->abort[1]);
                if (second)
                    resident_project<W>(I, L, IJ, 1 - s_par[0], bA, K, G, (const int *)off, O.part, &s_alpha, &s_abort);
                __syncthreads();
                if (s_abort || !second) break;
                if (tid == 0) s_list = 0;
                if (tid < K) keep[tid] = 0;
                distinct = 0;
                __syncthreads();
            }
            if (GS && s_abort) break;
            // ------------------------------------------------ 5. spawn for step n+2
            if (row_due) write_row();
            if (OV && ov_step >= 0) write_overlaps();
            if (A < ((i64)1 << 32)) {
                resident_spawn<W, MODEL, EARLY>(I, L, 1 - p, bA, G == 1, step1 + 1u, nS, A, live, off, cnt, base, own,
                                                lut, tri);
            } else if (tid == 0) {
                fail(I, L, FQE_CAP_SLAB, bA + k0);
            }
            if (tid == 0) {
                if (GS) s_live = nS;
                else s_len += nS;
                s_sp += EARLY ? L.misc[60] : A;
            }
            k0 = k1;
            if (k0 < K) __syncthreads();
        }
        if (GS && dead) {
            // the others end at the first barrier of their step
            if (tid == 0) __hip_atomic_store(&Y->abort[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            res_barrier(Y, meet, ++met, s_where);
            break;
        }
        if (s_go != 2 && !dead) break;
        if (GS && s_abort) {
            // the step is undone, with the errors of this launch
            if (g == 0 && tid == 0) {
                __hip_atomic_store(&ctrl->error, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ctrl->err_bucket = 0;
            }
            break;
        }

        // ---------------------------------------------------- 6. partial sums, barrier
        if (__any(inx) && lane == 0) s_inx = 1;
        // the next hash: at most 5/8 full if the addresses are no more
        slots = 8 * distinct <= 5 * BS ? BS : 8 * distinct <= 10 * BS ? 2 * BS : SLOTS;
        few = 8 * distinct <= 5 * SLOTS;
        __syncthreads();
        if (wid == 0) {
            ResPart &x = I.res->part[(round + 1) & 1][g];
            if (lane < 3) {
                const u64 *w = red + 4 * lane;
                u64 *to = lane == 0 ? x.norm : lane == 1 ? x.hproj : x.vproj;
                u64 c = w[0];
                u64 lo = c & 0xffffffffull;
                c = (c >> 32) + w[1];
                lo |= c << 32;
                c = (c >> 32) + w[2];
                to[0] = lo;
                to[1] = (c & 0xffffffffull) | (((c >> 32) + w[3]) << 32);
            }
            if (lane == 63) {
                x.items = ((u64)s_len << 40) + (u64)s_sp;
                if (GS) I.res->parents[(round + 1) & 1][g] = (u64)s_live;
                x.state = (s_inx ? 1 : 0) | (s_fail || dead ? 2 : 0) | (whole ? 0 : 4) | ((u64)s_load << 8) |
                          ((u64)s_ex << 32);
            }
        }
        if (wid == 1 && lane < K && !dead) {
            __hip_atomic_store(gmem(&I.slab_n[p][bA + lane]), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // consumed
            if (G == 1)
                __hip_atomic_store(gmem(&I.slab_n[1 - p][lane]), own[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            SpawnPart x{0, 0, 0, 0};
            if (lane == 0) x = SpawnPart{s_ex, (GS ? s_live : s_len) - s_ex, s_sp, 0};
            I.spart[(n + 2) & 1][bA + lane] = x;
        }
        round++;
        res_barrier(Y, meet, ++met, s_where);
        if (JOINT) {
            // the overlaps of step n are published now; the first barrier of a launch publishes none
            if (OV && me == 0 && g == 0 && wid == 0 && round > 1 && !dead) ov_step = n;
            if (tid < O.R) s_par[tid] ^= 1;
            __syncthreads();
        }
        concluded = false;
    }
    // the last completed step
    if (g == 0 && wid == 0) {
        if (row_due) write_row();
#pragma unroll 1
        for (int o = 32; o > 0; o >>= 1) max_load = max(max_load, __shfl_xor(max_load, o, 64));
        if (lane == 0) {
            ctrl->step = n;
            ctrl->parity = p;
            ctrl->shift = S;
            ctrl->norm = N0;
            ctrl->inexact_in = row_inx;
            ctrl->first_inexact = first_inx;
            if ((u32)max_load > ctrl->max_load) ctrl->max_load = (u32)max_load;
        }
    }
}

}  // namespace fq
