// Tree walk for gfx950 (Sec. 3.1 opening criteria and box rule, Sec. 3.2
// spline softening, Sec. 3.4 short-range truncation and cutoff).
//
// One wavefront walks the depth-first entry list for 64 active particles that
// are adjacent on the Peano-Hilbert curve.  The wave keeps ONE cursor: every
// lane owns a "next" index (the entry its own depth-first walk needs next,
// or an earlier one while it is inside a cube it opened); lanes whose next
// is at or before the cursor evaluate the entry, lanes that accepted or
// discarded an ancestor sit out until the cursor reaches their next.  The
// cursor descends (c + 1) when any lane opens the entry and otherwise jumps
// to the entry's skip pointer -- the next entry of some lane's walk, since
// subtrees nest.  Entries are read with wave-uniform (scalar) loads, so each
// lane sees exactly the entry sequence of its own recursive walk, in order:
// the FP64 path reproduces a sequential FP64 walk bit for bit apart from the
// last bits of erfc/exp.  With a cutoff, entries that can interact with no
// lane of the wavefront are skipped (particles of opened leaf parents beyond
// r_cut of the group's bounding box, cubes every lane discards).
#include "walk_device.h"

#include <algorithm>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

namespace tpm {
namespace {

using namespace wk;

// The wavefronts of one workgroup of the group walks.  Divided walks: the
// workgroup holds all shares of its groups (four wavefronts, eight for eight
// shares) and adds them up.
__host__ __device__ constexpr uint32_t group_waves(uint32_t shares) { return shares > 4u ? 8u : 4u; }

template <int WAVES>
__device__ __forceinline__ void clear_arrived(uint32_t *arrived) {
    if (threadIdx.x < WAVES)
        arrived[threadIdx.x] = 0u;
    __syncthreads();
}

template <bool SHARED, bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
__device__ __forceinline__ void group64(const WalkArgs &A) {
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (SHARED) {
        __shared__ GroupLds64 lds[kShareWaves64];
        __shared__ uint32_t arrived[kShareWaves64];
        clear_arrived<kShareWaves64>(arrived);
        walk_group64<kOneShare, PER, TPM, OPEN, POT, MIXED>(
            A, wave_id(), &lds[w].q, nullptr, &lds[w], arrived + (w >> A.shares_log));
    } else {
        IQ64 *Q = nullptr;  // the interaction queue, with a cutoff
        if constexpr (TPM) {
            __shared__ IQ64 q[kBlock / 64];
            Q = &q[w];
        }
        walk_group64<kWhole, PER, TPM, OPEN, POT, MIXED>(A, wave_id(), Q);
    }
}

template <bool SHARED, bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
__device__ __forceinline__ void group32(const WalkArgs &A) {
    if constexpr (SHARED) {
        const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        __shared__ GroupLds32 lds[kShareWaves32];
        __shared__ uint32_t arrived[kShareWaves32];
        clear_arrived<kShareWaves32>(arrived);
        walk_group32<kOneShare, PER, TPM, OPEN, POT, MIXED>(
            A, wave_id(group_waves(A.shares)), nullptr, &lds[w], arrived + (w >> A.shares_log));
    } else {
        walk_group32<kWhole, PER, TPM, OPEN, POT, MIXED>(A, wave_id());
    }
}

// With a cutoff held to 64 VGPRs (66 without the bound): eight wavefronts per
// SIMD, 7.18 -> 6.64 ms for the geometric pass over 128^3 clustered particles
// (six where potentials or individual softening need more registers).  Scalar
// registers spill into lanes of a vector register there; nothing goes to memory.
template <bool SHARED, bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(!TPM ? 4 : POT || MIXED ? 6 : 8))) void
k_walk64(const WalkArgs A) {
    group64<SHARED, PER, TPM, OPEN, POT, MIXED>(A);
}

template <bool SHARED, bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
__global__ __launch_bounds__(SHARED ? kShareWaves32 * 64 : kBlock) void k_walk32(const WalkArgs A) {
    group32<SHARED, PER, TPM, OPEN, POT, MIXED>(A);
}

// Sparse active sets: a census counts the compact groups (group_compact),
// then one of two launches walks every group -- with the shared cursor when
// at least half of the groups are compact (a set of dense clumps, as the
// deepest time bins are), with independent lanes otherwise; the other launch
// returns at once.  The two walks give the same results.
// Measured, relative walk, shared cursor against lanes (both in shares).
// Clustered 256^3 box, FP32: the densest 1 % 0.58 against 0.93 ms, random 3 %
// of 128^3 1.00 against 0.71.  Hernquist sphere of 2^20, FP32: the densest 10 %
// 0.80 against 1.55, the densest 2 % 0.63 against 1.11, random 20 % 1.03
// against 1.46, 10 % 0.97 against 1.16, 7 % 1.06 against 1.03, 5 % 0.98 against
// 0.76; of 2^18 (eight shares) random 20 % 0.54 against 0.71, 10 % 0.63 against
// 0.47.  With an isolated mesh the cutoff spans many such groups, so both tests
// apply; FP64, Hernquist sphere of 2^20, 64^3 mesh: random 2 % 2.50 against 1.44 (the
// geometric pass 3.98 against 1.95), 5 % 2.31 against 1.81, 10 % 2.29 against 2.74, the
// densest 2 % 2.21 against 2.75.
// (Choosing per group inside one kernel made its lane walk slower: 7.6
// against 6.0 ms on a random 10 % of the box.)
template <bool PER, bool TPM>
__global__ __launch_bounds__(kBlock) void k_census(const WalkArgs A, uint32_t *census) {
    const uint32_t wave = wave_id();
    if (wave * 64u >= load_count(A.nuniq))
        return;
    if (group_compact<PER, TPM>(A, wave) && (threadIdx.x & 63) == 0)
        atomicAdd(census, 1u);
}

__device__ __forceinline__ bool mostly_compact(const WalkArgs &A) {
    const uint32_t groups = (load_count(A.nuniq) + 63u) / 64u;
    return 2ull * load_count(A.census) >= groups;
}

template <bool SHARED, bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(!TPM ? 4 : POT || MIXED ? 6 : 8))) void
k_walk64m(const WalkArgs A) {
    if (mostly_compact(A))
        group64<SHARED, PER, TPM, OPEN, POT, MIXED>(A);
}

template <bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
__global__ __launch_bounds__(kBlock) void k_walk64im(const WalkArgs A) {
    if (!mostly_compact(A))
        walk_lanes64<kOneShare, PER, TPM, OPEN, POT, MIXED>(A, lane_wave_id<PER>());
}

template <bool SHARED, bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
__global__ __launch_bounds__(SHARED ? kShareWaves32 * 64 : kBlock) void k_walk32m(const WalkArgs A) {
    if (mostly_compact(A))
        group32<SHARED, PER, TPM, OPEN, POT, MIXED>(A);
}

template <bool SHARED, bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
__global__ __launch_bounds__(kBlock) void k_walk32im(const WalkArgs A) {
    if (!mostly_compact(A))
        walk_lanes32<SHARED ? kOneShare : kWhole, PER, TPM, OPEN, POT, MIXED>(A, lane_wave_id<PER>());
}

// one wavefront per target (sparse active sets)
template <bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
__global__ __launch_bounds__(kBlock) void k_walk64s(const WalkArgs A) {
    __shared__ uint32_t front[kBlock / 64][kFrontWords];
    walk_lanes64<kWhole, PER, TPM, OPEN, POT, MIXED, true>(A, wave_id(),
                                                              front[threadIdx.x >> 6]);
}

template <bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
__global__ __launch_bounds__(kBlock) void k_walk32s(const WalkArgs A) {
    __shared__ uint32_t front[kBlock / 64][kFrontWords];
    walk_lanes32<kWhole, PER, TPM, OPEN, POT, MIXED, true>(A, wave_id(),
                                                              front[threadIdx.x >> 6]);
}

// ---- active set -> slots in curve order --------------------------------------

__global__ __launch_bounds__(kBlock) void k_mark(const int32_t *__restrict__ idx, int64_t n_act,
                                                 int64_t n, const int32_t *__restrict__ rank,
                                                 uint8_t *__restrict__ mark, uint8_t epoch) {
    int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n_act)
        return;
    const int32_t i = idx[k];
    if (i < 0 || (int64_t)i >= n)
        return;  // reported by the output kernel
    mark[rank[i]] = epoch;
}

// Small trees: the slots of the active set in one launch by one workgroup (marks
// in LDS, then ranked) instead of four that are shorter than their gaps (mark,
// count, compact and, after a build, clear: 20 us against 6).  The marks in
// memory are cleared when the call asks for it, as later calls on the context
// rely on.  One workgroup reads a long list with many duplicates slower than the
// chip does: whole calls for 16384, 32768 and 65536 entries 47, 52 and 63 us against
// 51 in four launches (512 particles), 77, 83 and 96 against 87 (4096).
constexpr int kSelBlock = 1024;
constexpr int64_t kSelN = 8192;       // particles
constexpr int64_t kSelActive = 16384;  // entries of the active list
__global__ __launch_bounds__(kSelBlock) void k_select_small(
    const int32_t *__restrict__ idx, int n_act, int n, const int32_t *__restrict__ rank,
    uint8_t *__restrict__ mark, int clear, uint32_t *__restrict__ act,
    uint32_t *__restrict__ slot, uint32_t *__restrict__ d_total) {
    __shared__ uint8_t s_m[kSelN];
    __shared__ uint32_t s_w[kSelBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int r = tid; r < n; r += kSelBlock) {
        s_m[r] = 0;
        if (clear)
            mark[r] = 0;
    }
    __syncthreads();
    for (int k = tid; k < n_act; k += kSelBlock) {
        const int32_t i = idx[k];
        if (i >= 0 && i < n)
            s_m[rank[i]] = 1;  // out-of-range indices: reported by the output kernel
    }
    __syncthreads();
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    uint32_t pos = 0u;
    for (int base = 0; base < n; base += kSelBlock) {
        const int r = base + tid;
        const bool f = r < n && s_m[r];
        const uint64_t m = __ballot(f);
        if (lane == 0)
            s_w[w] = (uint32_t)__popcll(m);
        __syncthreads();
        uint32_t before = 0u, all = 0u;
        for (int q = 0; q < kSelBlock / 64; q++) {
            before += q < w ? s_w[q] : 0u;
            all += s_w[q];
        }
        if (f) {
            const uint32_t p = pos + before + (uint32_t)__popcll(m & lt);
            act[p] = (uint32_t)r;
            slot[r] = p;
        }
        pos += all;
        __syncthreads();
    }
    if (tid == 0)
        *d_total = pos;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_output(
    const int32_t *__restrict__ idx, int64_t n_act, int64_t n, const int32_t *__restrict__ rank,
    const uint32_t *__restrict__ slot, const uint32_t *__restrict__ nuniq,
    const T *__restrict__ res, const T *__restrict__ rpot, T *__restrict__ acc,
    T *__restrict__ pot, uint32_t *__restrict__ nint, uint32_t *__restrict__ err) {
    int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n_act)
        return;
    const int32_t i = idx[k];
    if (i < 0 || (int64_t)i >= n) {
        const T nan = (T)NAN;
        acc[k] = nan;
        acc[n_act + k] = nan;
        acc[2 * n_act + k] = nan;
        if (pot)
            pot[k] = nan;
        if (nint)
            nint[k] = 0xffffffffu;
        atomicOr(err, 1u);
        return;
    }
    // the slot's record: acceleration and interaction count together (with
    // every particle active the slots are the ranks, and the lookup is skipped)
    const uint32_t rk = (uint32_t)rank[i];
    const uint32_t sl = *nuniq == (uint32_t)n ? rk : slot[rk];
    const T *r = res + 4 * (size_t)sl;
    acc[k] = r[0];
    acc[n_act + k] = r[1];
    acc[2 * n_act + k] = r[2];
    if (pot)
        pot[k] = rpot[sl];
    if (nint)
        nint[k] = count_of(r[3]);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_accel_norm(const int32_t *__restrict__ idx,
                                                       int64_t n_act, int64_t n,
                                                       const T *__restrict__ a,
                                                       const T *__restrict__ b,
                                                       double *__restrict__ out,
                                                       uint32_t *__restrict__ err) {
    int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n_act)
        return;
    const int32_t i = idx[k];
    if (i < 0 || (int64_t)i >= n) {
        atomicOr(err, 1u);
        return;
    }
    double v[3];
#pragma unroll
    for (int d = 0; d < 3; d++) {
        v[d] = (double)a[d * n_act + k];
        if (b)
            v[d] += (double)b[d * n_act + k];
    }
    out[i] = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
}

struct Launch {
    bool fp32;
    Variant variant;
    unsigned blocks;
    unsigned lane_blocks;    // kGroupOrLanes: of the lane walk
    unsigned census_blocks;  // and of the census
};

// Undivided lanes have an instance of their own in FP32, where the geometric pass
// always is (random 2 to 10 % of Hernquist spheres, 1.53 -> 1.47 to 1.72 -> 1.60 ms); the
// FP64 one was slower (10 % of 2^20 with a mesh: 2.90 -> 3.48).
template <bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
void launch_lanes(const WalkArgs &A, bool fp32, unsigned blocks, hipStream_t st) {
    if (!fp32)
        k_walk64im<PER, TPM, OPEN, POT, MIXED><<<blocks, kBlock, 0, st>>>(A);
    else if (A.shares > 1u)
        k_walk32im<OPEN == TPM_OPEN_REL, PER, TPM, OPEN, POT, MIXED><<<blocks, kBlock, 0, st>>>(A);
    else
        k_walk32im<false, PER, TPM, OPEN, POT, MIXED><<<blocks, kBlock, 0, st>>>(A);
}

template <bool PER, bool TPM, int OPEN, bool POT, bool MIXED>
void launch_walk(const WalkArgs &A, const Launch &L, hipStream_t st) {
    if (L.variant == kSplitWalk) {
        if (L.fp32)
            k_walk32s<PER, TPM, OPEN, POT, MIXED><<<L.blocks, kBlock, 0, st>>>(A);
        else
            k_walk64s<PER, TPM, OPEN, POT, MIXED><<<L.blocks, kBlock, 0, st>>>(A);
    } else if (L.variant == kLaneWalk) {
        launch_lanes<PER, TPM, OPEN, POT, MIXED>(A, L.fp32, L.blocks, st);
    } else if (L.variant == kGroupOrLanes) {
        k_census<PER, TPM><<<L.census_blocks, kBlock, 0, st>>>(A, (uint32_t *)A.census);
        if (L.fp32) {
            if (A.shares > 1u)
                k_walk32m<OPEN == TPM_OPEN_REL, PER, TPM, OPEN, POT, MIXED>
                    <<<L.blocks, group_waves(A.shares) * 64, 0, st>>>(A);
            else
                k_walk32m<false, PER, TPM, OPEN, POT, MIXED><<<L.blocks, kBlock, 0, st>>>(A);
        } else {
            if (A.shares > 1u)
                k_walk64m<true, PER, TPM, OPEN, POT, MIXED><<<L.blocks, kBlock, 0, st>>>(A);
            else
                k_walk64m<false, PER, TPM, OPEN, POT, MIXED><<<L.blocks, kBlock, 0, st>>>(A);
        }
        launch_lanes<PER, TPM, OPEN, POT, MIXED>(A, L.fp32, L.lane_blocks, st);
    } else {
        if (L.fp32) {
            if (A.shares > 1u)
                k_walk32<OPEN == TPM_OPEN_REL, PER, TPM, OPEN, POT, MIXED>
                    <<<L.blocks, group_waves(A.shares) * 64, 0, st>>>(A);
            else
                k_walk32<false, PER, TPM, OPEN, POT, MIXED><<<L.blocks, kBlock, 0, st>>>(A);
        } else {
            if (A.shares > 1u)
                k_walk64<true, PER, TPM, OPEN, POT, MIXED><<<L.blocks, kBlock, 0, st>>>(A);
            else
                k_walk64<false, PER, TPM, OPEN, POT, MIXED><<<L.blocks, kBlock, 0, st>>>(A);
        }
    }
}

template <bool PER, bool TPM, bool MIXED>
void dispatch_open_pot(const WalkArgs &A, const Launch &L, int open, bool pot, hipStream_t st) {
    if (open == TPM_OPEN_BH) {
        if (pot)
            launch_walk<PER, TPM, TPM_OPEN_BH, true, MIXED>(A, L, st);
        else
            launch_walk<PER, TPM, TPM_OPEN_BH, false, MIXED>(A, L, st);
    } else {
        if (pot)
            launch_walk<PER, TPM, TPM_OPEN_REL, true, MIXED>(A, L, st);
        else
            launch_walk<PER, TPM, TPM_OPEN_REL, false, MIXED>(A, L, st);
    }
}

template <bool PER, bool TPM>
void dispatch_mixed(const WalkArgs &A, const Launch &L, int open, bool pot, bool mixed,
                    hipStream_t st) {
    if (mixed)
        dispatch_open_pot<PER, TPM, true>(A, L, open, pot, st);
    else
        dispatch_open_pot<PER, TPM, false>(A, L, open, pot, st);
}

}  // namespace

int accel_norm(tpm_ctx *c, int64_t n_act, const int32_t *idx, const void *a, const void *b,
               double *out) {
    if (n_act == 0)
        return TPM_OK;
    const unsigned g = grid_for(n_act, kBlock);
    if (c->P.precision == TPM_FP32)
        k_accel_norm<float><<<g, kBlock, 0, c->stream>>>(idx, n_act, c->n, (const float *)a,
                                                         (const float *)b, out,
                                                         (uint32_t *)c->err_flag.p);
    else
        k_accel_norm<double><<<g, kBlock, 0, c->stream>>>(idx, n_act, c->n, (const double *)a,
                                                          (const double *)b, out,
                                                          (uint32_t *)c->err_flag.p);
    TPM_LAUNCHED(c, "k_accel_norm");
    return TPM_OK;
}

int work_of_ctx(tpm_ctx *c, bool results, Work &w) {
    const int64_t n = c->n;
    TPM_TRY(ensure(c, c->mark, mark_bytes(n)));
    TPM_TRY(ensure(c, c->act, (size_t)n * 4));
    TPM_TRY(ensure(c, c->slot, (size_t)n * 4));
    TPM_TRY(ensure(c, c->scan_tmp, (size_t)compaction_tiles(n) * 4));
    if (results) {
        const size_t esz = c->P.precision == TPM_FP32 ? 4 : 8;
        TPM_TRY(ensure(c, c->res, (size_t)4 * n * esz));
        TPM_TRY(ensure(c, c->rpot, (size_t)n * esz));
    }
    w = Work{};
    w.mark = (uint8_t *)c->mark.p;
    w.clear = c->epoch == 0 || c->epoch == 255;  // fresh, or every mark was used
    w.epoch = w.clear ? 1 : (uint8_t)(c->epoch + 1);
    w.last = &c->epoch;
    w.act = (uint32_t *)c->act.p;
    w.slot = (uint32_t *)c->slot.p;
    w.counts = (uint32_t *)c->scan_tmp.p;
    w.nuniq = (uint32_t *)c->counters.p + 40;
    w.res = c->res.p;
    w.rpot = c->rpot.p;
    return TPM_OK;
}

int select_active_into(tpm_ctx *c, int64_t n_act, const int32_t *idx, const Work &w) {
    const int64_t n = c->n;
    hipStream_t st = c->stream;
    if (n <= kSelN && n_act <= kSelActive) {
        k_select_small<<<1, kSelBlock, 0, st>>>(idx, (int)n_act, (int)n,
                                                (const int32_t *)c->rank.p, w.mark, w.clear, w.act,
                                                w.slot, w.nuniq);
        TPM_LAUNCHED(c, "k_select_small");
        marks_queued(w);
        return TPM_OK;
    }
    if (w.clear)
        TPM_TRY(fill_u32(c, (uint32_t *)w.mark, 0u, (int64_t)(mark_bytes(n) / 4)));
    marks_queued(w);
    if (n_act > 0) {
        k_mark<<<grid_for(n_act, kBlock), kBlock, 0, st>>>(idx, n_act, n,
                                                           (const int32_t *)c->rank.p, w.mark,
                                                           w.epoch);
        TPM_LAUNCHED(c, "k_mark");
    }
    return compact_marked(c, w.mark, w.epoch, n, w.act, w.slot, w.nuniq, w.counts);
}

int select_active(tpm_ctx *c, int64_t n_act, const int32_t *idx) {
    Work w;
    TPM_TRY(work_of_ctx(c, false, w));
    return select_active_into(c, n_act, idx, w);
}

// The geometric pass over a sparse set of an isolated system in FP64: thousands
// of interactions for each target, and every share repeats the steps of the upper
// tree, so in lanes, one share each, shares stop paying early.  ms for 1, 2, 4
// shares, random | densest set (lanes | shared cursor): Hernquist 2^20, 4 % 2.04 1.65 1.97
// | 2.41 1.62 1.26, 6 % 2.04 1.83 2.87 | 2.11 1.64 1.32, 7.5 % 2.05 2.23 3.25 | 2.10 1.72
// 1.45; 2^22, 2 % 2.51 3.17 5.00 | 2.29 2.04 2.14, 4 % 3.73 5.33 9.42 | 2.68 3.00 3.37.  From a
// twelfth of the particles on, random sets too are compact on the curve (768
// particles for 64 targets) and take the shared cursor (10 % of 2^20: 2.96 2.57 2.13 |
// 2.45 1.97 1.65).
// With a mesh the cutoff spans tens of length units, and undivided lanes win from
// there on whatever the set (2^20, 64^3 mesh, lanes | shared cursor at the better of the
// two: 5 % random 2.44 | 3.48, densest 2.45 | 2.38; 10 % 2.86 | 3.60, 3.05 | 3.25; 2^21, 9 %
// 3.71 | 5.54, 3.85 | 4.97).
// With individual softening, whose interactions cost more, four shares pay as
// elsewhere (2^20, 10 % 4.48 3.36 2.75 | 3.24 2.57 2.21).
constexpr int64_t kGeoShares4 = 49152, kGeoShares2 = 98304;
static bool sparse_geometric(const tpm_ctx *c, int64_t n_act, int opening) {
    return !c->P.periodic && !c->mixed && opening == TPM_OPEN_BH && 4 * n_act < c->n;
}
// In FP32 that pass is undivided (below), and up to here lanes fill the chip
// better than groups.  Without a mesh, lanes | shared cursor: Hernquist 2^18, 10 %
// random 1.34 | 1.93, densest 1.28 | 1.41; 2^20, 10 % 1.64 | 2.14, 1.59 | 1.77, 20 %
// 2.30 | 1.89, 2.21 | 2.19; 2^22, the densest 3 % 1.82 | 1.91, 4 % 1.95 | 1.81.
constexpr int64_t kGeoLanes32 = 131072;

// Walk variant.  Independent lanes (results identical to the shared cursor)
// for sparse active sets whose groups are too spread out for a shared cursor
// (it would visit the union of their walks); the shared cursor otherwise.
// One wavefront per target for active sets
// of at most 4096 targets (16384 of a quarter or more of
// all particles, in FP64 with a cutoff), and of at most 65536 in
// trees of 2^22 particles or more: with that few wavefronts a lane's serial walk (the longest, which
// grows with the tree) is the critical path, while the frontier walk spreads
// each target over its wavefront and fills the chip.  Measured, FP32
// relative walk, lanes against one wavefront per target: the densest targets
// of the clustered 256^3 box, 16777 targets 1.41 / 0.35 ms, 41943: 1.41 /
// 0.75, 83886: 1.46 / 1.28, 167772: 1.73 / 2.41 (FP64 even at 84 k); the
// 4096-particle Plummer sphere 0.74 -> 0.32 ms.  In smaller trees the lane
// walks are short and the frontier walk's larger work per target loses
// (block steps of a 2^18 Hernquist sphere with sets up to 65536: 15.6 ms
// against 25.5 ms for the integration; the serving mix, up to 2^21
// particles per system: half the burst capacity).  In FP64 with a cutoff a
// target's work is bounded by its neighbourhood, and a step costs most where
// few lanes share it; one wavefront per target against the better of the other
// two, relative and geometric pass in us: whole boxes of 20^3 500 418 -> 146 118,
// 25^3 679 547 -> 385 268, 25^3 clustered 501 420 -> 379 318; isolated, 16000 with a
// mesh 578 928 -> 374 611; 16384 of 64,000 clustered 649 540 -> 392 341.  (Sparse sets
// would gain as much, but the shared cursor and the lanes give them the bits of
// the whole set at equal shares.)  Without a cutoff the geometric pass loses beyond 4096
// (8192 of 2^18: 986 -> 1623), and the FP32 geometric pass keeps its order of
// summation there (see set_shares).
// TPM_WALK_MODE (1 shared cursor, 2 lanes, 3 one wavefront per target)
// overrides the choice.
Variant wk::walk_variant(const tpm_ctx *c, int64_t n_act, int opening, bool census_ok) {
    if (c->walk_mode != 0)
        return c->walk_mode == 1 ? kGroupWalk : c->walk_mode == 2 ? kLaneWalk : kSplitWalk;
    const int64_t targets = std::min<int64_t>(n_act, c->n);
    const bool near64 = c->P.precision == TPM_FP64 && c->P.pm_grid > 0 && 4 * n_act >= c->n;
    if (targets <= (near64 ? 16384 : 4096) || (targets <= 65536 && c->n >= (int64_t(1) << 22)))
        return kSplitWalk;
    if (4 * n_act >= c->n)
        return kGroupWalk;
    // a sparse set: as the census of its groups decides
    const bool fp32 = c->P.precision == TPM_FP32, mesh = c->P.pm_grid > 0;
    if (sparse_geometric(c, n_act, opening) &&
        (fp32 ? !mesh && n_act <= kGeoLanes32 : mesh && n_act > kGeoShares4))
        return kLaneWalk;
    return census_ok ? kGroupOrLanes : kLaneWalk;
}

// Shares of a walk over t targets (walk_device.h): with groups of 64, t
// targets keep t / 64 of the chip's 8192 wavefront slots, each for the latency
// of a serial walk (some 400 ns a step at one wavefront per SIMD), so small
// sets are divided until the slots fill.  Milliseconds of the geometric and the
// relative pass for 1, 2, 4, 8, 16 shares:
//   Hernquist 10,000, FP64     1.00 .49 | .67 .35 | .47 .26 | .31 .20 | .26 .18
//   Hernquist 50,000, FP64     1.33 .74 | .99 .62 | .70 .46 | .64 .47 | .76 .64
//   clustered 40^3, FP32        .47 .66 | .33 .42 | .28 .32 | .28 .30 | .33 .35
//   Hernquist 100,000, FP64    1.87 1.66 | 1.41 1.17 | 1.14 .84 | 1.17 .78
//   densest 1 % of 256^3, FP32  1.17 | .73 | .62 | .62 (relative pass)
//   clustered 64^3, FP32        .68 .92 | .63 .78 | .69 .84
//   Hernquist 2^18, FP32       1.20 1.02 | 1.25 .80 | 1.46 .80
//   Zel'dovich 64^3, FP32       .32 .31 | .34 .32 | .39 .37
// and one and two shares beyond 2^18:
//   Hernquist 500,000, FP32    1.90 1.21 | 1.90 1.13
//   with a mesh, 400,000, FP32 1.96 1.79 | 1.92 1.38
//   with a mesh, 300,000, FP64 4.61 3.65 | 4.87 2.96
//   Zel'dovich 70^3, FP64      2.50 5.46 | 2.35 4.81
//   Zel'dovich 80^3, FP32       .99 1.29 |  .99 1.36
//   Hernquist 2^20, FP32       3.43 1.79 | 3.44 2.11
// Blocks of entries give each share some of a group's dense neighbourhood: 256
// entries in a periodic box, where the cutoff bounds the neighbourhood (128
// and 512: within 10 %), an isolated tree's entries over 128, 256 to 4096
// (Hernquist 50,000 in FP64: blocks of 256, 512, 1024, 2048 give 1.15, 1.02,
// .98, 1.19 ms for both passes).
// The FP32 geometric pass is not divided: its forces give the |a| by which the
// relative pass opens cubes; summed in another order they differ in the last
// bits, and the few decisions that then change move single forces by up to
// 1.7e-3 (one in five systems of 10^5 particles had one above 8e-4).  In FP64 no
// decision changes.
static uint32_t shares_log(const tpm_ctx *c, int64_t n_act, int opening, Variant v) {
    const int64_t t = std::min<int64_t>(n_act, c->n);
    const bool fp32 = c->P.precision == TPM_FP32, rel = opening == TPM_OPEN_REL;
    if (v == kSplitWalk || (fp32 && !rel))
        return 0u;
    if (sparse_geometric(c, n_act, opening) && (c->P.pm_grid > 0 || 12 * n_act < c->n))  // FP64
        return n_act <= kGeoShares4 ? 2u : n_act <= kGeoShares2 ? 1u : 0u;
    if (t <= 65536 && fp32)
        return 3u;
    if (t <= 196608)
        return 2u;  // (FP64: at most four, the sums that the server's LDS holds)
    if (t <= 262144)
        return 1u;
    return t <= 524288 && rel && !(fp32 && c->P.periodic) ? 1u : 0u;
}

void wk::set_shares(const tpm_ctx *c, int64_t n_act, int opening, Variant v, WalkArgs &A) {
    A.shares_log = shares_log(c, n_act, opening, v);
    A.shares = 1u << A.shares_log;
    A.shares_bh = 1u << shares_log(c, n_act, TPM_OPEN_BH, v);
    A.share_shift = 8;
    if (!c->P.periodic)
        while (A.share_shift < 12u && (c->E >> (A.share_shift + 7)) > 1)
            A.share_shift++;
}

void wk::fill_args(tpm_ctx *c, const double *anorm, const Work &w, WalkArgs &A) {
    const tpm_params &P = c->P;
    const int64_t n = c->n;
    const bool fp32 = P.precision == TPM_FP32;
    A.rec = fp32 ? c->rec32.p : c->rec64.p;
    A.E = (uint32_t)c->E;
    A.n = (uint32_t)n;
    A.act = w.act;
    A.nuniq = w.nuniq;
    A.ps = (const double *)c->ps.p;
    A.qs = (const uint64_t *)c->qs.p;
    A.pe = (const uint32_t *)c->pe.p;
    A.perm = (const int32_t *)c->perm.p;
    A.anorm = anorm;
    A.coherent = 0u;
    A.census = nullptr;
    for (int a = 0; a < 3; a++)
        A.x0[a] = c->frame_host.x0[a];
    A.L = c->frame_host.L;
    A.box = P.periodic ? P.box_size : 0.0;
    A.half = 0.5 * A.box;
    const bool tpm_on = P.pm_grid > 0;
    // split scale r_s = asmth x mesh spacing; the isolated mesh spans the
    // root cube in pm_grid - 4 cells
    double rs = 1.0;
    if (tpm_on)
        rs = P.periodic ? P.asmth * P.box_size / P.pm_grid
                        : P.asmth * (c->frame_host.L / (P.pm_grid - 4));
    const double rcut = tpm_on ? P.rcut * rs : 0.0;
    A.G = P.G;
    A.theta2 = P.theta * P.theta;
    A.alpha = P.alpha;
    A.h = 2.8 * P.eps;
    A.hinv = 1.0 / A.h;
    A.h3inv = A.hinv * A.hinv * A.hinv;
    A.rc2 = rcut * rcut;
    A.inv2rs = 0.5 / rs;
    // unit of the shifted integer coordinates of the FP32 records
    A.fu = (float)ldexp(A.L, -22 - (P.periodic ? kRecShiftPer : kRecShiftIso));
    A.fL = (float)A.L;
    A.ftheta2 = (float)A.theta2;
    A.falpha = (float)A.alpha;
    A.fh2 = (float)(A.h * A.h);
    A.fhinv = (float)A.hinv;
    A.fh3inv = (float)A.h3inv;
    A.frc2 = (float)A.rc2;
    {
        // the prefilter's rounding (positions relative to a group's reference
        // cell, all below L_root in magnitude) stays far below L_root 2^-16
        const double tol = ldexp(A.L, -16);
        A.fpf2 = (float)((rcut + tol) * (rcut + tol));
        A.fpf_ext = P.periodic ? (float)(0.5 * P.box_size - rcut - 2.0 * tol) : 3.0e38f;
        const double tol64 = ldexp(A.L, -40);
        A.pf2 = (rcut + tol64) * (rcut + tol64);
        A.pf_ext = P.periodic ? 0.5 * P.box_size - rcut - 2.0 * tol64 : 1.0e300;
    }
    A.group_ext2 = 0.25 * A.rc2;
    A.finv2rs = (float)A.inv2rs;
    A.fgexp = (float)(-1.4426950408889634 * A.inv2rs * A.inv2rs);
    A.res = w.res;
    A.rpot = w.rpot;
    A.L2r = A.L * A.L;
    A.limr = 0.6 * A.L;
    A.hlr = 0.5 * A.L;
    A.hs = c->mixed ? (const double *)c->hs.p : nullptr;
    A.eh = c->mixed ? (fp32 ? c->eh32.p : c->eh64.p) : nullptr;
    A.fL2r = A.fL * A.fL;
    A.flimr = 0.6f * A.fL;
    A.fhlr = 0.5f * A.fL;
}

int forces(tpm_ctx *c, int32_t opening, int64_t n_act, const int32_t *idx, const double *anorm,
           void *acc, void *pot, uint32_t *nint) {
    if (n_act == 0)
        return TPM_OK;
    Work w;
    TPM_TRY(work_of_ctx(c, true, w));
    return forces_into(c, opening, n_act, idx, anorm, acc, pot, nint, w, true);
}

int forces_into(tpm_ctx *c, int32_t opening, int64_t n_act, const int32_t *idx,
                const double *anorm, void *acc, void *pot, uint32_t *nint, const Work &w,
                bool timed) {
    const tpm_params &P = c->P;
    const int64_t n = c->n;
    hipStream_t st = c->stream;
    const bool fp32 = P.precision == TPM_FP32;
    if (n_act == 0)
        return TPM_OK;
    TPM_TRY(select_active_into(c, n_act, idx, w));

    WalkArgs A{};
    fill_args(c, anorm, w, A);
    const bool tpm_on = P.pm_grid > 0;
    const int64_t groups = (std::min<int64_t>(n_act, n) + 63) / 64;
    Launch LA;
    LA.fp32 = fp32;
    LA.variant = walk_variant(c, n_act, opening, true);
    set_shares(c, n_act, opening, LA.variant, A);
    if (LA.variant == kGroupOrLanes || LA.variant == kLaneWalk) {
        // the census word follows the unique count (no census: no compact group)
        A.census = w.nuniq + 1;
        TPM_TRY(fill_u32(c, w.nuniq + 1, 0u, 1));
    }
    const uint32_t targets = (uint32_t)std::min<int64_t>(n_act, n);
    const uint32_t wg = LA.variant == kLaneWalk ? kBlock / 64 : group_waves(A.shares);
    LA.blocks = (walk_waves(LA.variant, targets, A.shares) + wg - 1) / wg;
    LA.lane_blocks = (walk_waves(kLaneWalk, targets, A.shares) + 3) / 4;
    LA.census_blocks = (unsigned)((groups + 3) / 4);
    const bool want_pot = pot != nullptr && P.want_potential;
    const int tkind = opening == TPM_OPEN_REL ? TPM_TIMER_WALK_REL : TPM_TIMER_WALK;
    if (timed)
        TPM_TRY(timer_begin(c, tkind));
    // periodic boxes always carry the mesh (validated at creation)
    if (P.periodic)
        dispatch_mixed<true, true>(A, LA, opening, want_pot, c->mixed, st);
    else if (tpm_on)
        dispatch_mixed<false, true>(A, LA, opening, want_pot, c->mixed, st);
    else
        dispatch_mixed<false, false>(A, LA, opening, want_pot, c->mixed, st);
    TPM_LAUNCHED(c, "k_walk");
    if (timed)
        TPM_TRY(timer_end(c, tkind));
    const unsigned ob = grid_for(n_act, kBlock);
    if (fp32)
        k_output<float><<<ob, kBlock, 0, st>>>(
            idx, n_act, n, (const int32_t *)c->rank.p, w.slot, w.nuniq, (const float *)w.res,
            (const float *)w.rpot, (float *)acc, want_pot ? (float *)pot : nullptr,
            nint, (uint32_t *)c->err_flag.p);
    else
        k_output<double><<<ob, kBlock, 0, st>>>(
            idx, n_act, n, (const int32_t *)c->rank.p, w.slot, w.nuniq, (const double *)w.res,
            (const double *)w.rpot, (double *)acc, want_pot ? (double *)pot : nullptr,
            nint, (uint32_t *)c->err_flag.p);
    TPM_LAUNCHED(c, "k_output");
    return TPM_OK;
}

}  // namespace tpm

// ---- batched walks over many systems (continuous batching) -------------------
//
// One launch per precision walks the groups of every request staged in a
// batch: each request takes the workgroups it needs.  A workgroup runs the same
// per-group code as a single-system launch, so each result is the same whether
// its request runs alone or in a mix.

namespace tpm {
namespace {

struct BatchReq {
    WalkArgs A;
    uint32_t variant;  // bit 0 relative criterion, 1 TreePM, 3 periodic, 4 individual
                       // softening, bits 5-6 the walk variant (wk::Variant)
    uint32_t first;    // first workgroup of the request
};

// The batch kernel holds the shared-cursor and lane walks only; requests
// that take one wavefront per target are launched on their own (inlined
// here, that walk would push the kernel's registers into heavy spills).  FP32: 35
// VGPRs (eight wavefronts per SIMD), FP64: 67 (seven).
constexpr int batch_waves(bool fp32) { return fp32 ? kShareWaves32 : kShareWaves64; }
template <bool FP32>
struct BatchLds {
    typename std::conditional<FP32, GroupLds32, GroupLds64>::type w[batch_waves(FP32)];
    uint32_t arrived[batch_waves(FP32)];
};

template <bool FP32, bool PER, bool TPM, int OPEN, bool MIXED>
__device__ __forceinline__ void batch_group(const WalkArgs &A, uint32_t g, uint32_t var,
                                            BatchLds<FP32> &lds) {
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t *arrived = lds.arrived + (w >> A.shares_log);
    if constexpr (FP32) {
        if (var == kLaneWalk)
            walk_lanes32<OPEN == TPM_OPEN_REL ? kOneShare : kWhole, PER, TPM, OPEN, false, MIXED>(A, g);
        else if (OPEN == TPM_OPEN_REL && A.shares > 1u)
            walk_group32<kOneShare, PER, TPM, OPEN, false, MIXED>(A, g, nullptr, &lds.w[w], arrived);
        else
            walk_group32<kWhole, PER, TPM, OPEN, false, MIXED>(A, g);
    } else {
        if (var == kLaneWalk)
            walk_lanes64<kOneShare, PER, TPM, OPEN, false, MIXED>(A, g);
        else if (A.shares > 1u)
            walk_group64<kOneShare, PER, TPM, OPEN, false, MIXED>(A, g, &lds.w[w].q, nullptr,
                                                                  &lds.w[w], arrived);
        else
            walk_group64<kWhole, PER, TPM, OPEN, false, MIXED>(A, g, &lds.w[w].q);
    }
}

template <bool FP32, int OPEN, bool MIXED>
__device__ __forceinline__ void batch_geometry(const BatchReq &R, uint32_t g, uint32_t lanes,
                                               BatchLds<FP32> &lds) {
    if (R.variant & 8u)  // periodic box (always with the mesh)
        batch_group<FP32, true, true, OPEN, MIXED>(R.A, g, lanes, lds);
    else if (R.variant & 2u)  // isolated TreePM
        batch_group<FP32, false, true, OPEN, MIXED>(R.A, g, lanes, lds);
    else
        batch_group<FP32, false, false, OPEN, MIXED>(R.A, g, lanes, lds);
}

template <bool FP32>
__global__ __launch_bounds__(batch_waves(FP32) * 64) __attribute__((amdgpu_waves_per_eu(4))) void k_walk_batch(
    const BatchReq *__restrict__ reqs, uint32_t nreq) {
    __shared__ BatchLds<FP32> lds;
    clear_arrived<batch_waves(FP32)>(lds.arrived);
    uint32_t lo = 0, hi = nreq;  // the last request that starts at or before this workgroup
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (reqs[mid].first <= blockIdx.x)
            lo = mid;
        else
            hi = mid;
    }
    const BatchReq &R = reqs[lo];
    const uint32_t g = (blockIdx.x - R.first) * batch_waves(FP32) + (threadIdx.x >> 6);
    const uint32_t lanes = (R.variant >> 5) & 3u;  // walk variant
    const bool rel = (R.variant & 1u) != 0, mixed = (R.variant & 16u) != 0;
    if (rel) {
        if (mixed)
            batch_geometry<FP32, TPM_OPEN_REL, true>(R, g, lanes, lds);
        else
            batch_geometry<FP32, TPM_OPEN_REL, false>(R, g, lanes, lds);
    } else {
        if (mixed)
            batch_geometry<FP32, TPM_OPEN_BH, true>(R, g, lanes, lds);
        else
            batch_geometry<FP32, TPM_OPEN_BH, false>(R, g, lanes, lds);
    }
}

}  // namespace
}  // namespace tpm

struct tpm_batch {
    hipStream_t stream = nullptr;
    std::string err;
    struct Pending {
        tpm_ctx *c;
        int32_t opening;
        int64_t n_act;
        const int32_t *idx;
        const double *anorm;
        void *acc;
        uint32_t *nint;
    };
    std::vector<Pending> pend;
    tpm::BatchReq *host = nullptr;  // pinned staging of the request table
    size_t host_cap = 0;
    void *dev = nullptr;            // device request table
    size_t dev_cap = 0;
    hipEvent_t done = nullptr;      // last launch finished: staging reusable
    bool launched = false;
};

using namespace tpm;

static int bfail(tpm_batch *b, int code, const std::string &m) {
    b->err = m;
    return code;
}

#define BHIP(b, expr)                                                        \
    do {                                                                     \
        hipError_t _e = (expr);                                              \
        if (_e != hipSuccess)                                                \
            return bfail((b), _e == hipErrorOutOfMemory ? TPM_ENOMEM : TPM_EDEVICE, \
                         std::string(#expr) + ": " + hipGetErrorString(_e)); \
    } while (0)

extern "C" {

int tpm_batch_create(void *hip_stream, tpm_batch **out) {
    if (!out)
        return TPM_EINVAL;
    *out = nullptr;
    tpm_batch *b = new (std::nothrow) tpm_batch();
    if (!b)
        return TPM_ENOMEM;
    b->stream = (hipStream_t)hip_stream;
    if (hipEventCreateWithFlags(&b->done, hipEventDisableTiming) != hipSuccess) {
        delete b;
        return TPM_ENOMEM;
    }
    *out = b;
    return TPM_OK;
}

int tpm_batch_destroy(tpm_batch *b) {
    if (!b)
        return TPM_EINVAL;
    (void)hipStreamSynchronize(b->stream);
    if (b->host)
        (void)hipHostFree(b->host);
    if (b->dev)
        (void)hipFree(b->dev);
    if (b->done)
        (void)hipEventDestroy(b->done);
    delete b;
    return TPM_OK;
}

const char *tpm_batch_last_error(const tpm_batch *b) { return b ? b->err.c_str() : "NULL batch"; }

int tpm_batch_add(tpm_batch *b, tpm_ctx *c, int32_t opening, int64_t n_act,
                  const int32_t *idx, const double *anorm, void *acc, uint32_t *nint) {
    if (!b)
        return TPM_EINVAL;
    if (!c || !c->built)
        return bfail(b, TPM_ESTATE, "context missing or not built");
    if (opening != TPM_OPEN_BH && opening != TPM_OPEN_REL)
        return bfail(b, TPM_EINVAL, "opening must be TPM_OPEN_BH or TPM_OPEN_REL");
    if (n_act < 0 || n_act > (int64_t(1) << 31) - 1)
        return bfail(b, TPM_EINVAL, "n_act out of range");
    if (n_act > 0 && (!idx || !acc))
        return bfail(b, TPM_EINVAL, "active_idx and acc must not be NULL");
    if (opening == TPM_OPEN_REL && n_act > 0 && !anorm)
        return bfail(b, TPM_EINVAL, "the relative criterion needs a_old_norm");
    for (const auto &p : b->pend)
        if (p.c == c)
            return bfail(b, TPM_EINVAL, "a context may appear once per batch");
    b->pend.push_back({c, opening, n_act, idx, anorm, acc, nint});
    return TPM_OK;
}

int tpm_batch_launch(tpm_batch *b) {
    if (!b)
        return TPM_EINVAL;
    if (b->pend.empty())
        return TPM_OK;
    if (b->launched)
        BHIP(b, hipEventSynchronize(b->done));  // the staging table is free again
    const size_t np = b->pend.size();
    if (b->host_cap < np) {
        if (b->host)
            BHIP(b, hipHostFree(b->host));
        b->host = nullptr;
        BHIP(b, hipHostMalloc((void **)&b->host, 2 * np * sizeof(BatchReq), hipHostMallocDefault));
        b->host_cap = 2 * np;
    }
    if (b->dev_cap < np * sizeof(BatchReq)) {
        if (b->dev)
            BHIP(b, hipFree(b->dev));
        b->dev = nullptr;
        BHIP(b, hipMalloc(&b->dev, 2 * np * sizeof(BatchReq)));
        b->dev_cap = 2 * np * sizeof(BatchReq);
    }
    // stage: active sets of every request on the batch stream, FP32 first
    uint32_t blocks[2] = {0, 0}, nreq[2] = {0, 0};
    struct Own {  // a request walked by a launch of its own
        WalkArgs A;
        Launch L;
        int32_t opening;
        bool mixed, periodic, tpm;
    };
    std::vector<Own> own;
    std::vector<size_t> order;
    for (int pass = 0; pass < 2; pass++)
        for (size_t k = 0; k < np; k++)
            if ((b->pend[k].c->P.precision == TPM_FP32) == (pass == 0))
                order.push_back(k);
    for (size_t o = 0; o < np; o++) {
        const auto &p = b->pend[order[o]];
        tpm_ctx *c = p.c;
        const int which = c->P.precision == TPM_FP32 ? 0 : 1;
        hipStream_t saved = c->stream;
        c->stream = b->stream;
        Work w;
        int rc = work_of_ctx(c, true, w);
        if (rc == TPM_OK && p.n_act > 0)
            rc = select_active_into(c, p.n_act, p.idx, w);
        c->stream = saved;
        if (rc != TPM_OK)
            return bfail(b, rc, c->err);
        BatchReq &R = b->host[o];
        R = BatchReq{};
        fill_args(c, p.anorm, w, R.A);
        const Variant variant = walk_variant(c, p.n_act, p.opening);
        R.variant = (p.opening == TPM_OPEN_REL ? 1u : 0u) | (c->P.pm_grid > 0 ? 2u : 0u) |
                    ((uint32_t)variant << 5) | (c->P.periodic ? 8u : 0u) |
                    (c->mixed ? 16u : 0u);
        R.first = blocks[which];
        const uint32_t tg = (uint32_t)std::min<int64_t>(p.n_act, c->n);
        set_shares(c, p.n_act, p.opening, variant, R.A);
        const bool split = p.n_act > 0 && variant == kSplitWalk;
        if (split) {  // its own launch, after the staging below
            Launch LA{c->P.precision == TPM_FP32, kSplitWalk, (tg + 3) / 4, 0u, 0u};
            own.push_back({R.A, LA, p.opening, c->mixed != 0, c->P.periodic != 0,
                           c->P.pm_grid > 0});
        }
        if (p.n_act > 0 && !split) {
            const uint32_t wg = batch_waves(which == 0);
            blocks[which] += (walk_waves(variant, tg, R.A.shares) + wg - 1) / wg;
        }
        nreq[which]++;
    }
    BHIP(b, hipMemcpyAsync(b->dev, b->host, np * sizeof(BatchReq), hipMemcpyHostToDevice,
                           b->stream));
    const BatchReq *dreq = (const BatchReq *)b->dev;
    if (blocks[0]) {
        k_walk_batch<true><<<blocks[0], batch_waves(true) * 64, 0, b->stream>>>(dreq, nreq[0]);
        BHIP(b, hipGetLastError());
    }
    if (blocks[1]) {
        k_walk_batch<false><<<blocks[1], batch_waves(false) * 64, 0, b->stream>>>(dreq + nreq[0],
                                                                                  nreq[1]);
        BHIP(b, hipGetLastError());
    }
    for (const Own &o : own) {
        if (o.periodic)
            dispatch_mixed<true, true>(o.A, o.L, o.opening, false, o.mixed, b->stream);
        else if (o.tpm)
            dispatch_mixed<false, true>(o.A, o.L, o.opening, false, o.mixed, b->stream);
        else
            dispatch_mixed<false, false>(o.A, o.L, o.opening, false, o.mixed, b->stream);
        BHIP(b, hipGetLastError());
    }
    // outputs in each request's caller order
    for (size_t o = 0; o < np; o++) {
        const auto &p = b->pend[order[o]];
        if (p.n_act == 0)
            continue;
        tpm_ctx *c = p.c;
        const unsigned ob = grid_for(p.n_act, kBlock);
        if (c->P.precision == TPM_FP32)
            k_output<float><<<ob, kBlock, 0, b->stream>>>(
                p.idx, p.n_act, c->n, (const int32_t *)c->rank.p, (const uint32_t *)c->slot.p,
                (const uint32_t *)c->counters.p + 40, (const float *)c->res.p, (const float *)c->rpot.p, (float *)p.acc, nullptr,
                p.nint, (uint32_t *)c->err_flag.p);
        else
            k_output<double><<<ob, kBlock, 0, b->stream>>>(
                p.idx, p.n_act, c->n, (const int32_t *)c->rank.p, (const uint32_t *)c->slot.p,
                (const uint32_t *)c->counters.p + 40, (const double *)c->res.p, (const double *)c->rpot.p, (double *)p.acc, nullptr,
                p.nint, (uint32_t *)c->err_flag.p);
        BHIP(b, hipGetLastError());
    }
    BHIP(b, hipEventRecord(b->done, b->stream));
    b->launched = true;
    b->pend.clear();
    return TPM_OK;
}

}  // extern "C"
